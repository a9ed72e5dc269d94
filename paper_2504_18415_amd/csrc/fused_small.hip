// One-launch form of the forward pass for one to four tokens (INT4 activations, K >= 512, no norm): every workgroup quantises
// the rows for itself and multiplies them by its own output rows.
//
// At a batch of one the two launches of a projection (quantiser, weight streaming) are each little more than a launch: about
// 2.5 us of start-up and drain around 1 to 5 us of work, and HBM idles while one row is transformed on one CU.  Here a
// workgroup requests its whole share of the packed weights (16, 32 or 64 output rows x K) by global->LDS copies first, then
// transforms and quantises the rows with the code of the quantiser launches - the same row in every workgroup, which costs no
// time that the weights do not need anyway - into an image of records in LDS, and multiplies from there.  No workgroup waits
// for another one.
#include "large_rows.h"

namespace hbl {
namespace {

using gemm::fp4_operand;
using gemm::lds_dma16;
using gemm::v4i;
using gemm::v8i;
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kFusedRows = 4;                                // most tokens

struct FusedArgs {
    const void* x;
    const uint32_t* packed;
    const float* w_scales;
    uint16_t* y;
    int T, K, N;
    int rows_per_group;
    float eps;
    uint32_t codes_off, weights_off;   // LDS layout: rows | codes | weights
};

// Waits until at most `n` (rounded down to a multiple of 4) of this wave's copies are in flight.
__device__ __forceinline__ void wait_copies(int n) {
    switch (n >> 2) {   // uniform
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 1: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(20)" ::: "memory"); break;
        case 6: asm volatile("s_waitcnt vmcnt(24)" ::: "memory"); break;
        case 7: asm volatile("s_waitcnt vmcnt(28)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(32)" ::: "memory"); break;
    }
}
// ... of exactly N.
template <int N>
__device__ __forceinline__ void wait_copies() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Waves of a workgroup and log2 of the values per thread of a large row (large_rows.h).  Several rows are worked on side by
// side: plain ones by PW waves each, transformed ones of 512 and 1024 by one wave each, larger ones by K / 1024 (16384: 8).
constexpr int fused_values(int log2k) { return log2k == 14 ? 5 : 4; }
constexpr int fused_row_waves(int log2k, int pw) { return log2k == 0 ? pw : log2k < 11 ? 1 : (1 << log2k) >> (6 + fused_values(log2k)); }
constexpr int fused_waves(int log2k, int pw, int rb) {
    const int n = fused_row_waves(log2k, pw) * rb;
    return n < 4 ? 4 : n;
}

// LOG2K: Hadamard rows of 2^LOG2K (9..14); 0: plain rows of up to 1024 * PW features.  RB: most tokens.  RW: output rows per
// workgroup.
template <int LOG2K, int PW, bool BF16, int RB, int RW>
__global__ __launch_bounds__(64 * fused_waves(LOG2K, PW, RB)) void fused_small_kernel(const FusedArgs a) {
    constexpr int WAVES = fused_waves(LOG2K, PW, RB), R = fused_values(LOG2K);
    constexpr bool LARGE = LOG2K >= 11;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ float s_d[kFusedRows];
    constexpr int EB = BF16 ? 2 : 4;
    constexpr int BLOCK = RB * kRecordRowBytes;              // bytes of a K-block of the record image in LDS
    constexpr int NH = RW / 16;                              // 16-row halves of weight tiles
    constexpr int TILE = RW == 16 ? 512 : RW * 32;           // bytes of weights per K-block
    constexpr int KBU = RW == 16 ? 2 : 1;                    // K-blocks per copy unit (half tiles are copied two at a time)
    constexpr int CPU_ = RW == 64 ? 2 : 1;                   // copies per unit
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = LOG2K ? 1 << LOG2K : a.K;
    const int nkb = K / 128, units = (nkb + KBU - 1) / KBU;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    // 1. the rows' copies: each wave those that its own threads read back below
    constexpr int ROW_WAVES = fused_row_waves(LOG2K, PW), SLOTS = WAVES / ROW_WAVES;
    const int sub = wave / ROW_WAVES;                        // row slot of this wave
    const int row = sub < a.T ? sub : a.T - 1;               // (a slot past the last token repeats that one)
    const uint32_t rtid = tid - sub * ROW_WAVES * 64;
    char* const slot = lds + sub * (LOG2K == 0 ? PW * 1024 * EB : LARGE ? 4 << LOG2K : EB << LOG2K);
    if constexpr (LOG2K == 0) {
        const char* src = static_cast<const char*>(a.x) + (size_t)row * K * EB;
        for (int c = 0; c * PW * 64 < K / 8; ++c) {          // thread rtid reads chunk c * PW * 64 + rtid (8 elements)
            const int first = c * PW * 64 + (wave % ROW_WAVES) * 64;
            if (first >= K / 8) continue;
#pragma unroll
            for (int q = 0; q < EB / 2; ++q) {               // 64 chunks of 16 or 32 bytes; none past the row
                const uint32_t off = q * 1024 + lane * 16;
                const uint32_t most = (uint32_t)(K / 8 - first) * 8 * EB - 16;
                lds_dma16((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)slot + first * 8 * EB + q * 1024,
                          src + (size_t)first * 8 * EB, off < most ? off : most);
            }
        }
    } else if constexpr (!LARGE) {
        const char* src = static_cast<const char*>(a.x) + ((size_t)row * K) * EB;
#pragma unroll
        for (int q = 0; q < (EB << LOG2K) / 1024; ++q)
            lds_dma16((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)slot + q * 1024, src + q * 1024, lane * 16);
    } else {
        large_row_copy<LOG2K, R, BF16>(a.x, row, rtid, slot);
    }

    // 2. this workgroup's weights, unit wave, wave + WAVES, ...; tiles past N re-read the last one (never stored)
    const size_t wstride = (size_t)(a.N / 32) * 1024;
    const int tile0 = RW == 16 ? blockIdx.x >> 1 : blockIdx.x * (RW / 32);
    const int tile_last = a.N / 32 - 1;
    const uint32_t wlds = lds0 + a.weights_off;
    int copies = 0;
    for (int u = wave; u < units; u += WAVES) {
        if constexpr (RW == 16) {
            // lanes 0-31 K-block 2u, lanes 32-63 the next one: of a tile the lanes of rows 16 h .. 16 h + 15, both halves
            const int kb = 2 * u, next = kb + 1 < nkb ? 1 : 0;
            const uint32_t in_tile = (((lane >> 4) & 1) * 32 + 16 * (blockIdx.x & 1) + (lane & 15)) * 16;
            lds_dma16(wlds + u * 1024, reinterpret_cast<const char*>(a.packed) + (size_t)kb * wstride + (size_t)tile0 * 1024,
                      (lane >= 32 && next ? (uint32_t)wstride : 0u) + in_tile);
        } else {
#pragma unroll
            for (int m = 0; m < CPU_; ++m) {
                const int nt = tile0 + m < tile_last ? tile0 + m : tile_last;
                lds_dma16(wlds + u * TILE + m * 1024, reinterpret_cast<const char*>(a.packed) + (size_t)u * wstride + (size_t)nt * 1024, lane * 16);
            }
        }
        copies += CPU_;
    }
    // the rows have landed; the weights may be on their way
    if constexpr (LOG2K != 0 && ((1 << LOG2K) / 128 / KBU) % WAVES == 0) wait_copies<(1 << LOG2K) / 128 / KBU / WAVES * CPU_>();
    else wait_copies(copies < 32 ? copies : 32);

    // 3. transform and quantise into the record image
    int8_t* const codes = reinterpret_cast<int8_t*>(lds + a.codes_off);
    const RowParams rp{a.eps, nullptr, 0.0f, 1};
    if constexpr (LOG2K == 0) {
        if (K > 512 * PW)   // uniform
            quant_generic_body<4, BF16, 2, BLOCK, PW, SLOTS>(0, rtid, slot, K, codes + row * kRecordRowBytes, s_d + row, nullptr, rp, kCodesBf6, sub);
        else
            quant_generic_body<4, BF16, 1, BLOCK, PW, SLOTS>(0, rtid, slot, K, codes + row * kRecordRowBytes, s_d + row, nullptr, rp, kCodesBf6, sub);
    } else if constexpr (!LARGE) {
        fwht_quant_body<LOG2K, 1, 4, BF16, true, BLOCK>(0, rtid, slot, codes + row * kRecordRowBytes, s_d + row, nullptr, rp, kCodesBf6);
    } else {
        LargeRowRaw<R, BF16> raw;
        large_row_read<LOG2K, R, BF16>(rtid, slot, raw);
        large_row_body<LOG2K, R, 4, BF16, true, false, BLOCK, SLOTS>(
            0, rtid, raw, reinterpret_cast<float*>(slot), codes + row * kRecordRowBytes, s_d + row, nullptr, rp, 8, sub);
    }
    __syncthreads();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // a wave multiplies the weights that it copied itself

    // 4. 16x16x128 MFMAs: lane = (token lane & 15, feature group g = lane >> 4 of 32)
    const int g = lane >> 4, r = lane & 15;
    const int tok = r < a.T ? r : 0;
    const char* crow = lds + a.codes_off + tok * kRecordRowBytes;
    const int lo_off = record_lo_offset(tok, g >> 1, g & 1), hi_off = record_hi_offset(tok, g >> 1, g & 1);
    v4f acc[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) acc[h] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    for (int u = wave; u < units; u += WAVES)
#pragma unroll
        for (int k = 0; k < KBU; ++k) {
            const int kb = u * KBU + k;
            if (KBU > 1 && kb >= nkb) break;   // uniform
            const v4i lo = *reinterpret_cast<const v4i*>(crow + kb * BLOCK + lo_off);
            const int2 hi = *reinterpret_cast<const int2*>(crow + kb * BLOCK + hi_off);
            const v8i xop = {lo[0], lo[1], lo[2], lo[3], hi.x, hi.y, 0, 0};
            const char* w = lds + a.weights_off + (size_t)kb * TILE;
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const uint2 wp = RW == 16 ? *reinterpret_cast<const uint2*>(w + ((g & 1) * 16 + r) * 16 + 8 * (g >> 1))
                                          : *reinterpret_cast<const uint2*>(w + (h >> 1) * 1024 + ((g & 1) * 32 + 16 * (h & 1) + r) * 16 + 8 * (g >> 1));
                acc[h] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fp4_operand(wp.x, wp.y), xop, acc[h], 4 /*A: fp4*/,
                                                                          3 /*B: bf6*/, 0, 0, 0, 0);
            }
        }

    // 5. the waves' sums (exact integers) through LDS, then bf16: wave 0 holds 4 features of token lane & 15 per half
    __syncthreads();
    v4f* red = reinterpret_cast<v4f*>(lds);
    if (wave != 0) {
#pragma unroll
        for (int h = 0; h < NH; ++h) red[((wave - 1) * NH + h) * 64 + lane] = acc[h];
    }
    __syncthreads();
    if (wave != 0 || r >= a.T) return;
    const float sd = s_d[r];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        v4f v = acc[h];
#pragma unroll
        for (int w = 0; w < WAVES - 1; ++w) v += red[(w * NH + h) * 64 + lane];
        const int n0 = RW == 16 ? blockIdx.x * 16 : blockIdx.x * RW + h * 16;
        if (n0 < a.N)
            *reinterpret_cast<uint2*>(a.y + (size_t)r * a.N + n0 + 4 * g) =
                gemm::dequant_quad_f32(v[0], v[1], v[2], v[3], sd, a.w_scales[n0 / a.rows_per_group]);
    }
}

constexpr size_t kCuLds = 160 * 1024;

// LDS of a workgroup: rows (the transform's row buffers, or the rows as loaded), record image, weights; the sums reuse it.
struct FusedLayout {
    size_t codes_off, weights_off, bytes;
};
FusedLayout fused_layout(int log2k, int pw, int eb, int rb, int64_t K, int rw) {
    FusedLayout l;
    const int waves = fused_waves(log2k, pw, rb);
    const size_t slots = waves / fused_row_waves(log2k, pw);
    const size_t rows = slots * (log2k == 0 ? (size_t)pw * 1024 * eb : log2k < 11 ? (size_t)K * eb : (size_t)K * sizeof(float));
    const size_t nkb = (size_t)K / 128, per = rw == 16 ? 512 : (size_t)rw * 32;
    l.codes_off = round_up(rows, 1024);
    l.weights_off = l.codes_off + round_up(nkb * rb * kRecordRowBytes, 1024);
    l.bytes = l.weights_off + (nkb + (rw == 16 ? nkb & 1 : 0)) * per;
    const size_t sums = (size_t)(waves - 1) * (rw / 16) * 1024;
    if (l.bytes < sums) l.bytes = sums;
    return l;
}

template <int LOG2K, int PW, bool BF16, int RB, int RW>
int launch_cfg(FusedArgs a, const FusedLayout& l, hipStream_t stream) {
    a.codes_off = (uint32_t)l.codes_off;
    a.weights_off = (uint32_t)l.weights_off;
    constexpr auto kern = fused_small_kernel<LOG2K, PW, BF16, RB, RW>;
    if (const int rc = allow_dynamic_lds<kern, kCuLds - 1024>(); rc != HBL_OK) return rc;
    launch_kernel("fused_small_kernel", kern, dim3((unsigned)((a.N + RW - 1) / RW)), dim3(64 * fused_waves(LOG2K, PW, RB)), l.bytes, stream, a);
    return after_launch();
}

// Most workgroups per CU at which one launch is no slower than two, for 16, 32 and 64 output rows a workgroup; 0: not at all.
// Every workgroup quantises the rows for itself, so beyond one per CU that work is repeated side by side on the same SIMDs,
// while the two launches do it once: what is saved, a launch of about 2 us, is spent again.  Time against the two launches
// (bf16 rows, 256 to 32768 output rows; fp32 within 0.03):
//   16 rows, at most one per CU: 0.56-0.85 for one and two tokens, 0.61-0.85 for three, 0.61-0.97 for four
//   between one and two per CU 32 rows are as good or better: 1 x 8192 -> 8192 0.72 (16 rows: 0.91), 2 x 2048 -> 12288 0.80
//     (0.87), 3 x 2048 -> 8192 0.76 (0.90), 4 plain x 2048 -> 8192 0.81 (0.99)
//   32 rows per CU, transformed:  K = 512  3: 0.83  4: 0.95;  1024  3: 0.92  4: 1.10;  2048  one or two tokens 3: 0.97  4: 1.12, three
//     2: 0.97  3: 1.09, four 1: 0.81  1.5: 0.97-1.18;  4096  one token 3: 0.94, two 1: 0.78  1.5: 0.97, three 1: 0.91, four 1: 1.02;
//     8192  1: 0.72-0.96
//   32 rows, plain:  one token 3: 0.78-0.87 and 4: 0.83-0.99 (64 rows: 0.79-0.94);  two tokens 1: 0.66-0.80  1.5: 0.76-0.92 (64 rows:
//     0.75-0.91);  three 1: 0.70-0.89  2: 0.92-1.04 (512: 1.12);  four 1: 0.81-0.91  1.5: 1.04-1.20
//   one plain token beyond 4096:  up to 8192 features by eight waves, 16 rows 1: 0.50-0.56, 32 rows 1: 0.49-0.63  2: 0.60-0.77 (two of
//     16 waves do not share a CU: 1 x 4224 -> 16384 6.6 us with them, 5.4 by eight, 8.9 by two launches);  above, 16 rows 1: 0.49-0.58
//     2 (bf16 rows of at most 9728 have room for two): 0.83-0.92
//   64 rows, plain:  two tokens 1: 0.75-0.91  2: 0.88-0.98 (512: 1.07);  three 1.5: 1.09-1.32;  four 1: 1.06-1.31
// Four plain rows of at most 512 features (0.89-0.95), and 32 rows for four of at most 1024 (0.82-0.87), are left to the two
// launches: less than a microsecond, and more than one workgroup per CU is a loss from there on.
// (1 x 4096 -> 4096 transformed 6.3 us by two launches, 4.3 by one; 1 x 16384 -> 4096 9.9 and 7.5; 4 x 2048 -> 2048 6.3 and 4.6.)
int most_workgroups_per_cu(int64_t T, int64_t K, bool hadamard, int rw) {
    if (rw == 16) return T == 1 && !hadamard && K > 8192 ? 2 : (hadamard || T < 4 || K > 512 ? 1 : 0);
    if (rw == 64) return T == 1 ? 4 : (T == 2 ? (K < 1024 ? 1 : 2) : 0);   // (plain rows only)
    if (!hadamard) {
        if (T == 1) return K <= 4096 ? 3 : 2;
        if (T == 3) return K >= 1024 ? 2 : 1;
        return T == 2 || K > 1024 ? 1 : 0;
    }
    if (K <= 1024) return K <= 512 ? 4 : 3;
    if (K <= 2048) return T <= 2 ? 3 : (T == 3 ? 2 : 1);
    if (K <= 4096) return T == 1 ? 3 : (T <= 3 ? 1 : 0);
    return 1;
}

struct FusedPlan {
    int log2k, pw, rb, rw;   // rw = 0: not this kernel
    FusedLayout layout;
};
FusedPlan fused_plan(int64_t T, int64_t K, int64_t N, int x_dtype, bool hadamard) {
    FusedPlan p = {};
    const int eb = x_dtype == HBL_BF16 ? 2 : 4;
    if (hadamard) {
        while ((1 << p.log2k) < K) ++p.log2k;
    } else {
        p.pw = K <= 4096 ? 4 : K <= 8192 ? 8 : 16;
    }
    if (T > kFusedRows || (T > 1 && K > (hadamard && T == 2 ? 8192 : 4096))) return p;
    p.rb = T == 1 ? 1 : (fused_row_waves(p.log2k, p.pw) > 1 ? (int)T : kFusedRows);
    for (const int rw : {16, 32, 64}) {
        if ((rw == 64 && (hadamard || K > 4096)) || (rw == 32 && K > 8192)) continue;
        const FusedLayout l = fused_layout(p.log2k, p.pw, eb, p.rb, K, rw);
        if (l.bytes > kCuLds - 1024) continue;
        const int64_t wgs = (N + rw - 1) / rw, resident = (int64_t)(kCuLds / (l.bytes + 1024));
        const int64_t most = most_workgroups_per_cu(T, K, hadamard, rw);
        if (wgs > 256 * (resident < most ? resident : most)) continue;
        p.rw = rw;
        p.layout = l;
        break;
    }
    return p;
}

template <int LOG2K, int PW, bool BF16, int RB>
int launch_rows(const FusedArgs& a, const FusedPlan& p, hipStream_t stream) {
    if (p.rw == 16) return launch_cfg<LOG2K, PW, BF16, RB, 16>(a, p.layout, stream);
    if constexpr (LOG2K < 14) {
        if (p.rw == 32) return launch_cfg<LOG2K, PW, BF16, RB, 32>(a, p.layout, stream);
    }
    if constexpr (LOG2K == 0 && PW == 4) {
        if (p.rw == 64) return launch_cfg<LOG2K, PW, BF16, RB, 64>(a, p.layout, stream);
    }
    return HBL_E_SHAPE;
}
template <int LOG2K, int PW, bool BF16>
int launch_tokens(const FusedArgs& a, const FusedPlan& p, hipStream_t stream) {
    if constexpr (PW == 4 || (LOG2K >= 11 && LOG2K <= 13)) {
        if (p.rb == 2) return launch_rows<LOG2K, PW, BF16, 2>(a, p, stream);
    }
    if constexpr (PW == 4 || LOG2K == 11 || LOG2K == 12) {
        if (p.rb == 3) return launch_rows<LOG2K, PW, BF16, 3>(a, p, stream);
    }
    if constexpr (LOG2K < 13 && PW < 16) {
        if (p.rb == kFusedRows) return launch_rows<LOG2K, PW, BF16, kFusedRows>(a, p, stream);
    }
    return p.rb == 1 ? launch_rows<LOG2K, PW, BF16, 1>(a, p, stream) : HBL_E_SHAPE;
}

template <bool BF16>
int launch_kind(const FusedArgs& a, const FusedPlan& p, hipStream_t stream) {
    switch (p.log2k) {
        case 0:
            if (p.pw == 8) return launch_rows<0, 8, BF16, 1>(a, p, stream);
            return p.pw == 4 ? launch_tokens<0, 4, BF16>(a, p, stream) : launch_tokens<0, 16, BF16>(a, p, stream);
        case 9: return launch_tokens<9, 0, BF16>(a, p, stream);
        case 10: return launch_tokens<10, 0, BF16>(a, p, stream);
        case 11: return launch_tokens<11, 0, BF16>(a, p, stream);
        case 12: return launch_tokens<12, 0, BF16>(a, p, stream);
        case 13: return launch_tokens<13, 0, BF16>(a, p, stream);
        case 14: return launch_tokens<14, 0, BF16>(a, p, stream);
        default: return HBL_E_SHAPE;
    }
}

}  // namespace

bool fused_small_preferred(int64_t T, int64_t K, int64_t N, int x_dtype, int bits, bool hadamard) {
    return bits == 4 && K >= 512 && T >= 1 && fused_plan(T, K, N, x_dtype, hadamard).rw != 0;
}

int launch_fused_small(const void* x, int x_dtype, int64_t T, int64_t K, const void* packed, int64_t N, const float* w_scales,
                       int64_t groups, float eps, bool hadamard, void* y, hipStream_t stream) {
    const FusedPlan p = fused_plan(T, K, N, x_dtype, hadamard);
    if (p.rw == 0) return HBL_E_SHAPE;
    FusedArgs a = {};
    a.x = x;
    a.packed = static_cast<const uint32_t*>(packed);
    a.w_scales = w_scales;
    a.y = static_cast<uint16_t*>(y);
    a.T = (int)T;
    a.K = (int)K;
    a.N = (int)N;
    a.rows_per_group = (int)(N / groups);
    a.eps = eps;
    return x_dtype == HBL_BF16 ? launch_kind<true>(a, p, stream) : launch_kind<false>(a, p, stream);
}

}  // namespace hbl
