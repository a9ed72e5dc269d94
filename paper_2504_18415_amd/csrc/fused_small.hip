// One-launch form of the forward pass for one to four tokens (INT4 activations, K >= 512, no norm): every workgroup quantises
// the rows for itself and multiplies them by its own output rows.
//
// At a batch of one the two launches of a projection (quantiser, weight streaming) are each little more than a launch: about
// 2.5 us of start-up and drain around 1 to 5 us of work, and HBM idles while one row is transformed on one CU.  Here a
// workgroup requests its whole share of the packed weights (16, 32 or 64 output rows x K) by global->LDS copies first, then
// transforms and quantises the rows with the code of the quantiser launches - the same row in every workgroup, which costs no
// time that the weights do not need anyway - into an image of records in LDS, and multiplies from there.  No workgroup waits
// for another one.
#include <atomic>

#include "quant_bodies.h"

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

// LOG2K: Hadamard rows of 2^LOG2K (9..14); 0: plain rows of up to 2048 * MAXC.  RB: most tokens.  RW: output rows per
// workgroup.
template <int LOG2K, int MAXC, bool BF16, int RB, int RW>
__global__ __launch_bounds__(256) void fused_small_kernel(const FusedArgs a) {
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
    constexpr int ROW_WAVES = LOG2K == 0 ? 4 : (LOG2K <= 12 ? 1 : (LOG2K == 13 ? 2 : 4));   // waves that share a row
    const int sub = wave / ROW_WAVES;                        // Hadamard: row slot of this wave
    const int row = sub < a.T ? sub : a.T - 1;               // (a slot past the last token repeats that one)
    const uint32_t rtid = tid - sub * ROW_WAVES * 64;
    char* const slot = lds + (LOG2K >= 12 ? sub * (4 << LOG2K) : sub * (EB << (LOG2K ? LOG2K : 9)));
    if constexpr (LOG2K == 0) {
        for (int t = 0; t < a.T; ++t)
            for (int c = 0; c * 256 < K / 8; ++c) {          // thread tid reads chunk c * 256 + tid (8 elements)
                const int first = c * 256 + wave * 64;
                if (first >= K / 8) continue;
                const char* src = static_cast<const char*>(a.x) + ((size_t)t * K + (size_t)first * 8) * EB;
#pragma unroll
                for (int q = 0; q < EB / 2; ++q) {           // 64 chunks of 16 or 32 bytes; none past the row
                    const uint32_t off = q * 1024 + lane * 16;
                    const uint32_t most = (uint32_t)(K / 8 - first) * 8 * EB - 16;
                    lds_dma16(lds0 + (t * (MAXC * 2048) + first * 8) * EB + q * 1024, src, off < most ? off : most);
                }
            }
    } else if constexpr (LOG2K < 12) {
        const char* src = static_cast<const char*>(a.x) + ((size_t)row * K) * EB;
#pragma unroll
        for (int q = 0; q < (EB << LOG2K) / 1024; ++q)
            lds_dma16((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)slot + q * 1024, src + q * 1024, lane * 16);
    } else {
        bigrow_copy<LOG2K, BF16>(a.x, row, rtid, slot);
    }

    // 2. this workgroup's weights, unit wave, wave + 4, ...; tiles past N re-read the last one (never stored)
    const size_t wstride = (size_t)(a.N / 32) * 1024;
    const int tile0 = RW == 16 ? blockIdx.x >> 1 : blockIdx.x * (RW / 32);
    const int tile_last = a.N / 32 - 1;
    const uint32_t wlds = lds0 + a.weights_off;
    int copies = 0;
    for (int u = wave; u < units; u += 4) {
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
    wait_copies(copies < 32 ? copies : 32);   // the rows have landed; the weights may be on their way

    // 3. transform and quantise into the record image
    int8_t* const codes = reinterpret_cast<int8_t*>(lds + a.codes_off);
    const RowParams rp{a.eps, nullptr, 0.0f, 1};
    if constexpr (LOG2K == 0) {
        for (int t = 0; t < a.T; ++t) {
            if (t != 0) __syncthreads();   // every wave is done with the previous row's partial sums
            quant_generic_body<4, BF16, MAXC, BLOCK>(0, tid, lds + t * (MAXC * 2048) * EB, K, codes + t * kRecordRowBytes, s_d + t,
                                                     nullptr, rp, kCodesBf6);
        }
    } else if constexpr (LOG2K < 12) {
        fwht_quant_body<LOG2K, 1, 4, BF16, true, BLOCK>(0, rtid, slot, codes + row * kRecordRowBytes, s_d + row, nullptr, rp, kCodesBf6);
    } else {
        BigRowRaw<BF16> raw;
        bigrow_read<LOG2K, BF16>(rtid, slot, raw);
        fwht_quant_bigrow_body<LOG2K, 4, BF16, true, false, false, BLOCK>(
            0, rtid, raw, reinterpret_cast<float*>(slot), codes + row * kRecordRowBytes, s_d + row, nullptr, rp, 8);
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
    for (int u = wave; u < units; u += 4)
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

    // 5. the four waves' sums (exact integers) through LDS, then bf16: wave 0 holds 4 features of token lane & 15 per half
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
        for (int w = 0; w < 3; ++w) v += red[(w * NH + h) * 64 + lane];
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
FusedLayout fused_layout(int log2k, int maxc, int eb, int T, int rb, int64_t K, int rw) {
    FusedLayout l;
    size_t rows;
    if (log2k == 0) rows = (size_t)T * maxc * 2048 * eb;
    else if (log2k < 12) rows = (size_t)4 * K * eb;                                  // four row slots, as loaded
    else rows = (size_t)(log2k == 12 ? 4 : log2k == 13 ? 2 : 1) * K * sizeof(float); // row slots of K floats
    const size_t nkb = (size_t)K / 128, per = rw == 16 ? 512 : (size_t)rw * 32;
    l.codes_off = round_up(rows, 1024);
    l.weights_off = l.codes_off + round_up(nkb * rb * kRecordRowBytes, 1024);
    l.bytes = l.weights_off + (nkb + (rw == 16 ? nkb & 1 : 0)) * per;
    const size_t sums = (size_t)3 * (rw / 16) * 1024;
    if (l.bytes < sums) l.bytes = sums;
    return l;
}

template <int LOG2K, int MAXC, bool BF16, int RB, int RW>
int launch_cfg(FusedArgs a, const FusedLayout& l, hipStream_t stream) {
    a.codes_off = (uint32_t)l.codes_off;
    a.weights_off = (uint32_t)l.weights_off;
    auto kern = fused_small_kernel<LOG2K, MAXC, BF16, RB, RW>;
    static std::atomic<uint64_t> lds_allowed{0};   // per instantiation: devices already set up
    if (const int rc = allow_dynamic_lds(kern, kCuLds - 1024, lds_allowed); rc != HBL_OK) return rc;
    launch_kernel("fused_small_kernel", kern, dim3((unsigned)((a.N + RW - 1) / RW)), dim3(256), l.bytes, stream, a);
    return after_launch();
}

// Most workgroups per CU at which one launch is no slower than two, for 16, 32 and 64 output rows a workgroup; 0: not at all.
// Every workgroup quantises the rows for itself, so beyond one per CU that work is repeated side by side on the same SIMDs,
// while the two launches do it once: what is saved, a launch of about 2 us, is spent again.  Time against the two launches
// (both input types, 32 to 131072 output rows; by workgroups of 16 rows per CU):
//   transformed rows: K = 512  1: 0.6  2: 0.7  4: 0.87  6: 1.02  8: 1.2;  1024  1: 0.6  3: 0.8  4: 0.94  5: 1.07  8: 1.4;
//                     2048  1: 0.7  2: 0.85  3: 0.97  4: 1.17;  4096 and more  1: 0.75-0.85, LDS holds no more than two
//   plain rows, one token: 512  1: 0.7  4: 0.84  8: 1.07;  1024 to 4096  1: 0.55  4: 0.8
//   plain rows of several tokens are taken one after the other by the whole workgroup, whatever their length:
//                     2 tokens, 512  1: 0.85  3: 0.99  4: 1.07;  2048  1: 0.7  3: 0.87  4: 0.99
//                     3 tokens, 512  1: 0.95-1.02  2: 1.08;  1024  1: 0.85  2: 0.98  3: 1.07;  2560  1: 0.93  2: 1.02
//                     4 tokens, 512  1: 1.1;  1024  1: 0.97  2: 1.12;  1536  1: 0.93  2: 1.04;  2048  1: 0.95  2: 1.07
// 32 and 64 rows a workgroup start 0.05 and 0.1 higher (fewer wavefronts, longer sums) and rise in the same way.
// (us: 4 x 512 -> 12288 plain 7.0 by one launch, 5.1 by two; 1 x 1024 -> 32768 transformed 8.8, 6.4; 1 x 2048 -> 16384
// transformed 9.3 with 16 rows a workgroup, 7.0 with 32, 7.9 by two.)
int most_workgroups_per_cu(int64_t T, int64_t K, bool hadamard, int rw) {
    if (hadamard) return K <= 512 ? 4 : (K <= 1024 ? 3 : 2);
    if (T == 1) return 4;
    if (T == 2) return rw == 16 ? 3 : (K >= 1024 ? (rw == 32 ? 3 : 2) : (rw == 32 ? 2 : 1));
    if (T == 3) {
        if (rw == 16) return K >= 1024 && K <= 2048 ? 2 : 1;
        return rw == 64 || K < 640 ? 0 : (K >= 1280 && K <= 2048 ? 2 : 1);
    }
    return rw == 64 ? 0 : (K >= (rw == 16 ? 1024 : 1536) ? 1 : 0);
}

struct FusedPlan {
    int log2k, maxc, rb, rw;   // rw = 0: not this kernel
    FusedLayout layout;
};
FusedPlan fused_plan(int64_t T, int64_t K, int64_t N, int x_dtype, bool hadamard) {
    FusedPlan p = {};
    const int eb = x_dtype == HBL_BF16 ? 2 : 4;
    if (hadamard) {
        while ((1 << p.log2k) < K) ++p.log2k;
    } else {
        p.maxc = K <= 4096 ? 2 : 8;
    }
    // the rows of K <= 4096 are transformed side by side, one per wave; larger and plain ones take the whole workgroup in turn
    if (T > kFusedRows || (T > 1 && (hadamard ? K >= 8192 : T * K > 8192))) return p;
    p.rb = T == 1 ? 1 : kFusedRows;
    for (const int rw : {16, 32, 64}) {
        if ((rw == 64 && (hadamard || K > 4096)) || (rw == 32 && K > 8192)) continue;
        const FusedLayout l = fused_layout(p.log2k, p.maxc, eb, (int)T, p.rb, K, rw);
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

template <int LOG2K, int MAXC, bool BF16, int RB>
int launch_rows(const FusedArgs& a, const FusedPlan& p, hipStream_t stream) {
    if (p.rw == 16) return launch_cfg<LOG2K, MAXC, BF16, RB, 16>(a, p.layout, stream);
    if constexpr (LOG2K < 14) {
        if (p.rw == 32) return launch_cfg<LOG2K, MAXC, BF16, RB, 32>(a, p.layout, stream);
    }
    if constexpr (LOG2K == 0 && MAXC == 2) {
        if (p.rw == 64) return launch_cfg<LOG2K, MAXC, BF16, RB, 64>(a, p.layout, stream);
    }
    return HBL_E_SHAPE;
}
template <int LOG2K, int MAXC, bool BF16>
int launch_tokens(const FusedArgs& a, const FusedPlan& p, hipStream_t stream) {
    if constexpr (LOG2K < 13 && MAXC < 8) {
        if (p.rb != 1) return launch_rows<LOG2K, MAXC, BF16, kFusedRows>(a, p, stream);
    }
    return p.rb == 1 ? launch_rows<LOG2K, MAXC, BF16, 1>(a, p, stream) : HBL_E_SHAPE;
}

template <bool BF16>
int launch_kind(const FusedArgs& a, const FusedPlan& p, hipStream_t stream) {
    switch (p.log2k) {
        case 0: return p.maxc == 2 ? launch_tokens<0, 2, BF16>(a, p, stream) : launch_tokens<0, 8, BF16>(a, p, stream);
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
