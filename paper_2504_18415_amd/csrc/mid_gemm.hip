// Mid-size form of the fp6 x fp4 ternary GEMM (INT4 activations): batches of 65 tokens up to where the prefill kernel has
// enough 128 x 128 tiles for the chip.  There the output is too small to give every CU a tile and a CU that walks a long K
// range by itself is bound by the latency of one stage after another, so the K range is cut - over the waves of one
// workgroup, not over workgroups: a workgroup of 2 * KG waves owns 64 features x 64 tokens, K group g takes the K-blocks
// g, g + KG, ... and its two waves one token tile each (two 32 x 32 accumulator tiles per wave).  A pipeline stage is one
// K-block per group: KG x (64 token rows of the record image + two packed weight tiles) = KG x 8 KiB, copied to LDS as
// contiguous 1 KiB pieces.  The groups' accumulators (exact integers) are added through LDS at the end, on the way to
// whole-line stores: no partial tiles in memory and no second launch.
// Bound by the copies' trip through L2 (64 bytes per clock and CU) behind the start-up of the launch.  Whole call, against
// 128 x 128 tiles with K cut over workgroups and a reduction launch (K >= 8192) or uncut: 300 tokens x 8192 -> 3072
// 28.8 -> 19.4 us, 97 x 11008 -> 4096 26.6 -> 17.0, 200 x 8192 -> 2048 21.8 -> 13.4, 65 x 4096 -> 4096 16.3 -> 9.7,
// 512 x 16384 -> 4096 40 -> 37, 4000 x 16384 -> 512 89 -> 79.
#include <atomic>

#include "gemm_common.h"

namespace hbl {
namespace {

using namespace gemm;
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kMidN = 64;                     // features of a workgroup
constexpr int kMidSumRow = kMidN * 4 + 16;    // bytes of a token's sums in the reduction area (padded)

// Bytes of one K-block of a workgroup's tile (TB token tiles of 32): code records, then two packed weight tiles.
constexpr int mid_code_bytes(int tb) { return tb * 32 * kRecordRowBytes; }
constexpr int mid_block_bytes(int tb) { return mid_code_bytes(tb) + (kMidN / 32) * 1024; }

// KG: K groups of two waves, D: stages of LDS, TB: token tiles of 32.  With TB = 2 a wave multiplies both weight tiles by
// token tile `half`; with TB = 1 weight tile `half` by the token tile.
// RAW: the sums leave as int32 [T, N] (acc_out) without dequantisation.
template <int KG, int D, int TB, bool RAW>
__global__ __launch_bounds__(128 * KG) void mid_gemm_f6f4_kernel(const GemmArgs a) {
    constexpr int CODES = mid_code_bytes(TB), BLOCK = mid_block_bytes(TB), STAGE = KG * BLOCK;
    constexpr int BT = 32 * TB;
    constexpr int PIECES = BLOCK / 1024, COPIES = (PIECES + 1) / 2;   // 1 KiB pieces; wave 0 of a group copies COPIES of them
    constexpr int NI = TB;                                            // weight tiles (accumulators) per wave
    static_assert(D >= 2 && D <= 4 && (TB == 1 || TB == 2), "stages / token tiles");
    static_assert(KG * 128 >= BT * 8, "the store needs eight threads per token");
    extern __shared__ __attribute__((aligned(1024))) char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave >> 1, half = wave & 1;

    // workgroups are dealt round-robin over the 8 XCDs: each XCD gets a contiguous run of tiles, ordered so that the larger
    // operand (codes 3/4 T K bytes, weights 1/4 N K) is shared out over the XCDs' L2s and the smaller one read by all
    const int nwg = a.tiles_n * a.tiles_t, xcd = blockIdx.x & 7;
    const int tile = xcd * (nwg >> 3) + (xcd < (nwg & 7) ? xcd : (nwg & 7)) + (blockIdx.x >> 3);
    const bool by_token = 3 * (int64_t)a.T > a.N;
    const int n0 = (by_token ? tile % a.tiles_n : tile / a.tiles_t) * kMidN;
    const int t0 = (by_token ? tile / a.tiles_n : tile % a.tiles_t) * BT;
    const int nkb = a.K / kBK, stages = (nkb + KG - 1) / KG;

    // Copies of this wave: pieces half, half + 2, ... of its group's block (codes first, then weights).  A row tile past N
    // re-reads the last one (never stored); the record image holds whole panels, so rows past T exist.
    const size_t wstride = (size_t)(a.N / 32) * 1024;
    const char* src[COPIES];
    size_t step[COPIES];
#pragma unroll
    for (int m = 0; m < COPIES; ++m) {
        const int piece = 2 * m + half;
        if (piece < CODES / 1024) {
            src[m] = reinterpret_cast<const char*>(a.codes) + (size_t)(t0 / kPanelTokens) * nkb * kRecordBlockBytes +
                     (t0 % kPanelTokens) * kRecordRowBytes + piece * 1024;
            step[m] = kRecordBlockBytes;
        } else {
            int nt = n0 / 32 + piece - CODES / 1024;
            nt = nt < a.N / 32 ? nt : a.N / 32 - 1;
            src[m] = reinterpret_cast<const char*>(a.packed) + (size_t)nt * 1024;
            step[m] = wstride;
        }
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const uint32_t voff = lane * 16;
    auto issue = [&](int s, int slot) {
        int kb = s * KG + group;
        kb = kb < nkb ? kb : nkb - 1;   // a group without a block in the last stage re-reads the last one
#pragma unroll
        for (int m = 0; m < COPIES; ++m)
            if (2 * m + 1 < PIECES || half == 0)
                lds_dma16(lds0 + slot * STAGE + group * BLOCK + (2 * m + half) * 1024, src[m] + kb * step[m], voff);
    };
    // waits until at most `later` (0, 1 or D - 2) stages of this wave's copies are in flight
    auto wait_stage = [&](int later) {
        if (PIECES % 2 == 0 || half == 0) {
            if (later >= D - 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((D - 2) * COPIES) : "memory");
            else if (later == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(COPIES) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        } else {
            if (later >= D - 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((D - 2) * (COPIES - 1)) : "memory");
            else if (later == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(COPIES - 1) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        }
    };

    // what the store needs, requested ahead of the stream: thread -> token tid / 8, features 8 (tid % 8) .. + 7
    const int st = t0 + (tid >> 3), sn = n0 + (tid & 7) * 8;
    const bool stores = tid < BT * 8 && st < a.T && sn < a.N;
    float sd = 0.0f, alpha = 0.0f;
    if (!RAW && stores) {
        sd = a.s_dequant[st];
        alpha = a.w_scales[sn / a.rows_per_group];
    }

#pragma unroll
    for (int s = 0; s < D - 1; ++s)
        if (s < stages) issue(s, s);

    // operand offsets inside the group's block
    const int row = (TB == 2 ? half * 32 : 0) + (lane & 31);
    int xo_lo[2], xo_hi[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        xo_lo[s] = group * BLOCK + row * kRecordRowBytes + record_lo_offset(row, s, lane >> 5);
        xo_hi[s] = group * BLOCK + row * kRecordRowBytes + record_hi_offset(row, s, lane >> 5);
    }
    const int wtile = TB == 2 ? 0 : half;   // first weight tile of this wave
    const int wo = group * BLOCK + CODES + wtile * 1024 + lane * 16;

    v16f acc[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0.0f;

    int slot = 0;
    for (int s = 0; s < stages; ++s) {
        // stage s has landed once at most min(D - 2, stages - 1 - s) later stages of this wave are in flight; after the
        // barrier it is visible to every wave and the buffer of stage s - 1 is free
        wait_stage(stages - 1 - s);
        asm volatile("s_barrier" ::: "memory");
        const char* base = lds + slot * STAGE;
        v4i w[NI];
        v8i x[2];
#pragma unroll
        for (int i = 0; i < NI; ++i) w[i] = *reinterpret_cast<const v4i*>(base + wo + i * 1024);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const v4i lo = *reinterpret_cast<const v4i*>(base + xo_lo[k]);
            const int2 hi = *reinterpret_cast<const int2*>(base + xo_hi[k]);
            x[k] = v8i{lo[0], lo[1], lo[2], lo[3], hi.x, hi.y, 0, 0};
        }
        if (s + D - 1 < stages) issue(s + D - 1, slot == 0 ? D - 1 : slot - 1);
        if (s * KG + group < nkb) {   // uniform
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < NI; ++i)
                    acc[i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                        fp4_operand((uint32_t)w[i][2 * k], (uint32_t)w[i][2 * k + 1]), x[k], acc[i], 4 /*A: fp4*/, 3 /*B: bf6*/,
                        0, 0, 0, 0);
        }
        slot = slot + 1 == D ? 0 : slot + 1;
    }

    // the groups' sums by token row, then eight threads per token add them and store 16 bytes of bf16 each
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wave is done with the stage buffers
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(lds + (group * BT + row) * kMidSumRow + (32 * (wtile + i) + 8 * g + 4 * (lane >> 5)) * 4) =
                make_float4(acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]);
    __syncthreads();
    if (!stores) return;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.0f;
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float4 p = *reinterpret_cast<const float4*>(lds + (g * BT + (tid >> 3)) * kMidSumRow + (tid & 7) * 32 + q * 16);
            v[4 * q] += p.x; v[4 * q + 1] += p.y; v[4 * q + 2] += p.z; v[4 * q + 3] += p.w;
        }
    if constexpr (RAW) {
        v4i* dst = reinterpret_cast<v4i*>(a.acc_out + (size_t)st * a.N + sn);
        dst[0] = v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
        dst[1] = v4i{(int)v[4], (int)v[5], (int)v[6], (int)v[7]};
    } else {
        const uint2 lo = dequant_quad_f32(v[0], v[1], v[2], v[3], sd, alpha), hi = dequant_quad_f32(v[4], v[5], v[6], v[7], sd, alpha);
        store_y16(a.y + (size_t)st * a.N + sn, make_uint4(lo.x, lo.y, hi.x, hi.y));
    }
}

template <int KG, int D, int TB, bool RAW>
int launch_cfg(GemmArgs a, hipStream_t stream) {
    constexpr size_t stages = (size_t)D * KG * mid_block_bytes(TB), sums = (size_t)KG * 32 * TB * kMidSumRow;
    constexpr size_t lds = stages > sums ? stages : sums;
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    a.tiles_n = (a.N + kMidN - 1) / kMidN;
    a.tiles_t = (a.T + 32 * TB - 1) / (32 * TB);
    auto kern = mid_gemm_f6f4_kernel<KG, D, TB, RAW>;
    static std::atomic<uint64_t> lds_allowed{0};   // per instantiation: devices already set up
    if (const int rc = allow_dynamic_lds(kern, lds, lds_allowed); rc != HBL_OK) return rc;
    launch_kernel("mid_gemm_f6f4_kernel", kern, dim3((unsigned)(a.tiles_n * a.tiles_t)), dim3(128 * KG), lds, stream, a);
    return after_launch();
}

// 64 x 64 tiles of the output.  Up to 256 of them one workgroup per CU with three stages of LDS; up to 512 two per CU with
// two stages each (K = 4096, 128 tokens x 12288: 15.4 -> 14.0 us per call; but 300 tokens x 8192 -> 3072, 240 tiles, 19.6 ->
// 23.1 us).  Up to 128 the token tile is halved: half of the chip would idle; and a K range of 64 blocks and more goes to
// eight groups (128 tokens, 16384 -> 4096: 22.0 -> 20.0 us, with four groups 21.5; but at K = 1024 6.6 with four, 7.3 with
// eight).  Above 512 tiles the 128 x 128 tile of the prefill kernel is faster (256 tokens, 4096 -> 12288, 768 tiles:
// 18.0 against 20.5 us).
int64_t mid_tiles(int64_t T, int64_t N) { return ((N + kMidN - 1) / kMidN) * ((T + 63) / 64); }

template <bool RAW>
int launch_form(const GemmArgs& a, hipStream_t stream) {
    const int64_t tiles = mid_tiles(a.T, a.N);
    if (tiles <= 128) return a.K < 8192 ? launch_cfg<4, 4, 1, RAW>(a, stream) : launch_cfg<8, 3, 1, RAW>(a, stream);
    if (tiles <= 256) return launch_cfg<4, 3, 2, RAW>(a, stream);
    return launch_cfg<4, 2, 2, RAW>(a, stream);
}

}  // namespace

namespace gemm {
bool mid_gemm_preferred(int64_t T, int64_t N) { return mid_tiles(T, N) <= 512; }
int launch_mid_gemm_f6f4(const GemmArgs& a, hipStream_t stream) {
    return a.acc_out ? launch_form<true>(a, stream) : launch_form<false>(a, stream);
}
}  // namespace gemm

}  // namespace hbl
