// Mid-size form of the ternary GEMM, on both operand paths (code records for the fp6 x fp4 matrix cores; bytes for the int8
// ones: INT8 activations, rows shorter than 512): batches of 17 tokens up to where the prefill kernels have enough 128 x 128
// tiles for the chip, and smaller ones where the weight-streaming kernel has few workgroups with long chains.
// There the output is too small to give every CU a tile and a CU that walks a long K range by itself is bound by the latency
// of one stage after another, so the K range is cut - over the waves of one workgroup, not over workgroups: K group g of KG
// takes the K-blocks g, g + KG, ...  A pipeline stage is one K-block per group (code rows and packed weight tiles), copied to
// LDS in 1 KiB pieces.  The groups' accumulators (exact integers) are added through LDS at the end, on the way to whole-line
// stores: no partial tiles in memory and no second launch.
// Bound by the copies' trip through L2 and LDS (64 / 128 bytes per clock and CU) behind the start-up of the launch.  Whole
// call, both launches (transformed where K is a power of two), against what it replaced: 128 x 128 tiles above 64 tokens, with
// K >= 8192 cut over workgroups and a reduction launch: 300 tokens x 8192 -> 3072 27.9 -> 18.2 us, 97 x 11008 -> 4096 25.6 ->
// 15.8, 200 x 8192 -> 2048 23.8 -> 15.2, 65 x 4096 -> 4096 17.4 -> 10.7, 512 x 16384 -> 4096 45.5 -> 42.2, 4000 x 16384 -> 512
// 95.8 -> 84.1.  The shared form of the weight-streaming kernel up to 64: 64 x 16384 -> 4096 23.6 -> 15.1, 64 x 11008 -> 4096
// 22.6 -> 11.9, 17 x 4096 -> 4096 12.0 -> 8.9, 32 x 4096 -> 32768 14.9 -> 13.4 (beyond that many rows: decode_shared_preferred).
// INT8 activations: 64 x 16384 -> 4096 24.4 -> 16.9, 24 x 8192 -> 3072 15.2 -> 11.2, 97 x 11008 -> 4096 33.7 -> 16.8, 128 x
// 4096 -> 4096 24.4 -> 11.9, 300 x 8192 -> 3072 34.9 -> 22.1 us.
#include <type_traits>

#include "gemm_common.h"

namespace hbl {
namespace {

using namespace gemm;
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// A form: KG K groups of NF waves, D stages of LDS, NF feature tiles and TB token tiles of 32.  TB = 1: each wave of a group
// multiplies one weight tile by the token tile.  TB = 2, records: waves 2p, 2p + 1 multiply weight tiles 2p and 2p + 1 by one
// token tile each (fewer LDS operand bytes); bytes (I8): a wave multiplies one weight tile by both token tiles (the weights'
// expansion is the larger cost there).
template <int KG_, int D_, int NF_, int TB_, bool I8_ = false>
struct MidForm {
    static constexpr int KG = KG_, D = D_, NF = NF_, TB = TB_;
    static constexpr bool I8 = I8_;
    static constexpr int BN = 32 * NF, BT = 32 * TB;
    static constexpr int WI = TB == 2 && !I8 ? 2 : 1;            // weight tiles and ...
    static constexpr int TI = I8 ? TB : 1;                       // ... token tiles of a wave
    static constexpr int NI = WI * TI;                           // 32 x 32 accumulator tiles per wave
    static constexpr int GW = NF * TB / NI;                      // waves per group
    static constexpr int THREADS = 64 * GW * KG;
    static constexpr int CODES = BT * (I8 ? kBK : kRecordRowBytes);   // bytes of a K-block: codes, then weight tiles
    static constexpr int BLOCK = CODES + NF * 1024;
    static constexpr int STAGE = KG * BLOCK;
    static constexpr int PIECES = BLOCK / 1024;                  // 1 KiB copies per group and stage
    static constexpr int COPIES = (PIECES + GW - 1) / GW;        // ... of wave 0 of the group
    static constexpr int SUMROW = BN * 4 + 16;                   // bytes of a token's sums in the reduction area (padded)
    static constexpr int TPT = BN / 8;                           // threads per token at the store (8 features each)
    static constexpr size_t STAGES_LDS = (size_t)D * STAGE, SUMS_LDS = (size_t)KG * BT * SUMROW;
    static constexpr size_t LDS = STAGES_LDS > SUMS_LDS ? STAGES_LDS : SUMS_LDS;
    static_assert(D >= 2 && D <= 4 && (NF == 1 || NF == 2 || NF == 4) && (TB == 1 || TB == 2 || (TB == 4 && I8)) && TB <= NF && LDS <= 160 * 1024, "form");
    static constexpr int STORES = (BT * TPT + THREADS - 1) / THREADS;   // 16-byte stores per thread
    static int64_t tiles_n(int64_t N) { return (N + BN - 1) / BN; }
    static int64_t tiles_t(int64_t T) { return (T + BT - 1) / BT; }
};

// Workgroup `wg` of the problem.  RAW: the sums leave as int32 [T, N] (acc_out) without dequantisation.
template <typename F, bool RAW>
__device__ __forceinline__ void mid_gemm_body(const MidProblem& a, int wg, char* lds) {
    constexpr int KG = F::KG, D = F::D, TB = F::TB, BT = F::BT, CODES = F::CODES, BLOCK = F::BLOCK, STAGE = F::STAGE;
    constexpr int GW = F::GW, PIECES = F::PIECES, COPIES = F::COPIES, NI = F::NI, SUMROW = F::SUMROW, TPT = F::TPT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave / GW, half = wave % GW;

    // workgroups are dealt round-robin over the 8 XCDs: each XCD gets a contiguous run of tiles, ordered so that the larger
    // operand (codes 3/4 T K or T K bytes, weights 1/4 N K) is shared out over the XCDs' L2s and the smaller one read by all
    const int nwg = a.tiles_n * a.tiles_t, xcd = wg & 7;
    const int tile = xcd * (nwg >> 3) + (xcd < (nwg & 7) ? xcd : (nwg & 7)) + (wg >> 3);
    const bool by_token = (F::I8 ? 4 : 3) * (int64_t)a.T > a.N;
    const int n0 = (by_token ? tile % a.tiles_n : tile / a.tiles_t) * F::BN;
    const int t0 = (by_token ? tile / a.tiles_n : tile % a.tiles_t) * BT;
    const int nkb = a.K / kBK, stages = (nkb + KG - 1) / KG;

    // Copies of this wave: pieces half, half + GW, ... of its group's block (codes first, then weights).  A row tile past N
    // re-reads the last one (never stored); the record image holds whole panels, so rows past T exist.  Bytes: piece q is
    // token rows 8q .. 8q + 7, lane l -> row 8q + l/8, LDS slot l%8 of the row, 16-byte chunk (l%8) ^ ((row/2) % 8); rows past
    // T re-read the last one.
    const size_t wstride = (size_t)(a.N / 32) * 1024;
    const char* src[COPIES];
    size_t step[COPIES];
    uint32_t voff[COPIES];
#pragma unroll
    for (int m = 0; m < COPIES; ++m) {
        const int piece = GW * m + half;
        voff[m] = lane * 16;
        if (piece < CODES / 1024 && F::I8) {
            const int r = 8 * piece + (lane >> 3), t = t0 + r < a.T ? r : a.T - 1 - t0;
            src[m] = reinterpret_cast<const char*>(a.codes) + (size_t)t0 * a.K;
            step[m] = kBK;
            voff[m] = (uint32_t)t * (uint32_t)a.K + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
        } else if (piece < CODES / 1024) {
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
    auto issue = [&](int s, int slot) {
        int kb = s * KG + group;
        kb = kb < nkb ? kb : nkb - 1;   // a group without a block in the last stage re-reads the last one
#pragma unroll
        for (int m = 0; m < COPIES; ++m)
            if (GW * m + GW - 1 < PIECES || half < PIECES % GW)
                lds_dma16(lds0 + slot * STAGE + group * BLOCK + (GW * m + half) * 1024, src[m] + kb * step[m], voff[m]);
    };
    // waits until at most `later` (0, 1 or D - 2) stages of this wave's copies are in flight
    auto wait_stage = [&](int later) {
        if (PIECES % GW == 0 || half < PIECES % GW) {
            if (later >= D - 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((D - 2) * COPIES) : "memory");
            else if (later == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(COPIES) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        } else {
            if (later >= D - 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((D - 2) * (COPIES - 1)) : "memory");
            else if (later == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(COPIES - 1) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        }
    };

    // what the stores need, requested ahead of the stream: unit u -> token u / TPT, features 8 (u % TPT) .. + 7
    float sd[F::STORES], alpha[F::STORES];
    auto unit_token = [&](int i) { return t0 + (tid + i * F::THREADS) / TPT; };
    auto unit_feature = [&](int i) { return n0 + ((tid + i * F::THREADS) % TPT) * 8; };
    auto unit_stores = [&](int i) { return tid + i * F::THREADS < BT * TPT && unit_token(i) < a.T && unit_feature(i) < a.N; };
#pragma unroll
    for (int i = 0; i < F::STORES; ++i) {
        sd[i] = alpha[i] = 0.0f;
        if (!RAW && unit_stores(i)) {
            sd[i] = a.s_dequant[unit_token(i)];
            alpha[i] = a.w_scales[unit_feature(i) / a.rows_per_group];
        }
    }

#pragma unroll
    for (int s = 0; s < D - 1; ++s)
        if (s < stages) issue(s, s);

    // operand offsets inside the group's block; accumulator i of this wave: weight tile, token tile
    constexpr int WI = F::WI, TI = F::TI;
    auto tile_of = [&](int i) { return half / (TB / TI) * WI + i / TI; };
    auto token_tile_of = [&](int i) { return half % (TB / TI) * TI + i % TI; };
    const int row = token_tile_of(0) * 32 + (lane & 31);   // of accumulator 0
    int xo_lo[2], xo_hi[2], xo_byte[4];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        xo_lo[k] = group * BLOCK + row * kRecordRowBytes + record_lo_offset(row, k, lane >> 5);
        xo_hi[k] = group * BLOCK + row * kRecordRowBytes + record_hi_offset(row, k, lane >> 5);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        xo_byte[k] = group * BLOCK + row * kBK + ((code_chunk_of_dword(k, lane >> 5) ^ ((row >> 1) & 7)) << 4);
    const int wo = group * BLOCK + CODES + tile_of(0) * 1024 + lane * 16;

    typedef typename std::conditional<F::I8, v16i, v16f>::type acc_t;
    typedef typename std::conditional<F::I8, v4i, v4f>::type sum_t;
    acc_t acc[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0;

    int slot = 0;
    for (int s = 0; s < stages; ++s) {
        // stage s has landed once at most min(D - 2, stages - 1 - s) later stages of this wave are in flight; after the
        // barrier it is visible to every wave and the buffer of stage s - 1 is free
        wait_stage(stages - 1 - s);
        if constexpr (GW > 1) asm volatile("s_barrier" ::: "memory");   // (a group of one wave shares its block with nobody)
        const char* base = lds + slot * STAGE;
        const bool live = s * KG + group < nkb;   // uniform
        if constexpr (F::I8) {
            v4i w[WI];
#pragma unroll
            for (int i = 0; i < WI; ++i) w[i] = *reinterpret_cast<const v4i*>(base + wo + i * 1024);
            v4i x[4][TI];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < TI; ++i) x[k][i] = *reinterpret_cast<const v4i*>(base + xo_byte[k] + i * 32 * kBK);
            if (s + D - 1 < stages) issue(s + D - 1, slot == 0 ? D - 1 : slot - 1);
            if (live) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
#pragma unroll
                    for (int n = 0; n < WI; ++n) {
                        const v4i wop = expand_weights_i8((uint32_t)w[n][k]);
#pragma unroll
                        for (int i = 0; i < TI; ++i)
                            acc[n * TI + i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wop, x[k][i], acc[n * TI + i], 0, 0, 0);
                    }
                }
            }
        } else {
            v4i w[WI];
            v8i x[2][TI];
#pragma unroll
            for (int i = 0; i < WI; ++i) w[i] = *reinterpret_cast<const v4i*>(base + wo + i * 1024);
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < TI; ++i) {
                    const v4i lo = *reinterpret_cast<const v4i*>(base + xo_lo[k] + i * 32 * kRecordRowBytes);
                    const int2 hi = *reinterpret_cast<const int2*>(base + xo_hi[k] + i * 32 * kRecordRowBytes);
                    x[k][i] = v8i{lo[0], lo[1], lo[2], lo[3], hi.x, hi.y, 0, 0};
                }
            if (s + D - 1 < stages) issue(s + D - 1, slot == 0 ? D - 1 : slot - 1);
            if (live) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int n = 0; n < WI; ++n) {
                        const v8i wop = fp4_operand((uint32_t)w[n][2 * k], (uint32_t)w[n][2 * k + 1]);
#pragma unroll
                        for (int i = 0; i < TI; ++i)
                            acc[n * TI + i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wop, x[k][i], acc[n * TI + i], 4 /*A: fp4*/,
                                                                                              3 /*B: bf6*/, 0, 0, 0, 0);
                    }
            }
        }
        slot = slot + 1 == D ? 0 : slot + 1;
    }

    // the groups' sums by token row, then eight threads per token add them and store 16 bytes of bf16 each
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wave is done with the stage buffers
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<sum_t*>(lds + (group * BT + token_tile_of(i) * 32 + (lane & 31)) * SUMROW +
                                      (32 * tile_of(i) + 8 * g + 4 * (lane >> 5)) * 4) =
                sum_t{acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]};
    __syncthreads();
#pragma unroll
    for (int i = 0; i < F::STORES; ++i) {
        if (!unit_stores(i)) continue;
        const int unit = tid + i * F::THREADS;
        sum_t v[2] = {sum_t{0, 0, 0, 0}, sum_t{0, 0, 0, 0}};
#pragma unroll
        for (int g = 0; g < KG; ++g)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                v[q] += *reinterpret_cast<const sum_t*>(lds + (g * BT + unit / TPT) * SUMROW + (unit % TPT) * 32 + q * 16);
        const size_t at = (size_t)unit_token(i) * a.N + unit_feature(i);
        if constexpr (RAW) {
            v4i* dst = reinterpret_cast<v4i*>(a.acc_out + at);
#pragma unroll
            for (int q = 0; q < 2; ++q) dst[q] = v4i{(int)v[q][0], (int)v[q][1], (int)v[q][2], (int)v[q][3]};
        } else {
            uint2 o[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if constexpr (F::I8) o[q] = dequant_quad(v[q], sd[i], alpha[i], a.code_offset, a.w_row_sum + unit_feature(i) + 4 * q);
                else o[q] = dequant_quad_f32(v[q][0], v[q][1], v[q][2], v[q][3], sd[i], alpha[i]);
            }
            store_y16(a.y + at, make_uint4(o[0].x, o[0].y, o[1].x, o[1].y));
        }
    }
}

template <typename F, bool RAW>
__global__ __launch_bounds__(F::THREADS) void mid_gemm_kernel(const MidProblem a) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    mid_gemm_body<F, RAW>(a, blockIdx.x, lds);
}

// Several problems of at most 64 tokens in one grid: workgroup -> problem, and one of two forms by the problem.
template <typename FA, typename FB>
__global__ __launch_bounds__(FA::THREADS) void mid_gemm_grouped_kernel(const MidArgs args) {
    static_assert(FA::THREADS == FB::THREADS, "one workgroup size");
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const MidProblem p = args.p[group_index_of(args.wg_begin, args.n, (int)blockIdx.x)];
    const int wg = (int)blockIdx.x - p.wg_begin;
    if (std::is_same<FA, FB>::value || p.form == 0) mid_gemm_body<FA, false>(p, wg, lds);   // uniform over the workgroup
    else if constexpr (!std::is_same<FA, FB>::value) mid_gemm_body<FB, false>(p, wg, lds);
}

template <typename F, bool RAW>
int launch_cfg(MidProblem a, hipStream_t stream) {
    a.tiles_n = (int)F::tiles_n(a.N);
    a.tiles_t = (int)F::tiles_t(a.T);
    constexpr auto kern = mid_gemm_kernel<F, RAW>;
    if (const int rc = allow_dynamic_lds<kern, F::LDS>(); rc != HBL_OK) return rc;
    launch_kernel("mid_gemm_kernel", kern, dim3((unsigned)(a.tiles_n * a.tiles_t)), dim3(F::THREADS), F::LDS, stream, a);
    return after_launch();
}

// Tiles of 64 x 64 outputs.  Up to 256 of them one workgroup per CU with three stages of LDS; up to 512 two per CU with two
// stages each (128 tokens, 4096 -> 12288: 15.4 -> 14.0 us per call; but 300 tokens, 8192 -> 3072, 240 tiles, 19.6 -> 23.1 us).
// Up to 128 the token tile is halved: half of the chip would idle; with a K range of 64 blocks and more eight groups (128
// tokens, 16384 -> 4096: 22.0 -> 20.0 us, with four groups 21.5).  Where 32 x 32 outputs give at most one workgroup per CU and
// each of eight one-wave groups at least one K-block, that form needs no barrier and half of the stages (64 tokens, 16384 ->
// 4096: 18.5 -> 14.4 us; 32 x 4096 -> 4096 9.3 -> 7.6; 64 x 1024 -> 4096 6.3 -> 6.0).  Above 512 tiles the 128 x 128 tile of
// the prefill kernel is faster (256 tokens, 4096 -> 12288, 768 tiles: 18.0 against 20.5 us).
// Up to 64 tokens there is no such tile: four weight tiles per code stage move fewer bytes (64 tokens, 4096 -> 131072: 47 -> 35
// us).  At most 32 tokens get three stages of LDS, so that three workgroups share a CU (with four stages, two: INT8 17 x 4096
// -> 131072 33.5 -> 32.1 us, INT4 24 x 16384 -> 65536 49.3 -> 48.3).  The same form with one stage less from 257 tiles on where
// K is at most 1024: with one or two stages per K group, what counts is how many workgroups start at once (24 x 512 -> 32768
// INT4 6.8 -> 6.3, 17 x 512 -> 32768 INT8 6.5 -> 6.2; 64 x 256 -> 24576 7.3 -> 6.5 us; at K = 2048 1.0 to 1.06, at 8192 1.07 to
// 1.25 times the time).
int64_t mid_tiles(int64_t T, int64_t N) { return MidForm<4, 2, 2, 2>::tiles_n(N) * MidForm<4, 2, 2, 2>::tiles_t(T); }

constexpr int64_t kMidResident = 512;   // workgroups of 8 waves and up to 80 KiB of LDS that the chip holds at once

// Bytes, more than 512 tiles of 64 x 64: 8-wave workgroups of two K groups on 128 x 64 outputs, of which a CU holds two, or 128 x
// 128 ones, one a CU.  The prefill kernel's 128 x 128 tile issues the 15 instructions that expand 16 weights from four waves; where a
// launch is one round, two waves a SIMD of one tile hide it better.  Time of the GEMM, 1100 sizes, against that tile (two stages) and
// the 256 x 128 one (H):
//   all 128 x 64 tiles resident at once (512; at most 256 of 128 x 128 are): K up to 1024 0.93 to 0.99 of the small tile, 2048 0.95,
//     4096 0.92, 8192 0.90, H 1.3 to 1.5 times as slow.  Rows beyond 1024: 128 x 128 outputs, 0.91 to 1.01 of 128 x 64
//   more, up to 384 tiles of 128 x 128: K = 128 1.10 to 1.15 of the small tile, 256 1.04, 384 1.03, 512 0.95, 768 0.97, 1024 0.97 (H
//     1.03), 1152 to 1536 0.98 to 1.03 of H, 2048 1.04, 3072 1.06, 4096 1.09, 8192 1.2
//   385 to 512: 1.04 to 1.34 of the better of the two
// (2048 x 2048 -> 2048 with the quantiser 19.6 -> 18.6 us, 1536 x 1024 -> 3072 15.4 -> 13.9.)  Records expand 16 weights by three
// instructions: 1.0 to 1.35 there.
int64_t mid_large_tiles(int64_t T, int64_t N) { return ((N + 127) / 128) * ((T + 127) / 128); }

template <bool I8, bool RAW>
int launch_form(const MidProblem& a, hipStream_t stream) {
    const int64_t tiles = mid_tiles(a.T, a.N);
    if constexpr (I8) {
        if (a.T > 64 && tiles > kMidResident)
            return a.K > 1024 && mid_large_tiles(a.T, a.N) <= 256 ? launch_cfg<MidForm<2, 3, 4, 4, true>, RAW>(a, stream)
                                                                  : launch_cfg<MidForm<2, 3, 4, 2, true>, RAW>(a, stream);
    }
    using Narrow = MidForm<8, 3, 1, 1, I8>;
    if (a.K >= 1024 && Narrow::tiles_n(a.N) * Narrow::tiles_t(a.T) <= 256) return launch_cfg<Narrow, RAW>(a, stream);
    if (tiles <= 128) return a.K < 8192 ? launch_cfg<MidForm<4, 4, 2, 1, I8>, RAW>(a, stream) : launch_cfg<MidForm<8, 3, 2, 1, I8>, RAW>(a, stream);
    const bool many = tiles > kMidResident, short_rows = a.T <= 64 && a.K <= 1024 && tiles > 256;   // (many: at most 64 tokens)
    if (a.T <= 32 && (many || short_rows)) return launch_cfg<MidForm<2, 3, 4, 1, I8>, RAW>(a, stream);
    if (many) return launch_cfg<MidForm<2, 3, 4, 2, I8>, RAW>(a, stream);
    if (short_rows) return launch_cfg<MidForm<2, 2, 4, 2, I8>, RAW>(a, stream);
    if (a.T <= 32) return launch_cfg<MidForm<4, 3, 2, 1, I8>, RAW>(a, stream);
    if (tiles <= 256) return launch_cfg<MidForm<4, 3, 2, 2, I8>, RAW>(a, stream);
    return launch_cfg<MidForm<4, 2, 2, 2, I8>, RAW>(a, stream);
}

template <typename FA, typename FB>
int launch_grouped_forms(MidArgs& args, hipStream_t stream) {
    int wgs = 0;
    for (int i = 0; i < args.n; ++i) {
        MidProblem& p = args.p[i];
        p.tiles_n = (int)(p.form == 0 ? FA::tiles_n(p.N) : FB::tiles_n(p.N));
        p.tiles_t = (int)(p.form == 0 ? FA::tiles_t(p.T) : FB::tiles_t(p.T));
        p.wg_begin = args.wg_begin[i] = wgs;
        wgs += p.tiles_n * p.tiles_t;
    }
    constexpr size_t lds = FA::LDS > FB::LDS ? FA::LDS : FB::LDS;
    constexpr auto kern = mid_gemm_grouped_kernel<FA, FB>;
    if (const int rc = allow_dynamic_lds<kern, lds>(); rc != HBL_OK) return rc;
    launch_kernel("mid_gemm_grouped_kernel", kern, dim3((unsigned)wgs), dim3(FA::THREADS), lds, stream, args);
    return after_launch();
}

// Short rows, more than 256 tiles: as for single calls.  (Four projections 256 -> 8192, 47 tokens 8.6 -> 7.9 us; 512 -> 8192 at
// 17 tokens 7.5 -> 6.9.)  A kernel of one form alone where the group needs no other: its LDS is that form's.
template <typename F>
int launch_grouped_one(MidArgs& args, hipStream_t stream) { return launch_grouped_forms<F, F>(args, stream); }

template <bool I8>
int launch_grouped(MidArgs& args, int max_t, int64_t tiles, bool any_long, hipStream_t stream) {
    const bool few = max_t <= 32, fits = tiles <= kMidResident, short_rows = args.p[0].K <= 1024 && tiles > 256;
    if (short_rows) return few ? launch_grouped_one<MidForm<2, 3, 4, 1, I8>>(args, stream) : launch_grouped_one<MidForm<2, 2, 4, 2, I8>>(args, stream);
    if (few && fits)   // (more tiles of records than that stay with the shared form)
        return launch_grouped_forms<MidForm<4, 3, 2, 1, I8>, MidForm<8, 2, 1, 1, I8>>(args, stream);
    if constexpr (I8) {
        if (few) return any_long ? launch_grouped_forms<MidForm<2, 3, 4, 1, true>, MidForm<8, 2, 1, 1, true>>(args, stream)
                                 : launch_grouped_one<MidForm<2, 3, 4, 1, true>>(args, stream);
    }
    if (fits) return launch_grouped_forms<MidForm<4, 2, 2, 2, I8>, MidForm<8, 2, 1, 1, I8>>(args, stream);
    return launch_grouped_forms<MidForm<2, 3, 4, 2, I8>, MidForm<4, 3, 2, 1, I8>>(args, stream);
}

}  // namespace

// Up to 64 tokens, beyond 512 tiles, rows of at most 1024 bytes: a workgroup has at most eight K-blocks and nothing is gained
// by cutting them over its waves; the int8 kernel's tiles of 128 features by 32 or 64 tokens are up to 1.2 times as fast (20 x
// 128 -> 131072 7.4 us against 8.7, 64 x 384 -> 98304 9.1 against 10.3; from K = 1536 on they are 1.0 to 1.1 times as slow, and
// above 32 tokens already from K = 512 on up to 65536 output rows).
bool mid_gemm_preferred(int64_t T, int64_t K, int64_t N, bool records) {
    if (mid_tiles(T, N) <= kMidResident) return true;
    return T <= 64 && (records || K > (T <= 32 || N > 65536 ? 1024 : 384));
}

bool mid_large_bytes_preferred(int64_t T, int64_t K, int64_t N) {
    if (T <= 64) return false;
    return MidForm<2, 3, 4, 2, true>::tiles_n(N) * MidForm<2, 3, 4, 2, true>::tiles_t(T) <= 512 ||
           (K >= 512 && K <= 1536 && mid_large_tiles(T, N) <= 384);
}

int launch_mid_gemm(const MidProblem& a, bool records, hipStream_t stream) {
    if (records) return a.acc_out ? launch_form<false, true>(a, stream) : launch_form<false, false>(a, stream);
    return a.acc_out ? launch_form<true, true>(a, stream) : launch_form<true, false>(a, stream);
}

int launch_mid_gemm_grouped(MidArgs& args, hipStream_t stream) {
    if (args.n <= 0) return HBL_OK;
    // long K ranges first: their workgroups run longest
    for (int i = 1; i < args.n; ++i)
        for (int j = i; j > 0 && args.p[j].K > args.p[j - 1].K; --j) {
            const MidProblem t = args.p[j];
            args.p[j] = args.p[j - 1];
            args.p[j - 1] = t;
        }
    int max_t = 0, bytes = 0;
    int64_t tiles = 0, narrow = 0;
    for (int i = 0; i < args.n; ++i) {
        max_t = args.p[i].T > max_t ? args.p[i].T : max_t;
        bytes += args.p[i].bytes != 0;
        tiles += mid_tiles(args.p[i].T, args.p[i].N);
        narrow += MidForm<8, 2, 1, 1>::tiles_n(args.p[i].N) * MidForm<8, 2, 1, 1>::tiles_t(args.p[i].T);
    }
    if (bytes != 0 && bytes != args.n) {
        // Records and bytes: one launch with a form for either.  Two launches cost 2 to 3 us more (24 tokens, 256 -> 4096 and 512
        // -> 2048: 9.5 us, 6.4 as one; 47 tokens, 384 / 1536 four projections 12.2, 7.8).
        for (int i = 0; i < args.n; ++i) args.p[i].form = args.p[i].bytes != 0;
        if (narrow <= kMidResident) return launch_grouped_forms<MidForm<8, 2, 1, 1, false>, MidForm<8, 2, 1, 1, true>>(args, stream);
        return max_t <= 32 ? launch_grouped_forms<MidForm<4, 3, 2, 1, false>, MidForm<4, 3, 2, 1, true>>(args, stream)
                           : launch_grouped_forms<MidForm<4, 2, 2, 2, false>, MidForm<4, 2, 2, 2, true>>(args, stream);
    }
    // While everything is resident at once: small tiles.  Beyond that four weight tiles per code stage move fewer bytes (47
    // tokens, four 7B projections, 832 tiles: 36.2 -> 30.5 us per layer), and a K range much longer than the others' takes more
    // groups and smaller tiles so that it does not outlast them (with eight one-wave groups it is 640 workgroups: 36.5 us).  Not
    // so where all are long: 33 to 64 tokens, two projections 8192 -> 16384, 36 us with the smaller tiles, 23 without; three
    // 8192 -> 8192 28 and 22.
    const int shortest = args.p[args.n - 1].K;
    bool any_long = false;
    for (int i = 0; i < args.n; ++i) {
        MidProblem& p = args.p[i];
        p.form = narrow <= kMidResident ? p.K >= 2048 : p.K >= 8192 && p.K >= 2 * shortest;
        any_long = any_long || p.form != 0;
    }
    return bytes == 0 ? launch_grouped<false>(args, max_t, tiles, any_long, stream) : launch_grouped<true>(args, max_t, tiles, any_long, stream);
}

// A group at 47 tokens: 2048 / 8192 projections 21.2 -> 14.7 us per layer against the shared form of the weight-streaming
// kernel, 7B 31.8 -> 30.5; up to 32 tokens that form's 512 workgroups of four waves are the better one once the tiles do not
// fit at once (7B, 20 tokens: 25.3 against 26.0 us per layer; 2048 / 8192, 24 tokens: 17.0 against 14.0).
// INT8 activations: 7B 20 tokens 27.2 -> 25.2, 64 tokens 36.8 -> 32, 2048 / 8192 40 tokens 24.4 -> 14.6; but rows of at most
// 1024 bytes, up to 32 tokens, that do not fit at once are faster in the shared form: four projections 256 -> 24576, 17 tokens
// 7.4 us against 8.6, 1024 -> 16384 9.0 against 10.4.
bool mid_group_preferred(const DecodeProblem* p, int n) {
    int max_t = 0, max_k = 0, records = 0;
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) {
        max_t = p[i].T > max_t ? p[i].T : max_t;
        max_k = p[i].K > max_k ? p[i].K : max_k;
        records += p[i].f6 != 0;
        tiles += mid_tiles(p[i].T, p[i].N);
    }
    if (max_t <= 16) return false;
    if (records != 0 && records != n) return true;   // (the shared form takes one kind)
    return max_t > 32 || tiles <= kMidResident || (records == 0 && max_k > 1024);
}

}  // namespace hbl
