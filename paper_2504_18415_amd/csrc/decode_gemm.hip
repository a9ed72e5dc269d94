// Small-batch (decode) form of the ternary GEMM of Eq. 7: T <= 16 tokens (32 in the shared form), so the packed weights are
// read once from HBM and dominate the traffic, and the job is to keep as many weight tiles in flight as
// the memory system needs.  One launch serves up to kMaxGroup independent projections.
//
// A wave owns one 32-row weight tile at a time and walks its K range tile by tile (1 KiB of packed
// weights = 32 rows x 128 features).  Weights and activation codes both arrive by direct global->LDS
// copies, D = 4 stages deep per wave.  Per problem one of two operand paths:
//  - fp6 x fp4 (INT4 activations, K >= 512): codes from the record image (96 bytes per token and stage),
//    weights to fp4 with 3 vector-ALU instructions per 16; two 16x16x128 MFMAs per tile for up to 16 tokens,
//    two 32x32x64 per tile above that.  fp32 accumulators hold exact integers.
//  - int8 (INT8 activations, short rows): codes as bytes (128 per token and stage), weights to signed bytes
//    (15 instructions per 16), four 32x32x32 MFMAs per tile and 32 tokens.
//
// Two forms:
//  - streaming (T <= 16): a wave's code stage is private (8 or 16 rows), so the waves never meet at a
//    barrier.  The K range of one row tile may be split over the 2 or 4 waves of a workgroup; their
//    accumulators are added through LDS at the end (exact).
//  - shared (17 to 32 tokens, where there are too many output rows for the mid-size kernel, mid_gemm.hip; a launch of
//    records or of bytes): the four waves take four row tiles over one K range and share the code stage (32 rows): one
//    barrier per stage.  A K range split over workgroups leaves int32 slices in the workspace; the workgroup of a K range
//    that finishes last (an arrival counter) adds the others' slices to its own accumulators and dequantises.  (A group
//    with more split row groups than a slot has counters runs without the split.)
#include <atomic>

#include "gemm_common.h"

namespace hbl {
namespace {

using namespace gemm;
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

// The 16-byte-per-lane global -> LDS copy of gemm_common.h by the first 48 lanes only: 768 contiguous bytes, eight
// 96-byte rows of the record image.  (The 12-byte-per-lane form of the instruction strides the LDS side by 16
// bytes per lane - measured - so it cannot lay down contiguous rows.)  The execution mask is narrowed around
// the copy inside one asm block and put back.
__device__ __forceinline__ void lds_dma16_first48(uint32_t lds_addr, const void* base, uint32_t voff) {
    uint64_t saved;
    asm volatile(
        "s_mov_b64 %0, exec\n\ts_bfm_b64 exec, 48, 0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
        : "=&s"(saved)
        : "s"(lds_addr), "v"(voff), "s"(base)
        : "memory", "m0");
}

// NW = waves per workgroup.  Four everywhere except the streaming form on a single long-K problem with few row
// tiles (W_down alone): there 8 waves share a row tile's K range, which shortens each wave's serial chain of
// tiles (128 workgroups cannot be made more without narrower row tiles).
// F6: the problem's codes are bf6 records and the fp6 x fp4 matrix cores do the work.
template <bool SHARE, int RQ, int D, int NW, bool F6>
__device__ __forceinline__ void decode_body(const DecodeProblem& p, const int w, char* lds, unsigned int* p_arrive) {
    constexpr int ROWS = SHARE ? 32 : RQ * 8;         // token rows of one code stage
    constexpr int ROWB = F6 ? kRecordRowBytes : kBK;  // bytes of one token row of a stage
    constexpr int XB = ROWS * ROWB;                   // bytes of one code stage
    constexpr int XW = SHARE ? XB : NW * XB;          // code bytes per stage in the workgroup
    constexpr int STAGE = XW + NW * 1024;             // + one packed weight tile per wave
    constexpr int XL = SHARE ? 1 : RQ;                // code copies per wave per stage (8 rows each)
    static_assert(D >= 3 && (ROWS & (ROWS - 1)) == 0, "pipeline depth / row count");
    static_assert(!SHARE || NW == 4, "the shared form is written for four waves");
    static_assert(NW * 4096 <= D * STAGE, "the in-workgroup reduction reuses the stage buffers");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kl = __builtin_ctz((unsigned)p.ksplit);   // p.ksplit is a power of two, at most NW
    const int nkb_total = p.K / kBK;
    const int nkb = nkb_total >> kl;
    int nt, ks;
    if constexpr (SHARE) {
        nt = 4 * (w >> kl) + wave;
        ks = w & (p.ksplit - 1);
    } else {
        nt = w * (NW >> kl) + (wave >> kl);
        ks = wave & (p.ksplit - 1);
    }
    const int nt_max = p.N / 32 - 1;
    const bool live = nt <= nt_max;          // a wave past the last row tile streams that tile again, writes nothing
    const int ntc = live ? nt : nt_max;
    const int kb0 = ks * nkb;

    // packed tiles are stored K-block-major (tile (nt, kb) at (kb * N/32 + nt) KiB): at any moment the waves
    // of a launch, all at about the same kb, read one window of consecutive addresses
    const size_t wstride = (size_t)(p.N / 32) * 1024;
    const char* wbase = reinterpret_cast<const char*>(p.packed) + (size_t)kb0 * wstride + (size_t)ntc * 1024;
    const uint32_t wlane = lane * 16;
    // Code copy m of a stage covers rows 8q..8q+7.
    //  bytes: lane l -> row 8q + l/8, LDS slot l%8 of that row, global 16-byte chunk (l%8) ^ ((row/2) % 8); rows
    //         past T re-read the last token;
    //  records: the rows are 768 contiguous bytes of the stage's block of the record image (rows past T exist
    //         there and hold finite garbage that is never stored).
    const char* xbase = reinterpret_cast<const char*>(p.codes) + (size_t)kb0 * (F6 ? kRecordBlockBytes : kBK);
    uint32_t xlane[XL];
#pragma unroll
    for (int m = 0; m < XL; ++m) {
        const int q = SHARE ? wave + 4 * m : m;
        if constexpr (F6) {
            xlane[m] = q * 768 + lane * 16;   // 8 rows of 96 bytes: the first 48 lanes of a 16-byte-per-lane copy
        } else {
            const int row = 8 * q + (lane >> 3);
            const int t = row < p.T ? row : p.T - 1;
            const int c = (lane & 7) ^ ((row >> 1) & 7);
            xlane[m] = (uint32_t)t * (uint32_t)p.K + c * 16;
        }
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const uint32_t xarea = SHARE ? 0 : wave * XB;

    // Copies of stage kb into buffer `slot`.
    auto issue = [&](int kb, int slot) {
#pragma unroll
        for (int m = 0; m < XL; ++m) {
            const int q = SHARE ? wave + 4 * m : m;
            if constexpr (F6) lds_dma16_first48(lds0 + slot * STAGE + xarea + q * 768, xbase + (size_t)kb * kRecordBlockBytes, xlane[m]);
            else lds_dma16(lds0 + slot * STAGE + xarea + q * 1024, xbase + (size_t)kb * kBK, xlane[m]);
        }
        lds_dma16(lds0 + slot * STAGE + XW + wave * 1024, wbase + (size_t)kb * wstride, wlane);
    };

    // Operand read offsets inside a stage.
    //  int8: token row (lane & 31) of tile j (rows beyond the stage wrap onto loaded rows; their results are
    //        never written), the 16-byte chunk that matches packed dword k4, swizzled like the copy.
    //  fp6 x fp4, streaming: 16x16x128 MFMA - lane = (token lane & 15, feature group g = lane >> 4 of 32);
    //        the weights of row 16 hf + (lane & 15), features 32 g + 0..31, are dwords 2 (g >> 1), +1 of tile
    //        lane row + 32 (g & 1).
    //  fp6 x fp4, shared: 32x32x64 MFMA as in the prefill kernel - lane = (token lane & 31, half lane >> 5).
    int xoff[4];
    int xo_lo[2], xo_hi[2], wo[2];
    if constexpr (!F6) {
        const int r0 = (lane & 31) & (ROWS - 1);
#pragma unroll
        for (int k4 = 0; k4 < 4; ++k4) xoff[k4] = r0 * kBK + ((code_chunk_of_dword(k4, lane >> 5) ^ ((r0 >> 1) & 7)) << 4);
    } else if constexpr (!SHARE) {
        const int r0 = (lane & 15) & (ROWS - 1), g = lane >> 4;
        xo_lo[0] = r0 * kRecordRowBytes + record_lo_offset(r0, g >> 1, g & 1);
        xo_hi[0] = r0 * kRecordRowBytes + record_hi_offset(r0, g >> 1, g & 1);
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) wo[hf] = (16 * hf + (lane & 15) + 32 * (g & 1)) * 16 + 8 * (g >> 1);
    } else {
        const int r0 = lane & 31;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            xo_lo[s] = r0 * kRecordRowBytes + record_lo_offset(r0, s, lane >> 5);
            xo_hi[s] = r0 * kRecordRowBytes + record_hi_offset(r0, s, lane >> 5);
        }
    }

    v16i acc[2];             // int8 path: two accumulators take turns so that consecutive MFMAs do not depend on each other
    v4f facc[2];             // fp6 x fp4, streaming: row halves 0..15, 16..31 of the tile
    v16f wacc;               // fp6 x fp4, shared
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) facc[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r < 16; ++r) wacc[r] = 0.0f;

    // Stage kb may be consumed once at most min(D - 2, nkb - 1 - kb) later stages are still in flight
    // (copies return in order).  Nothing is requested past the end of the K range, so the count
    // shrinks over the last D - 2 stages.
    auto wait_stage = [&](int later) {
        if (later >= D - 2) {
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((D - 2) * (XL + 1)) : "memory");
            return;
        }
        switch (later) {
            case 0: asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); break;
            case 1: asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(1 * (XL + 1)) : "memory"); break;
            case 2: asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * (XL + 1)) : "memory"); break;
            case 3: asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(3 * (XL + 1)) : "memory"); break;
            case 4: asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 * (XL + 1)) : "memory"); break;
            default: asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(5 * (XL + 1)) : "memory"); break;
        }
    };
    static_assert(D - 2 <= 6, "wait_stage covers up to 5 later stages below the steady state");

#pragma unroll
    for (int s = 0; s < D - 1; ++s)
        if (s < nkb) issue(s, s);

    // Epilogue operands, requested right behind the first stages: under a saturated memory system a load
    // issued after the loop would add its whole latency to the workgroup's run time, and ahead of the first
    // copies they would delay the stream.  (They return in order behind the D - 1 stages in flight, which
    // only makes the first waits below stricter than they need to be.)
    const bool write_partial = SHARE && p.ksplit > 1;
    const bool writer = live && (SHARE || ks == 0);
    constexpr bool TOK16 = F6 && !SHARE;     // the 16x16 accumulator layout: token = lane & 15
    float alpha = 0.0f, sd = 0.0f;
    v4i wsum[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) wsum[g] = v4i{0, 0, 0, 0};
    if (writer) {   // (with a K range split over workgroups any of them may turn out to be the one that dequantises)
        alpha = p.w_scales[(nt * 32) / p.rows_per_group];
        const int t = lane & (TOK16 ? 15 : 31);
        if (t < p.T) sd = p.s_dequant[t];
        if (!F6 && p.code_offset != 0) {
#pragma unroll
            for (int g = 0; g < 4; ++g)
                wsum[g] = *reinterpret_cast<const v4i*>(p.w_row_sum + nt * 32 + 8 * g + 4 * (lane >> 5));
        }
    }

    // One stage: its operand reads go out first, then `copies()` (the copies of a later stage), then the MFMAs, so
    // that the LDS latency passes while the copies are being accepted (worth 0.1-0.2 us per launch in the streaming
    // form: the stream itself already runs at what HBM delivers, a shorter stage only lengthens the wait).
    auto stage_work = [&](const char* st, auto&& copies) {
        if constexpr (!F6) {
            const v4i wpk = *reinterpret_cast<const v4i*>(st + XW + wave * 1024 + lane * 16);
            v4i xop[4];
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) xop[k4] = *reinterpret_cast<const v4i*>(st + xarea + xoff[k4]);
            copies();
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4)
                acc[k4 & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(expand_weights_i8((uint32_t)wpk[k4]), xop[k4], acc[k4 & 1], 0, 0, 0);
        } else if constexpr (!SHARE) {
            const v4i lo = *reinterpret_cast<const v4i*>(st + xarea + xo_lo[0]);
            const int2 hi = *reinterpret_cast<const int2*>(st + xarea + xo_hi[0]);
            uint2 wp[2];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) wp[hf] = *reinterpret_cast<const uint2*>(st + XW + wave * 1024 + wo[hf]);
            copies();
            const v8i xop = {lo[0], lo[1], lo[2], lo[3], hi.x, hi.y, 0, 0};
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
                facc[hf] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fp4_operand(wp[hf].x, wp[hf].y), xop, facc[hf],
                                                                            4 /*A: fp4*/, 3 /*B: bf6*/, 0, 0, 0, 0);
        } else {
            const v4i wpk = *reinterpret_cast<const v4i*>(st + XW + wave * 1024 + lane * 16);
            v8i xop[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const v4i lo = *reinterpret_cast<const v4i*>(st + xo_lo[s]);
                const int2 hi = *reinterpret_cast<const int2*>(st + xo_hi[s]);
                xop[s] = v8i{lo[0], lo[1], lo[2], lo[3], hi.x, hi.y, 0, 0};
            }
            copies();
#pragma unroll
            for (int s = 0; s < 2; ++s)
                wacc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp4_operand((uint32_t)wpk[2 * s], (uint32_t)wpk[2 * s + 1]),
                                                                       xop[s], wacc, 4, 3, 0, 0, 0, 0);
        }
    };
    // Stage kb has landed (for every wave, if the code stage is shared); the buffer read in the previous iteration is free
    // for stage kb + D - 1.  The last D - 1 stages, which request nothing and wait for fewer copies, stand apart, one by one:
    // with few workgroups a wave has its SIMD to itself and walks its stages one after another, so every branch of the
    // steady loop is waited for.  In one loop, three or four branches each, the time even hung on where the compiler had put
    // it: GEMM launch alone, 3 tokens x 16256 -> 24576 records 21.8 to 23.6 us, now 20.0; 3 x 11008 -> 12288 9.5 to 10.0, now
    // 8.3; INT8 8 x 16128 -> 24576 25.2 to 26.4, now 23.6; groups of INT8 projections at 8 tokens, 2048 / 8192 8.2 to 8.4,
    // now 7.6, 7B 15.5 to 16.0, now 14.8.
    int slot = 0, kb = 0;
    for (; kb < nkb - (D - 1); ++kb) {
        wait_stage(D - 2);
        if constexpr (SHARE) asm volatile("s_barrier" ::: "memory");
        stage_work(lds + slot * STAGE, [&]() { issue(kb + D - 1, slot == 0 ? D - 1 : slot - 1); });
        slot = slot + 1 == D ? 0 : slot + 1;
    }
#pragma unroll
    for (int later = D - 2; later >= 0; --later) {
        if (nkb <= later) continue;   // (uniform)
        wait_stage(later);
        if constexpr (SHARE) asm volatile("s_barrier" ::: "memory");
        stage_work(lds + slot * STAGE, []() {});
        slot = slot + 1 == D ? 0 : slot + 1;
    }
    if constexpr (!F6) acc[0] += acc[1];

    if constexpr (!SHARE) {
        if (p.ksplit > 1) {   // uniform over the workgroup
            __syncthreads();  // every wave is done with the stage buffers
            int* red = reinterpret_cast<int*>(lds);
            float* fred = reinterpret_cast<float*>(lds);
            if (ks != 0) {
                if constexpr (F6) {
#pragma unroll
                    for (int r = 0; r < 8; ++r) fred[(wave * 8 + r) * 64 + lane] = facc[r >> 2][r & 3];
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = acc[0][r];
                }
            }
            __syncthreads();
            if (ks == 0) {
                for (int kk = 1; kk < p.ksplit; ++kk) {
                    if constexpr (F6) {
#pragma unroll
                        for (int r = 0; r < 8; ++r) facc[r >> 2][r & 3] += fred[((wave + kk) * 8 + r) * 64 + lane];
                    } else {
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[0][r] += red[((wave + kk) * 16 + r) * 64 + lane];
                    }
                }
            }
        }
        if (ks != 0) return;
    }
    if constexpr (!SHARE) {
        if (!writer) return;
    }

    if constexpr (TOK16) {
        // lane holds token lane & 15; facc[hf] holds features 16 hf + 4 (lane >> 4) + 0..3 of the row tile
        const int t = lane & 15;
        if (t >= p.T) return;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const int n = nt * 32 + 16 * hf + 4 * (lane >> 4);
            *reinterpret_cast<uint2*>(p.y + (size_t)t * p.N + n) =
                dequant_quad_f32(facc[hf][0], facc[hf][1], facc[hf][2], facc[hf][3], sd, alpha);
        }
        return;
    }
    // lane holds token (lane & 31); register quad g holds features 8g + 4*(lane >> 5) + 0..3 of the weight tile
    v4i tot[4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (F6) tot[g][r] = (int)wacc[4 * g + r];
            else tot[g][r] = acc[0][4 * g + r];
        }
    if constexpr (SHARE) {
        if (write_partial) {   // uniform over the workgroup
            // This workgroup's slice of the K range, as int32 tiles (exact).  A slice is only ever read by a workgroup
            // of the same shape, so it is kept as the lanes hold it - quad g of wave `wave` of slice k at v4i index
            // (((k * groups + group) * 4 + wave) * 4 + g) * 64 + lane: every store and load instruction moves 1 KiB of consecutive bytes.  The
            // stores are device-scope (write-through): readable from the other XCDs without a write-back of this L2.
            const int groups = (p.N / 32 + 3) / 4;
            v4i* const frag = reinterpret_cast<v4i*>(p.partial);
            auto frag_index = [&](int k, int q) { return ((((size_t)k * groups + (w >> kl)) * 4 + wave) * 4 + q) * 64 + lane; };
#pragma unroll
            for (int q = 0; q < 4; ++q)
                asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(frag + frag_index(ks, q)), "v"(tot[q]) : "memory");
            // Arrival: once a workgroup's stores have completed it counts itself in; the counter wraps at ksplit, so
            // the workgroup that brings it back to zero is the last of its K range and every slice is in memory.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();   // (every wave of the workgroup is here: the stage buffers are free)
            unsigned int* arrived = reinterpret_cast<unsigned int*>(lds);
            if (tid == 0) *arrived = atomicInc(p_arrive + p.arrive_begin + (w >> kl), (unsigned)p.ksplit - 1u);
            __syncthreads();
            if (*arrived != (unsigned)p.ksplit - 1u || !writer) return;
            // (device-scope loads, 8 bytes each: they do not stop at this XCD's L2)
            for (int k = 0; k < p.ksplit; ++k) {
                if (k == ks) continue;   // (uniform)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint64_t* src = reinterpret_cast<const uint64_t*>(frag + frag_index(k, q));
                    const uint64_t lo = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const uint64_t hi = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    tot[q] += v4i{(int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi, (int)(uint32_t)(hi >> 32)};
                }
            }
        } else if (!writer) {
            return;
        }
    }
    const int t = lane & 31;
    if (t >= p.T) return;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        uint2* const dst = reinterpret_cast<uint2*>(p.y + (size_t)t * p.N + nt * 32 + 8 * g + 4 * (lane >> 5));
        if constexpr (F6) *dst = dequant_quad_f32((float)tot[g][0], (float)tot[g][1], (float)tot[g][2], (float)tot[g][3], sd, alpha);
        else *dst = dequant_quad_sums(tot[g], sd, alpha, p.code_offset, wsum[g]);
    }
}

// BYTES (shared form): the problems' codes are bytes, else records.  (A streaming launch takes either, problem by problem.)
template <bool SHARE, int RQ, int D, int NW, bool BYTES>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void decode_gemm_kernel(const DecodeArgs args) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const DecodeProblem p = args.p[group_index_of(args.wg_begin, args.n, (int)blockIdx.x)];
    const int w = (int)blockIdx.x - p.wg_begin;
    if constexpr (SHARE) {
        decode_body<SHARE, RQ, D, NW, !BYTES>(p, w, lds, args.arrive);
    } else {
        if (p.f6) decode_body<SHARE, RQ, D, NW, true>(p, w, lds, args.arrive);      // uniform over the workgroup
        else decode_body<SHARE, RQ, D, NW, false>(p, w, lds, args.arrive);
    }
}

// Arrival counters of the shared form's in-kernel reduction: one per group of four row tiles whose K range is split
// over workgroups.  A counter wraps at the number of slices, so it is back at zero when its launch is over and needs
// no initialisation beyond the zeros the array is loaded with.  The host hands the kArriveSlots slots out round-robin:
// launches that overlap on one GPU (other streams) count in different words unless more than that many are in flight.
constexpr int kArriveWords = 2048;
constexpr int kArriveSlots = 128;
__device__ __attribute__((aligned(256))) unsigned int g_arrive[kArriveSlots * kArriveWords];

// This device's copy of the array (each GPU holds its own, at its own address), advanced to the next slot.
int next_arrive_slot(unsigned int** out) {
    static std::atomic<unsigned int*> base[64];
    static std::atomic<unsigned int> next{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return note_hip_error(e);
    unsigned int* ptr = base[dev & 63].load(std::memory_order_acquire);
    if (!ptr) {
        e = hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(g_arrive));
        if (e != hipSuccess) return note_hip_error(e);
        base[dev & 63].store(ptr, std::memory_order_release);
    }
    *out = ptr + (size_t)(next.fetch_add(1, std::memory_order_relaxed) % kArriveSlots) * kArriveWords;
    return HBL_OK;
}

template <bool SHARE, int RQ, int D, int NW = 4, bool BYTES = false>
int launch_form(const DecodeArgs& planned, int wgs, int counters, hipStream_t stream) {
    DecodeArgs a = planned;
    a.arrive = nullptr;
    if (counters != 0) {   // some K range is split over workgroups
        if (const int rc = next_arrive_slot(&a.arrive); rc != HBL_OK) return rc;
    }
    constexpr int ROWS = SHARE ? 32 : RQ * 8;
    constexpr size_t lds = (size_t)D * ((SHARE ? 1 : NW) * ROWS * kBK + NW * 1024);
    constexpr auto kern = decode_gemm_kernel<SHARE, RQ, D, NW, BYTES>;
    if (const int rc = allow_dynamic_lds<kern, lds>(); rc != HBL_OK) return rc;
    launch_kernel("decode_gemm_kernel", kern, dim3((unsigned)wgs), dim3(64 * NW), lds, stream, a);
    return after_launch();
}

// Workgroups a problem occupies in the GEMM grid for a given K split.
int problem_wgs(const DecodeProblem& p, bool share) {
    const int tiles = p.N / 32;
    return share ? ((tiles + 3) / 4) * p.ksplit : (tiles * p.ksplit + 3) / 4;
}


// K split of every problem, then each problem's first workgroup in the grid and its first arrival counter.
// About 32 weight tiles (32 KiB) per wave; while the grid is too small to occupy the chip (256 CUs x
// 2 workgroups) split further, down to 8 tiles per wave.  The streaming form adds the slices inside a
// workgroup, so a split is free; the shared form needs the partial buffer and ends with the last workgroup of a
// K range adding the others' slices, so it splits further only when less than three quarters of the CUs would get
// a workgroup.
void plan(DecodeArgs& a, bool share, int* wgs_out, int* counters_out) {
    const int enough = share ? 192 : 384;
    int total = 0;
    for (int i = 0; i < a.n; ++i) {
        DecodeProblem& p = a.p[i];
        const int nkb = p.K / 128;
        const bool may_split = !share || p.partial != nullptr;
        p.ksplit = 1;
        while (may_split && p.ksplit < kMaxDecodeSplit && nkb % (2 * p.ksplit) == 0 && nkb / (2 * p.ksplit) >= 32)
            p.ksplit *= 2;
        total += problem_wgs(p, share);
    }
    for (int pass = 0; pass < 2 && total < enough; ++pass) {
        total = 0;
        for (int i = 0; i < a.n; ++i) {
            DecodeProblem& p = a.p[i];
            const int nkb = p.K / 128;
            const bool may_split = !share || p.partial != nullptr;
            if (may_split && p.ksplit < kMaxDecodeSplit && nkb % (2 * p.ksplit) == 0 && nkb / (2 * p.ksplit) >= 8)
                p.ksplit *= 2;
            total += problem_wgs(p, share);
        }
    }
    // a K range split over workgroups (shared form) needs one arrival counter per group of four row tiles; a group
    // with more of them than a slot holds runs without that split
    int counters = 0;
    for (int i = 0; i < a.n; ++i)
        if (share && a.p[i].ksplit > 1) counters += (a.p[i].N / 32 + 3) / 4;
    if (counters > kArriveWords) {
        for (int i = 0; i < a.n; ++i) a.p[i].ksplit = 1;
        counters = 0;
    }
    int wgs = 0, next_counter = 0;
    for (int i = 0; i < a.n; ++i) {
        DecodeProblem& p = a.p[i];
        p.wg_begin = a.wg_begin[i] = wgs;
        wgs += problem_wgs(p, share);
        p.arrive_begin = next_counter;
        if (share && p.ksplit > 1) next_counter += (p.N / 32 + 3) / 4;
    }
    *wgs_out = wgs;
    *counters_out = counters;
}

// A single streaming-form problem whose four-wave plan would leave long serial chains of tiles on few
// workgroups (W_down alone: 128 row tiles, 128 K blocks): waves per workgroup for the wide form, or 0.
int wide_waves(const DecodeArgs& a, int max_t) {
    if (a.n != 1 || max_t > 16) return 0;
    const DecodeProblem& p = a.p[0];
    const int nkb = p.K / 128, tiles = p.N / 32;
    if (nkb < 64 || tiles > 192) return 0;
    const int nw = 8;   // 16 waves measured equal at batch 1 and 5 % slower at batch 8 and 16
    return nkb % nw == 0 ? nw : 0;
}
void plan_wide(DecodeArgs& a, int nw, int* wgs_out) {
    DecodeProblem& p = a.p[0];
    p.ksplit = nw;   // one row tile per workgroup, its K range over all waves: 8 tiles or more per wave (nkb >= 64)
    p.wg_begin = a.wg_begin[0] = 0;
    p.arrive_begin = 0;
    *wgs_out = (p.N / 32 * p.ksplit + nw - 1) / nw;
}

}  // namespace

// A wave's tiles are a serial chain: few workgroups with long chains leave most of the chip idle, and there the mid-size
// kernel cuts K further.  Call time by that kernel against this one, 1 to 16 tokens, chains of more than 16 tiles: records,
// up to 128 workgroups 0.75 (K in one piece) and 0.92 (in two), from there on 1.08 and 1.18 (3 x 11008 -> 10240: 16.4 us,
// 12.9 here); bytes, up to 128 workgroups 0.5 to 0.7, up to 192 0.91 and 1.02.
bool decode_stream_preferred(int64_t T, int64_t K, int64_t N, bool records) {
    if (T <= 0 || T > 16) return false;
    DecodeArgs a = {};
    a.n = 1;
    a.p[0].T = (int)T;
    a.p[0].K = (int)K;
    a.p[0].N = (int)N;
    if (wide_waves(a, (int)T) != 0) return true;
    int wgs, counters;
    plan(a, false, &wgs, &counters);
    return (K / 128) / a.p[0].ksplit <= 16 || wgs > (records ? 128 : 191);
}

// Against the mid-size kernel, 17 to 32 tokens: this form reads each code stage once per four weight tiles too and has no
// sums to add up, but its waves meet at a barrier per K-block.  Call time here against there: up to 32768 output rows 1.0
// at K = 512 to 1024, up to 1.2 above; beyond them K = 512 0.82 to 0.97, 2048 0.92 to 0.97, 4096 0.95 to 1.0, 5504 0.94 to
// 0.98, and where the K range is split over workgroups 11008 0.91 up to 45056 rows, 8192 0.94 to 1.0; above that 1.05 to 1.6.
bool decode_shared_preferred(int64_t T, int64_t K, int64_t N) {
    return T > 16 && T <= 32 && N > 32768 && (K < 8192 || (K < 12288 && N <= 45056));
}

int decode_plan_for_tests(DecodeArgs& a, int* wgs, int* counters) {
    int max_t = 0;
    for (int i = 0; i < a.n; ++i) max_t = a.p[i].T > max_t ? a.p[i].T : max_t;
    if (a.n <= 0 || max_t > 32) return HBL_E_SHAPE;
    if (const int nw = wide_waves(a, max_t); nw != 0) {
        plan_wide(a, nw, wgs);
        *counters = 0;
        return HBL_OK;
    }
    plan(a, max_t > 16, wgs, counters);
    return HBL_OK;
}

int launch_decode_gemm(DecodeArgs& a, hipStream_t stream) {
    if (a.n <= 0) return HBL_OK;
    int max_t = 0;
    for (int i = 0; i < a.n; ++i) max_t = a.p[i].T > max_t ? a.p[i].T : max_t;
    if (max_t > 32) return HBL_E_SHAPE;   // (the mid-size kernel's)
    int records = 0;
    for (int i = 0; i < a.n; ++i) records += a.p[i].f6 != 0;
    if (max_t > 16 && records != 0 && records != a.n) return HBL_E_SHAPE;
    int wgs, counters;
    if (const int nw = wide_waves(a, max_t); nw != 0) {
        plan_wide(a, nw, &wgs);
        return max_t <= 8 ? launch_form<false, 1, 4, 8>(a, wgs, 0, stream)
                          : launch_form<false, 2, 4, 8>(a, wgs, 0, stream);
    }
    plan(a, max_t > 16, &wgs, &counters);
    // Stages in flight per wave: 4.  Shallow is best (3 to 8 measured): the memory-level parallelism comes from
    // the 2048 waves of a full grid, and deeper rings only cost LDS and queueing.
    if (max_t <= 8) return launch_form<false, 1, 4>(a, wgs, 0, stream);
    if (max_t <= 16) return launch_form<false, 2, 4>(a, wgs, 0, stream);
    return records != 0 ? launch_form<true, 1, 4>(a, wgs, counters, stream) : launch_form<true, 1, 4, 4, true>(a, wgs, counters, stream);
}

}  // namespace hbl
