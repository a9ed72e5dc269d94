// Device body of the activation front end (Eq. 3-6) for transformed rows of 2048 features and more: one row by K / 2^R
// threads of 2^R values (16 or 32) each, one exchange through LDS.
#pragma once

#include "quant_bodies.h"

namespace hbl {
namespace {

// A SIMD takes a single-precision instruction of a wave every 2 cycles, but one wave issues only every 5: what counts is
// how many waves share a SIMD.  (Measured: 2.1 ns per instruction with one wave per SIMD, 1.15 with two, 1.05 with four; the
// DPP and double-precision forms take 4 cycles: 2.1 ns with four.)  So a row is spread over many threads of few values.
//
// Index bits of a row of K = 2^m elements.  Layout A (as loaded): a thread holds 2^(R-3) chunks of 8 consecutive elements
//   [0-2: inside the chunk][3-6: low four lane bits][7..R+3: chunk number][then lane bits 4, 5 and the wave]
// and runs the stages in ascending order: 0-2 in registers, 3-6 between lanes, 7..R+3 in registers.  Then the row goes
// through LDS once (one float per element), and in layout B element f = f_t(tid) + RS * r is register r of thread tid: its r
// bits are the index bits from R+4 on (and, below them, SPARE finished ones if m < 2 R + 4).  If m > 2 R + 4, the EXTRA = 1 or
// 2 highest index bits are lane bits of B (bit 3; bits 0 and 1) and their stages run between lanes, last.
// Both sides of the exchange are free of bank conflicts: in A eight consecutive lanes write 16-byte pieces that are 32
// bytes apart; in B consecutive lanes read consecutive dwords at compile-time offsets from one address, and where the
// highest index bits sit in the low lane bits, these bits are also xored into bits 4 and 5 of the slot (slot()).
//
// Stages between lanes.  v <- partner * c + v with the partner read through a DPP lane permutation and c = +1 where the bit
// is 0 (a + b) and -1 where it is 1 (b - a): the product is exact and the sum rounds once, so the lower lane holds the
// reference's a + b and the upper lane the negative of its a - b.  Negation commutes with every later rounding, so a lane
// simply carries the sign (-1)^(number of its index bits 3-6 that are set); in layout B those bits belong to the thread
// number, all values of a thread share the sign, and it leaves through the factor the values are multiplied with anyway
// (1/sqrt(K) or the quantiser's gain).  DPP offers xor 1, xor 2 (quad permutes), xor 7 (half-row mirror) and xor 8 (row
// rotation by 8) inside a row of 16 lanes, so the thread of position p is lane p ^ (3 if bit 2 of p): flipping index bit 5
// (bit 2 of p) then flips lane bits 0-2 together.
template <int LOG2K, int R>
struct LargeRow {
    static constexpr int K = 1 << LOG2K, E = 1 << R, NT = K >> R, W = NT / 64;
    static constexpr int CHUNKS = E / 8;                 // chunks of 8 elements per thread
    static constexpr int SPARE = 2 * R + 4 > LOG2K ? 2 * R + 4 - LOG2K : 0;   // low bits of B's register number that are finished
    static constexpr int EXTRA = LOG2K > 2 * R + 4 ? LOG2K - 2 * R - 4 : 0;   // index bits left for lane stages in B
    static constexpr int RS = NT >> EXTRA;               // elements between the registers of a thread in B
    static constexpr int WAVE_FLOATS = 64 * E;           // a wave's elements in layout A are consecutive
    static_assert(R >= 4 && R <= 5 && SPARE < R && EXTRA <= 2 && RS >= 128, "split");
    __device__ static uint32_t position(uint32_t tid) { return (tid & 15u) ^ (((tid >> 2) & 1u) * 3u); }
    // first element, in layout A, of chunk c of this thread; without the wave's part
    __device__ static uint32_t in_wave(uint32_t tid, int c) {
        return 8u * position(tid) + 128u * c + 128u * CHUNKS * ((tid >> 4) & 3u);
    }
    // element of register 0 of this thread in layout B
    __device__ static uint32_t thread_b(uint32_t tid) {
        if constexpr (EXTRA == 1) return (tid & 7u) | ((tid >> 4) << 3) | (((tid >> 3) & 1u) << (LOG2K - 1));
        if constexpr (EXTRA == 2) return (tid >> 2) | ((tid & 3u) << (LOG2K - 2));
        return tid;
    }
    // place of element f in the row buffer (floats, and later the codes)
    __device__ static uint32_t slot(uint32_t f) {
        return EXTRA == 0 ? f : f ^ ((f >> (LOG2K - EXTRA)) << (EXTRA == 1 ? 5 : 4));
    }
};
// One row's input as loaded.
template <int R, bool BF16>
struct LargeRowRaw {
    static constexpr int Q = BF16 ? 1 : 2;   // 16-byte pieces of a chunk
    uint4 q[Q << (R - 3)];
};
template <int LOG2K, int R, bool BF16>
__device__ __forceinline__ void large_row_load(const void* __restrict__ x, int64_t row, uint32_t tid, LargeRowRaw<R, BF16>& raw) {
    using L = LargeRow<LOG2K, R>;
    constexpr int Q = LargeRowRaw<R, BF16>::Q;
    const char* base = static_cast<const char*>(x) + row * (int64_t)L::K * (BF16 ? 2 : 4);
    const uint32_t first = (L::in_wave(tid, 0) + (tid >> 6) * L::WAVE_FLOATS) * (BF16 ? 2 : 4);
#pragma unroll
    for (int c = 0; c < L::CHUNKS; ++c)
#pragma unroll
        for (int i = 0; i < Q; ++i)
            raw.q[c * Q + i] = *reinterpret_cast<const uint4*>(base + first + c * 128 * (BF16 ? 2 : 4) + i * 16);
}

// The same through LDS, for a caller that has its row copied there (global -> LDS copies, one wave at a time, each the elements
// of its own threads: nobody else reads them) into the row buffer, where the wave later writes its floats.
template <int LOG2K, int R, bool BF16>
__device__ __forceinline__ void large_row_copy(const void* __restrict__ x, int64_t row, uint32_t tid, char* row_buffer) {
    using L = LargeRow<LOG2K, R>;
    constexpr int EB = BF16 ? 2 : 4;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const char* src = static_cast<const char*>(x) + (row * L::K + wave * L::WAVE_FLOATS) * EB;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(row_buffer + wave * L::WAVE_FLOATS * 4);
#pragma unroll
    for (int i = 0; i < L::WAVE_FLOATS * EB / 1024; ++i) gemm::lds_dma16(lds0 + i * 1024, src + i * 1024, (tid & 63) * 16);
}
template <int LOG2K, int R, bool BF16>
__device__ __forceinline__ void large_row_read(uint32_t tid, const char* row_buffer, LargeRowRaw<R, BF16>& raw) {
    using L = LargeRow<LOG2K, R>;
    constexpr int Q = LargeRowRaw<R, BF16>::Q, EB = BF16 ? 2 : 4;
    const char* part = row_buffer + __builtin_amdgcn_readfirstlane(tid >> 6) * L::WAVE_FLOATS * 4;
#pragma unroll
    for (int c = 0; c < L::CHUNKS; ++c)
#pragma unroll
        for (int i = 0; i < Q; ++i) raw.q[c * Q + i] = *reinterpret_cast<const uint4*>(part + L::in_wave(tid, c) * EB + i * 16);
}

// BF6OUT (INT4 only): records (code_records.h) instead of one byte per code.  NORM: compiled with the RMS-normalisation prologue
// (taken when rp.ln_gain is set).  BITS = 0: the transform alone; `codes` is the output array and `code_offset` its element type.
// row_lds: K floats.  GROUPS: rows that a workgroup works on side by side, this one by its threads [group * NT, (group + 1) * NT)
// (tid counts from the first of them).
template <int LOG2K, int R, int BITS, bool BF16, bool BF6OUT, bool NORM, int BLOCKB = kRecordBlockBytes, int GROUPS = 1>
__device__ __forceinline__ void large_row_body(int64_t row, uint32_t tid, const LargeRowRaw<R, BF16>& raw, float* row_lds,
                                               int8_t* __restrict__ codes, float* __restrict__ s_dequant,
                                               int32_t* __restrict__ code_sum, RowParams rp, int code_offset, int group = 0) {
    using L = LargeRow<LOG2K, R>;
    constexpr int few_rows = 1;
    constexpr int K = L::K, E = L::E, NT = L::NT, W = L::W, CHUNKS = L::CHUNKS, RS = L::RS;
    static_assert(!BF6OUT || BITS == 4, "records carry INT4 codes only");
    __shared__ double red_ds[GROUPS][W];
    __shared__ float red_fs[GROUPS][W];
    __shared__ int red_is[GROUPS][W];
    double* const red_d = red_ds[GROUPS == 1 ? 0 : group];
    float* const red_f = red_fs[GROUPS == 1 ? 0 : group];
    int* const red_i = red_is[GROUPS == 1 ? 0 : group];
    const int lane = tid & 63, wave = tid >> 6;
    const uint32_t pos = L::position(tid);
    const uint32_t first = L::in_wave(tid, 0) + wave * L::WAVE_FLOATS;

    float a[CHUNKS][8];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        if constexpr (BF16) {
            const uint32_t w[4] = {raw.q[c].x, raw.q[c].y, raw.q[c].z, raw.q[c].w};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                a[c][2 * h] = as_f(w[h] << 16);
                a[c][2 * h + 1] = as_f(w[h] & 0xFFFF0000u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[c][4 * i] = as_f(raw.q[2 * c + i].x); a[c][4 * i + 1] = as_f(raw.q[2 * c + i].y);
                a[c][4 * i + 2] = as_f(raw.q[2 * c + i].z); a[c][4 * i + 3] = as_f(raw.q[2 * c + i].w);
            }
        }
    }

    if (NORM && rp.ln_gain) {   // uniform: RMS normalisation ahead of the transform
        __shared__ double red_n[GROUPS][W];
        double ss = 0.0;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += (double)a[c][e] * (double)a[c][e];
        const float rn = rms_factor<W>(ss, red_n[GROUPS == 1 ? 0 : group], lane, wave, K, rp.ln_eps, few_rows);
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            float g[8];
            load_chunk<8, false>(rp.ln_gain, first + 128 * c, g);
#pragma unroll
            for (int e = 0; e < 8; ++e) a[c][e] = (a[c][e] * rn) * g[e];
        }
    }

#pragma unroll
    for (int h = 1; h < 8; h <<= 1)           // index bits 0-2
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if ((e & h) == 0) {
                    const float p = a[c][e], q = a[c][e + h];
                    a[c][e] = p + q;
                    a[c][e + h] = p - q;
                }
    lane_stage_fma<0xB1>(a, pos & 1u);        // index bit 3: lane ^ 1 (quad_perm [1,0,3,2])
    lane_stage_fma<0x4E>(a, pos & 2u);        // index bit 4: lane ^ 2 (quad_perm [2,3,0,1])
    lane_stage_fma<0x141>(a, pos & 4u);       // index bit 5: lane ^ 7 (row_half_mirror)
    lane_stage_fma<0x128>(a, pos & 8u);       // index bit 6: lane ^ 8 (row_ror:8)
#pragma unroll
    for (int h = 1; h < CHUNKS; h <<= 1)      // index bits 7..R+3
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c)
            if ((c & h) == 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float p = a[c][e], q = a[c + h][e];
                    a[c][e] = p + q;
                    a[c + h][e] = p - q;
                }
            }

    float* const put = row_lds + L::slot(first);
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            *reinterpret_cast<float4*>(put + 128 * c + 4 * i) = make_float4(a[c][4 * i], a[c][4 * i + 1], a[c][4 * i + 2], a[c][4 * i + 3]);
    __syncthreads();
    float v[E / 8][8];
    const uint32_t f_t = L::thread_b(tid), slot_t = L::slot(f_t);
#pragma unroll
    for (int r = 0; r < E; ++r) v[r / 8][r % 8] = row_lds[slot_t + RS * r];
#pragma unroll
    for (int h = 1 << L::SPARE; h < E; h <<= 1)   // index bits R+4..
#pragma unroll
        for (int r = 0; r < E; ++r)
            if ((r & h) == 0) {
                const float p = v[r / 8][r % 8], q = v[(r + h) / 8][(r + h) % 8];
                v[r / 8][r % 8] = p + q;
                v[(r + h) / 8][(r + h) % 8] = p - q;
            }
    if constexpr (L::EXTRA == 1) lane_stage_fma<0x128>(v, tid & 8u);
    if constexpr (L::EXTRA == 2) {
        lane_stage_fma<0xB1>(v, tid & 1u);
        lane_stage_fma<0x4E>(v, tid & 2u);
    }

    // c_n = (float)(1/sqrt(K)).  For even log2 K it is a power of two: scaling by it commutes exactly with every later
    // rounding (max, fp64 sum, the gain product), so it is applied to the row statistics and folded into the gain instead of
    // costing one multiply per element.  c_s: with the sign that this thread's values carry out of the lane stages.
    const float c_n = (float)(1.0 / sqrt((double)K));
    const float c_s = (__builtin_popcount((f_t >> 3) & 15u) ^ __builtin_popcount(f_t >> (LOG2K - L::EXTRA))) & 1 ? -c_n : c_n;
    constexpr bool FOLD = (LOG2K % 2) == 0 && BITS != 0;
    if constexpr (!FOLD) {   // (a multiply-add with zero rounds the product once, and turns a zero that carries the sign into +0)
#pragma unroll
        for (int r = 0; r < E; ++r) v[r / 8][r % 8] = __builtin_fmaf(v[r / 8][r % 8], c_s, 0.0f);
    }

    if constexpr (BITS == 0) {
        if (code_offset != HBL_BF16 && L::EXTRA == 0) {   // consecutive lanes, consecutive floats
            float* out = reinterpret_cast<float*>(codes) + row * K + f_t;
#pragma unroll
            for (int r = 0; r < E; ++r)
                __builtin_nontemporal_store(v[r / 8][r % 8], out + RS * r);
        } else if (code_offset != HBL_BF16) {   // through the row buffer (1 row of 16384: 4.6 us -> 3.9)
#pragma unroll
            for (int r = 0; r < E; ++r) row_lds[slot_t + RS * r] = v[r / 8][r % 8];   // where this thread has read
            __syncthreads();
#pragma unroll
            for (int i = 0; i < E / 4; ++i)
                store_stream16(reinterpret_cast<float*>(codes) + row * K + (tid + NT * i) * 4,
                               reinterpret_cast<const uint4*>(row_lds)[L::slot((tid + NT * i) * 4) >> 2]);
        } else {
            __syncthreads();
            __bf16* h = reinterpret_cast<__bf16*>(row_lds);
#pragma unroll
            for (int r = 0; r < E; ++r) h[slot_t + RS * r] = (__bf16)v[r / 8][r % 8];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < E / 8; ++i)
                store_stream16(reinterpret_cast<uint16_t*>(codes) + row * K + (tid + NT * i) * 8,
                               reinterpret_cast<const uint4*>(row_lds)[L::slot((tid + NT * i) * 8) >> 3]);
        }
        return;
    }

    float gain, s_d;
    if constexpr (BITS == 8) {
        float m = 0.0f;
#pragma unroll
        for (int r = 0; r < E; ++r) m = fmaxf(m, fabsf(v[r / 8][r % 8]));
        m = wave_max(m, few_rows);
        if (lane == 0) red_f[wave] = m;
        __syncthreads();
        m = red_f[0];
#pragma unroll
        for (int w = 1; w < W; ++w) m = fmaxf(m, red_f[w]);
        if constexpr (FOLD) m = m * c_n;
        gain = 127.0f / (m + rp.eps);
        s_d = m / 127.0f;
    } else {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < E; ++r) s += (double)fabsf(v[r / 8][r % 8]);
        s = wave_sum(s, few_rows);
        if (lane == 0) red_d[wave] = s;
        __syncthreads();
        s = red_d[0];
#pragma unroll
        for (int w = 1; w < W; ++w) s += red_d[w];
        if constexpr (FOLD) s = s * (double)c_n;
        const float beta = (float)(s / (double)K);
        gain = kRoot7 / (beta + rp.eps);
        s_d = beta / kRoot7;
    }
    // (the barrier above also says that every thread has read its values out of the row buffer: the codes go there next)

    constexpr float lo = BITS == 8 ? -128.0f : -8.0f;
    constexpr float hi = BITS == 8 ? 127.0f : 7.0f;
    if constexpr (FOLD) gain = gain * c_s;   // (the statistics took |v| and the positive c_n)
    int isum = 0;
    if constexpr (!BF6OUT) {
        // adding 1.5 * 2^23 rounds to the nearest (even) integer and leaves its two's complement in the low mantissa byte
        const float magic = kMagic + (float)code_offset;
        uint8_t* b = reinterpret_cast<uint8_t*>(row_lds);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const uint32_t bits = as_u(__builtin_amdgcn_fmed3f(v[r / 8][r % 8] * gain, lo, hi) + magic);
            b[slot_t + RS * r] = (uint8_t)bits;
            if (code_sum) isum += (int)(bits - as_u(magic));
        }
        __syncthreads();
        // (Plain stores: the GEMM reads the codes next.  With the non-temporal hint the launch alone is 5 to 12 % faster - 8192 rows of
        // 16384 82.5 -> 76.6 us - but the call is not: 0.98 to 1.02 with it from 1024 output rows on, 1.02 to 1.34 below - 64 rows of
        // 16384 against 32 output rows 13.7 -> 18.4.  Only 6 to 8 MiB of codes gain, 1 to 7 %.)
#pragma unroll
        for (int i = 0; i < E / 16; ++i)
            *reinterpret_cast<uint4*>(codes + row * K + (tid + NT * i) * 16) = reinterpret_cast<const uint4*>(row_lds)[L::slot((tid + NT * i) * 16) >> 4];
    } else {
        // The codes as fp32 integers (adding and removing 1.5 * 2^23 also turns -0 into +0) have at most four significant bits:
        // the upper half of the register is the same number in bf16.  It goes to LDS by feature, and the thread of a record
        // (32 features) reads 64 bytes and converts them in one instruction (exact for integers in [-8, 7]).  16-byte piece u
        // of the row lies at u ^ ((u >> 4) & 3) (and slot()), so that the reads, 64 bytes apart, spread over the banks.
        char* h = reinterpret_cast<char*>(row_lds);
        const uint32_t at = (2 * slot_t) ^ (((f_t >> 7) & 3u) << 4);
        float fsum = 0.0f;
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const float q = (__builtin_amdgcn_fmed3f(v[r / 8][r % 8] * gain, lo, hi) + kMagic) - kMagic;
            *reinterpret_cast<uint16_t*>(h + (at ^ ((((RS * r) >> 7) & 3) << 4)) + 2 * RS * r) = (uint16_t)(as_u(q) >> 16);
            if (code_sum) fsum += q;   // uniform, and off on the forward path: small integers, exact in any order
        }
        isum = (int)fsum;
        __syncthreads();
        if (R == 5 || tid < K / 32) {
            typedef __bf16 v32h __attribute__((ext_vector_type(32)));
            typedef uint32_t v6u __attribute__((ext_vector_type(6)));
            struct alignas(16) Half32 { uint4 q[4]; } in;
#pragma unroll
            for (int i = 0; i < 4; ++i) in.q[i] = *reinterpret_cast<const uint4*>(h + ((2 * L::slot(32 * tid + 8 * i)) ^ (((tid >> 2) & 3u) << 4)));
            const v6u d = __builtin_bit_cast(v6u, __builtin_amdgcn_cvt_scalef32_pk32_bf6_bf16(__builtin_bit_cast(v32h, in), 1.0f));
            store_code_record<BLOCKB>(codes, row, K, (int)tid, d[0], d[1], d[2], d[3], d[4], d[5]);
        }
    }
    if (code_sum) {   // uniform: the fp6 x fp4 GEMM needs no code sum
        isum = wave_sum(isum, few_rows);
        if (lane == 0) red_i[wave] = isum;
        __syncthreads();
        isum = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) isum += red_i[w];
        if (tid == 0) code_sum[row] = isum;
    }
    if (tid == 0) s_dequant[row] = s_d;
}

}  // namespace
}  // namespace hbl
