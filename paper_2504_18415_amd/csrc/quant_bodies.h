// Device bodies of the activation front end (Eq. 3-6): one token row per call, by one or more waves of a workgroup.  The
// launches of fwht_quant.hip and the one-launch small-batch kernels (fused_small.hip, fused_bytes.hip) run the same code;
// transformed rows of 2048 and more in launches of their own: large_rows.h.
#pragma once

#include <type_traits>

#include "gemm_common.h"

namespace hbl {
namespace {


constexpr float kRoot7 = 2.6457513110645907f;  // (float)sqrt(7.0), bit pattern 0x402953FD
constexpr float kMagic = 12582912.0f;          // 1.5 * 2^23: adding it rounds to an integer (nearest-even)

__device__ __forceinline__ float as_f(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t as_u(float f) { return __builtin_bit_cast(uint32_t, f); }

// Value held by lane (lane ^ MASK).
template <int MASK>
__device__ __forceinline__ float lane_xor(float v) {
    const int iv = (int)as_u(v);
    if constexpr (MASK == 1) {
        return as_f((uint32_t)__builtin_amdgcn_mov_dpp(iv, 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
    } else if constexpr (MASK == 2) {
        return as_f((uint32_t)__builtin_amdgcn_mov_dpp(iv, 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
    } else if constexpr (MASK == 8) {
        return as_f((uint32_t)__builtin_amdgcn_mov_dpp(iv, 0x128, 0xF, 0xF, false));  // row_ror:8
    } else if constexpr (MASK == 4) {
        return as_f((uint32_t)__builtin_amdgcn_ds_swizzle(iv, 0x101F));  // xor 4 inside 32 lanes
    } else if constexpr (MASK == 16) {
        return as_f((uint32_t)__builtin_amdgcn_ds_swizzle(iv, 0x401F));  // xor 16 inside 32 lanes
    } else {
        return __shfl_xor(v, MASK, 64);
    }
}

// Whole-wave reductions whose result every lane receives; all 64 lanes must be active.
// Form 1, data-parallel moves: inside a row of 16 lanes two quad permutes, then the half-row and row mirrors
// (each step adds the same two partial results in both lanes of a pair, so all lanes of the row agree); the
// four row results are then read lane by lane and combined in a fixed order.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, false);
}
// v <- v(partner lane) * c + v for the four registers of a chunk, the partner reached by DPP permutation CTRL:
// v_fmac_f32 with a DPP source, which the compiler does not form by itself (it emits a DPP move and a separate
// multiply-add).  A DPP operand must not be read within two wait states of a vector-ALU write to the same
// register, and the compiler does not look inside an asm statement: the leading s_nop covers whatever
// precedes the block, and inside it the four instructions touch four different registers.  (Blocks of 16
// with one s_nop measured slower: the compiler can no longer place other work between the chunks.)
template <int CTRL>
__device__ __forceinline__ void lane_butterfly4(float (&a)[4], float c) {
    static_assert(CTRL == 0xB1 || CTRL == 0x4E || CTRL == 0x141 || CTRL == 0x128, "lane xor 1, 2, 7 or 8");
#define HBL_F(N, SEL) "v_fmac_f32_dpp %" #N ", %" #N ", %4 " SEL " row_mask:0xf bank_mask:0xf\n\t"
#define HBL_LANE_FMAC4(SEL) asm("s_nop 1\n\t" HBL_F(0, SEL) HBL_F(1, SEL) HBL_F(2, SEL) HBL_F(3, SEL) : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]) : "v"(c))
    if constexpr (CTRL == 0xB1) HBL_LANE_FMAC4("quad_perm:[1,0,3,2]");
    else if constexpr (CTRL == 0x4E) HBL_LANE_FMAC4("quad_perm:[2,3,0,1]");
    else if constexpr (CTRL == 0x141) HBL_LANE_FMAC4("row_half_mirror");
    else HBL_LANE_FMAC4("row_ror:8");
#undef HBL_LANE_FMAC4
#undef HBL_F
}
template <int CTRL>
__device__ __forceinline__ void lane_butterfly2(float (&a)[2], float c) {
#define HBL_F(N, SEL) "v_fmac_f32_dpp %" #N ", %" #N ", %2 " SEL " row_mask:0xf bank_mask:0xf\n\t"
#define HBL_LANE_FMAC2(SEL) asm("s_nop 1\n\t" HBL_F(0, SEL) HBL_F(1, SEL) : "+v"(a[0]), "+v"(a[1]) : "v"(c))
    if constexpr (CTRL == 0xB1) HBL_LANE_FMAC2("quad_perm:[1,0,3,2]");
    else if constexpr (CTRL == 0x4E) HBL_LANE_FMAC2("quad_perm:[2,3,0,1]");
    else if constexpr (CTRL == 0x141) HBL_LANE_FMAC2("row_half_mirror");
    else HBL_LANE_FMAC2("row_ror:8");
#undef HBL_LANE_FMAC2
#undef HBL_F
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint64_t r = (uint64_t)dpp_move<CTRL>((uint32_t)u) | ((uint64_t)dpp_move<CTRL>((uint32_t)(u >> 32)) << 32);
    return __builtin_bit_cast(double, r);
}
__device__ __forceinline__ uint32_t read_lane(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ double read_lane(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint64_t r = (uint64_t)read_lane((uint32_t)u, lane) | ((uint64_t)read_lane((uint32_t)(u >> 32), lane) << 32);
    return __builtin_bit_cast(double, r);
}
__device__ __forceinline__ double wave_sum_dpp(double s) {
    s += dpp_move<0xB1>(s);    // quad_perm [1,0,3,2]
    s += dpp_move<0x4E>(s);    // quad_perm [2,3,0,1]
    s += dpp_move<0x141>(s);   // row_half_mirror
    s += dpp_move<0x140>(s);   // row_mirror
    return ((read_lane(s, 0) + read_lane(s, 16)) + read_lane(s, 32)) + read_lane(s, 48);
}
__device__ __forceinline__ int wave_sum_dpp(int value) {   // modulo 2^32
    uint32_t s = (uint32_t)value;
    s += dpp_move<0xB1>(s);
    s += dpp_move<0x4E>(s);
    s += dpp_move<0x141>(s);
    s += dpp_move<0x140>(s);
    return (int)(read_lane(s, 0) + read_lane(s, 16) + read_lane(s, 32) + read_lane(s, 48));
}
__device__ __forceinline__ float wave_max_dpp(float m) {
    m = fmaxf(m, as_f(dpp_move<0xB1>(as_u(m))));
    m = fmaxf(m, as_f(dpp_move<0x4E>(as_u(m))));
    m = fmaxf(m, as_f(dpp_move<0x141>(as_u(m))));
    m = fmaxf(m, as_f(dpp_move<0x140>(as_u(m))));
    return fmaxf(fmaxf(as_f(read_lane(as_u(m), 0)), as_f(read_lane(as_u(m), 16))),
                 fmaxf(as_f(read_lane(as_u(m), 32)), as_f(read_lane(as_u(m), 48))));
}
// Form 2, six xor-shuffle rounds through the LDS crossbar: long dependent latency but no vector-ALU work.
// A launch that keeps every SIMD busy with other waves runs faster with these (5 % on 8192 rows of 16384); a
// launch of a few rows runs faster with form 1 (1.5 us per decode layer; the limits: launch_fwht_quant).
// `few_rows` is uniform.
__device__ __forceinline__ double wave_sum(double s, int few_rows) {
    if (few_rows) return wave_sum_dpp(s);
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) s += __shfl_xor(s, sft, 64);
    return s;
}
__device__ __forceinline__ int wave_sum(int s, int few_rows) {
    if (few_rows) return wave_sum_dpp(s);
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) s += __shfl_xor(s, sft, 64);
    return s;
}
__device__ __forceinline__ float wave_max(float m, int few_rows) {
    if (few_rows) return wave_max_dpp(m);
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) m = fmaxf(m, __shfl_xor(m, sft, 64));
    return m;
}

// Butterfly between lanes in one multiply-add per element (lane_butterfly4): v <- partner * c + v, c = -1 on the
// lane whose index bit is set.  That lane then holds the negative of the reference's a - b; see large_rows.h
// for why a lane may simply carry that sign until the values meet their 1/sqrt(K) factor.
template <int CTRL, int R, int CH>
__device__ __forceinline__ void lane_stage_fma(float (&v)[R][CH], bool upper) {
    const float c = upper ? -1.0f : 1.0f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if constexpr (CH == 2) {
            lane_butterfly2<CTRL>(v[r], c);
        } else {
#pragma unroll
            for (int e = 0; e < CH; e += 4) {
                float (&q)[4] = *reinterpret_cast<float (*)[4]>(&v[r][e]);
                lane_butterfly4<CTRL>(q, c);
            }
        }
    }
}

template <int MASK, int R, int CH>
__device__ __forceinline__ void lane_stage(float (&v)[R][CH], int lane) {
    // lanes with the bit clear compute a + b, lanes with it set compute a - b = partner - own
    const uint32_t sign = (lane & MASK) ? 0x80000000u : 0u;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const float own = v[r][e];
            const float partner = lane_xor<MASK>(own);
            v[r][e] = partner + as_f(as_u(own) ^ sign);
        }
}

template <int BYTES>
struct Raw;
template <>
struct Raw<2> { using type = uint16_t; };
template <>
struct Raw<4> { using type = uint32_t; };
template <>
struct Raw<8> { using type = uint2; };
template <>
struct Raw<16> { using type = uint4; };
template <>
struct Raw<32> { struct type { uint4 a, b; }; };

// Load CH consecutive elements starting at element offset `off` and widen to fp32.
template <int CH, bool BF16>
__device__ __forceinline__ void load_chunk(const void* x, int64_t off, float (&dst)[CH]) {
    if constexpr (BF16) {
        using V = typename Raw<CH * 2>::type;
        V raw = *reinterpret_cast<const V*>(static_cast<const uint16_t*>(x) + off);
        const uint16_t* h = reinterpret_cast<const uint16_t*>(&raw);
#pragma unroll
        for (int e = 0; e < CH; ++e) dst[e] = as_f((uint32_t)h[e] << 16);
    } else {
        using V = typename Raw<CH * 4>::type;
        V raw = *reinterpret_cast<const V*>(static_cast<const float*>(x) + off);
        const float* f = reinterpret_cast<const float*>(&raw);
#pragma unroll
        for (int e = 0; e < CH; ++e) dst[e] = f[e];
    }
}

// Four stored bytes code + 8 (0..15) -> their bf6 (e3m2) bit patterns, 6 bits each, as 24 contiguous
// bits.  Two 8-entry byte-permute look-ups and a select:
//   -8..-5 = 38 37 36 35, -4..-1 = 34 32 30 2c, 0..3 = 00 0c 10 12, 4..7 = 14 15 16 17 (hex)
__device__ __forceinline__ uint32_t bf6_pack4(uint32_t packed) {
    const uint32_t sel = packed & 0x07070707u;
    const uint32_t neg = __builtin_amdgcn_perm(0x2C303234u, 0x35363738u, sel);
    const uint32_t pos = __builtin_amdgcn_perm(0x17161514u, 0x12100C00u, sel);
    // byte i of the result: byte i of `pos` if bit 3 of the index is set, else byte i of `neg`
    const uint32_t pick = ((packed >> 1) & 0x04040404u) | 0x03020100u;
    const uint32_t r = __builtin_amdgcn_perm(pos, neg, pick);
    // four 6-bit fields, one per byte -> 24 contiguous bits
    const uint32_t t2 = (r & 0x003F003Fu) | ((r & 0x3F003F00u) >> 2);
    return (t2 & 0xFFFu) | ((t2 >> 4) & 0xFFF000u);
}

// bf6 record output for a lane that holds the 8 features of chunk `chunk8` of token `row` as two 24-bit
// halves, where neighbouring lanes hold neighbouring chunks: the even lane of each pair fetches its
// partner's halves and stores the pair's 16 features (96 bits) into the record image (code_records.h).
// Every lane of a quad must call this.
template <int BLOCKB>
__device__ __forceinline__ void bf6_store_pair(int8_t* codes, int64_t row, int K, int chunk8, uint32_t lo, uint32_t hi) {
    const uint32_t p_lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)lo, 0xB1, 0xF, 0xF, false);   // lane ^ 1
    const uint32_t p_hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)hi, 0xB1, 0xF, 0xF, false);
    if ((chunk8 & 1) == 0)
        store_code_quad<BLOCKB>(codes, row, K, chunk8 >> 1, lo | (hi << 24), (hi >> 8) | (p_lo << 16), (p_lo >> 16) | (p_hi << 8));
}

// Per-row scalars of the front end: the quantiser's epsilon and, if ln_gain != nullptr, the RMS
// normalisation that precedes the transform in Eq. 7 (LN; the model's norm is RMSNorm, Section 2):
//   x_n[k] = (x[k] * r) * ln_gain[k],  r = (float)(1 / sqrt(mean_k x[k]^2 + ln_eps)),
// mean of squares accumulated in fp64 (each square is exact there), r rounded to fp32 once, two fp32
// multiplies per element.
struct RowParams {
    float eps;
    const float* ln_gain;   // [K] fp32 or nullptr
    float ln_eps;
    int few_rows;           // few rows per SIMD: a row's latency matters, not throughput (reduction form)
};

// r of the row from this thread's partial sum of squares `ss`: wave butterfly, then a fixed-order
// combine of the NW per-wave sums through `red` (NW doubles of LDS; one barrier).
template <int NW>
__device__ __forceinline__ float rms_factor(double ss, double* red, int lane, int wave, int K, float ln_eps,
                                            int few_rows) {
    ss = wave_sum(ss, few_rows);
    if constexpr (NW > 1) {
        if (lane == 0) red[wave] = ss;
        __syncthreads();
        ss = red[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) ss += red[w];
    }
    return (float)(1.0 / sqrt(ss / (double)K + (double)ln_eps));
}

// Outputs of the transform alone leave with the non-temporal hint: written once and not read by the kernel, they need not
// stay in L2 until the launch ends and has to write them back.  4096 rows of 4096, bf16 -> fp32, 16.0 -> 14.0 us; 2048 of 2048
// fp32 6.0 -> 4.9.
__device__ __forceinline__ void store_stream16(void* dst, uint4 val) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store((u32x4){val.x, val.y, val.z, val.w}, reinterpret_cast<u32x4*>(dst));
}

// Transform-only output (BITS == 0 in the bodies below): N consecutive values of x_r as fp32 or, rounded
// to nearest even, as bf16.
template <int N>
__device__ __forceinline__ void store_xr(void* out, int out_dtype, int64_t elem, const float* v) {
    static_assert(N % 2 == 0, "pairs");
    if (out_dtype == HBL_BF16) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        uint32_t h[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i)
            h[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){v[2 * i], v[2 * i + 1]}, bf16x2));
        uint32_t* dst = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(out) + elem);
        if constexpr (N == 2) dst[0] = h[0];
        else if constexpr (N == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(h[0], h[1]);
        else {
#pragma unroll
            for (int i = 0; i < N / 8; ++i)
                store_stream16(reinterpret_cast<uint4*>(dst) + i, make_uint4(h[4 * i], h[4 * i + 1], h[4 * i + 2], h[4 * i + 3]));
        }
    } else {
        float* dst = static_cast<float*>(out) + elem;
        if constexpr (N == 2) *reinterpret_cast<float2*>(dst) = make_float2(v[0], v[1]);
        else {
#pragma unroll
            for (int i = 0; i < N / 4; ++i)
                store_stream16(reinterpret_cast<float4*>(dst) + i, make_uint4(as_u(v[4 * i]), as_u(v[4 * i + 1]), as_u(v[4 * i + 2]), as_u(v[4 * i + 3])));
        }
    }
}

// One token row per workgroup of 64*W threads (transformed rows: W = 1); `row` and `tid` come from the caller so that the grouped
// launch (several projections' rows in one grid) can run the same body.
template <int LOG2K, int W, int BITS, bool BF16, bool HADAMARD, int BLOCKB = kRecordBlockBytes>
__device__ __forceinline__ void fwht_quant_body(int64_t row, int tid, const void* __restrict__ x,
                                                int8_t* __restrict__ codes, float* __restrict__ s_dequant,
                                                int32_t* __restrict__ code_sum, RowParams rp, int code_offset) {
    const int few_rows = rp.few_rows;
    constexpr int K = 1 << LOG2K;
    constexpr int NT = 64 * W;
    constexpr int E = K / NT;            // elements per thread
    constexpr int CH = E < 8 ? E : 8;    // contiguous elements per chunk
    constexpr int R = E / CH;            // chunks per thread
    static_assert(E >= 1 && R >= 1 && (W == 1 || !HADAMARD), "transformed rows belong to one wave");

    __shared__ double red_d[W];
    __shared__ float red_f[W];
    __shared__ int red_i[W];

    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t row_off = row * (int64_t)K;
    // Position of this lane's chunks inside a group of 64.  With the transform, lane ^ (3 if bit 2 is set): flipping
    // position bit 2 then flips lane bits 0-2 together, which is the one xor-4-like permutation DPP offers inside a
    // row of 16 lanes (the half-row mirror, lane ^ 7); bits 0, 1 and 3 flip by quad permutes and a row rotation.
    const int pos = HADAMARD ? lane ^ (((lane >> 2) & 1) * 3) : lane;

    float v[R][CH];
#pragma unroll
    for (int r = 0; r < R; ++r) load_chunk<CH, BF16>(x, row_off + (int64_t)((wave * R + r) * 64 + pos) * CH, v[r]);

    if (rp.ln_gain) {   // uniform: RMS normalisation ahead of the transform
        __shared__ double red_n[W];
        double ss = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < CH; ++e) ss += (double)v[r][e] * (double)v[r][e];
        const float rn = rms_factor<W>(ss, red_n, lane, wave, K, rp.ln_eps, few_rows);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float gv[CH];
            load_chunk<CH, false>(rp.ln_gain, (int64_t)((wave * R + r) * 64 + pos) * CH, gv);
#pragma unroll
            for (int e = 0; e < CH; ++e) v[r][e] = (v[r][e] * rn) * gv[e];
        }
    }

    if constexpr (HADAMARD) {
        // e bits
#pragma unroll
        for (int h = 1; h < CH; h <<= 1)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < CH; ++e)
                    if ((e & h) == 0) {
                        const float a = v[r][e], b = v[r][e + h];
                        v[r][e] = a + b;
                        v[r][e + h] = a - b;
                    }
        // lane bits
        lane_stage_fma<0xB1>(v, pos & 1);    // lane ^ 1 (quad_perm [1,0,3,2])
        lane_stage_fma<0x4E>(v, pos & 2);    // lane ^ 2 (quad_perm [2,3,0,1])
        lane_stage_fma<0x141>(v, pos & 4);   // lane ^ 7 (row_half_mirror)
        lane_stage_fma<0x128>(v, pos & 8);   // lane ^ 8 (row_ror:8)
        lane_stage<16>(v, lane);             // (partners share position bits 0-3, hence the sign they carry)
        lane_stage<32>(v, lane);
        // r bits
#pragma unroll
        for (int h = 1; h < R; h <<= 1)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if ((r & h) == 0) {
#pragma unroll
                    for (int e = 0; e < CH; ++e) {
                        const float a = v[r][e], b = v[r + h][e];
                        v[r][e] = a + b;
                        v[r + h][e] = a - b;
                    }
                }
        // 1/sqrt(K), with the sign the lane stages left on this lane's values: (-1)^(set bits among position bits 0-3)
        const float c_n = (__builtin_popcount(pos & 15) & 1) ? -(float)(1.0 / sqrt((double)K)) : (float)(1.0 / sqrt((double)K));
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < CH; ++e) v[r][e] = v[r][e] * c_n;
    }

    if constexpr (BITS == 0) {
        // transform only (Eq. 3-4 by themselves, and the backward pass of Eq. 8): `codes` is the output
        // array and `code_offset` its element type
        static_assert(CH >= 2, "transform-only rows hold at least two elements per lane");
#pragma unroll
        for (int r = 0; r < R; ++r) {
            store_xr<CH>(codes, code_offset, row_off + (int64_t)((wave * R + r) * 64 + pos) * CH, v[r]);
        }
        return;
    }

    // per-token scale
    float gain, s_d;
    if constexpr (BITS == 8) {
        float m = 0.0f;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < CH; ++e) m = fmaxf(m, fabsf(v[r][e]));
        m = wave_max(m, few_rows);
        if constexpr (W > 1) {
            if (lane == 0) red_f[wave] = m;
            __syncthreads();
            m = red_f[0];
#pragma unroll
            for (int w = 1; w < W; ++w) m = fmaxf(m, red_f[w]);
        }
        gain = 127.0f / (m + rp.eps);
        s_d = m / 127.0f;
    } else {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < CH; ++e) s += (double)fabsf(v[r][e]);
        s = wave_sum(s, few_rows);
        if constexpr (W > 1) {
            if (lane == 0) red_d[wave] = s;
            __syncthreads();
            s = red_d[0];
#pragma unroll
            for (int w = 1; w < W; ++w) s += red_d[w];
        }
        const float beta = (float)(s / (double)K);
        gain = kRoot7 / (beta + rp.eps);
        s_d = beta / kRoot7;
    }

    // codes: clamp, then add 1.5*2^23 so that the fp32 adder rounds to the nearest (even) integer and
    // leaves its two's complement in the low mantissa bits
    constexpr float lo = BITS == 8 ? -128.0f : -8.0f;
    constexpr float hi = BITS == 8 ? 127.0f : 7.0f;
    // bf6 records (INT4, 8-element chunks only; the launcher rejects the rest) are built from code + 8
    const bool bf6 = BITS == 4 && CH == 8 && code_offset == kCodesBf6;
    if (bf6) code_offset = 8;
    // stored byte = code + code_offset: folding the offset into the rounding constant costs nothing
    const float magic = kMagic + (float)code_offset;
    int isum = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t packed[(CH + 3) / 4];
#pragma unroll
        for (int p = 0; p < (CH + 3) / 4; ++p) packed[p] = 0;
#pragma unroll
        for (int e = 0; e < CH; ++e) {
            const float y = v[r][e] * gain;
            const float t = __builtin_amdgcn_fmed3f(y, lo, hi);
            packed[e / 4] |= (as_u(t + magic) & 0xFFu) << (8 * (e % 4));
        }
        if (code_sum) {   // uniform, and off on the forward path: += the stored bytes
#pragma unroll
            for (int p = 0; p < (CH + 3) / 4; ++p) isum = __builtin_amdgcn_sdot4((int)packed[p], 0x01010101, isum, false);
        }
        const int g = wave * R + r;
        int8_t* dst = codes + row_off + (int64_t)(g * 64 + pos) * CH;
        if constexpr (CH == 8) {
            if (bf6) bf6_store_pair<BLOCKB>(codes, row, K, g * 64 + pos, bf6_pack4(packed[0]), bf6_pack4(packed[1]));
            else *reinterpret_cast<uint2*>(dst) = make_uint2(packed[0], packed[1]);
        } else if constexpr (CH == 4) {
            *reinterpret_cast<uint32_t*>(dst) = packed[0];
        } else if constexpr (CH == 2) {
            *reinterpret_cast<uint16_t*>(dst) = (uint16_t)packed[0];
        } else {
            *reinterpret_cast<uint8_t*>(dst) = (uint8_t)packed[0];
        }
    }
    if (code_sum) {
        isum = wave_sum(isum - E * code_offset, few_rows);
        if constexpr (W > 1) {
            if (lane == 0) red_i[wave] = isum;
            __syncthreads();
            isum = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) isum += red_i[w];
        }
        if (tid == 0) code_sum[row] = isum;
    }
    if (tid == 0) s_dequant[row] = s_d;
}

// Plain BitLinear front end for K that is not a power of two (K % 128 == 0, K <= 16384): the same
// quantiser with the row held as chunks of 8 elements by the threads of NW waves.
// MAXC = chunk slots per thread (K <= 512 * NW * MAXC): the launcher picks the smallest that covers the row, so
// that short rows do not walk empty slots; every MAXC performs the same arithmetic in the same order.  GROUPS: rows that a
// workgroup works on side by side, this one by the NW waves of `group`.
// All slots but the last must be full (K > 512 * NW * (MAXC - 1)): only the last one is tested for the row's end (3001 rows of
// 3072 by two waves 8.05 -> 7.68 us, 64 rows of 16256 by four 5.9 -> 5.05).
template <int BITS, bool BF16, int MAXC, int BLOCKB = kRecordBlockBytes, int NW = 4, int GROUPS = 1>
__device__ __forceinline__ void quant_generic_body(int64_t row, int tid, const void* __restrict__ x, int K,
                                                   int8_t* __restrict__ codes, float* __restrict__ s_dequant,
                                                   int32_t* __restrict__ code_sum, RowParams rp, int code_offset, int group = 0) {
    const int few_rows = rp.few_rows;
    constexpr int NT = 64 * NW;
    __shared__ double red_ds[GROUPS][NW];
    __shared__ float red_fs[GROUPS][NW];
    __shared__ int red_is[GROUPS][NW];
    double* const red_d = red_ds[GROUPS == 1 ? 0 : group];
    float* const red_f = red_fs[GROUPS == 1 ? 0 : group];
    int* const red_i = red_is[GROUPS == 1 ? 0 : group];
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t row_off = row * K;
    const int nchunks = K / 8;
    float v[MAXC][8];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int ch = c * NT + tid;
        if (c < MAXC - 1 || ch < nchunks) {
            load_chunk<8, BF16>(x, row_off + (int64_t)ch * 8, v[c]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[c][e] = 0.0f;
        }
    }
    if (rp.ln_gain) {   // uniform: RMS normalisation of the row (chunks past the row hold zeros)
        __shared__ double red_n[GROUPS][NW];
        double ss = 0.0;
#pragma unroll
        for (int c = 0; c < MAXC; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) ss += (double)v[c][e] * (double)v[c][e];
        const float rn = rms_factor<NW>(ss, red_n[GROUPS == 1 ? 0 : group], lane, wave, K, rp.ln_eps, few_rows);
#pragma unroll
        for (int c = 0; c < MAXC; ++c) {
            const int ch = c * NT + tid;
            if (c < MAXC - 1 || ch < nchunks) {
                float gv[8];
                load_chunk<8, false>(rp.ln_gain, (int64_t)ch * 8, gv);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[c][e] = (v[c][e] * rn) * gv[e];
            }
        }
    }
    float gain, s_d;
    if constexpr (BITS == 8) {
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < MAXC; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(v[c][e]));
        m = wave_max(m, few_rows);
        if constexpr (NW > 1) {
            if (lane == 0) red_f[wave] = m;
            __syncthreads();
            m = red_f[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) m = fmaxf(m, red_f[w]);
        }
        gain = 127.0f / (m + rp.eps);
        s_d = m / 127.0f;
    } else {
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < MAXC; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) s += (double)fabsf(v[c][e]);
        s = wave_sum(s, few_rows);
        if constexpr (NW > 1) {
            if (lane == 0) red_d[wave] = s;
            __syncthreads();
            s = red_d[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) s += red_d[w];
        }
        const float beta = (float)(s / (double)K);
        gain = kRoot7 / (beta + rp.eps);
        s_d = beta / kRoot7;
    }
    constexpr float lo = BITS == 8 ? -128.0f : -8.0f;
    constexpr float hi = BITS == 8 ? 127.0f : 7.0f;
    const bool bf6 = BITS == 4 && code_offset == kCodesBf6;   // bf6 records are built from code + 8
    if (bf6) code_offset = 8;
    // stored byte = code + code_offset: folding the offset into the rounding constant costs nothing
    const float magic = kMagic + (float)code_offset;
    int isum = 0;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int ch = c * NT + tid;
        if (c < MAXC - 1 || ch < nchunks) {
            uint32_t packed[2] = {0u, 0u};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float t = __builtin_amdgcn_fmed3f(v[c][e] * gain, lo, hi);
                packed[e / 4] |= (as_u(t + magic) & 0xFFu) << (8 * (e % 4));
            }
            if (code_sum) {   // uniform, and off on the forward path: += the stored bytes
                isum = __builtin_amdgcn_sdot4((int)packed[0], 0x01010101, isum - 8 * code_offset, false);
                isum = __builtin_amdgcn_sdot4((int)packed[1], 0x01010101, isum, false);
            }
            // K / 8 is a multiple of 16: the lanes of a quad are in or out of this branch together
            if (bf6) bf6_store_pair<BLOCKB>(codes, row, K, ch, bf6_pack4(packed[0]), bf6_pack4(packed[1]));
            else *reinterpret_cast<uint2*>(codes + row_off + (int64_t)ch * 8) = make_uint2(packed[0], packed[1]);
        }
    }
    if (code_sum) {
        isum = wave_sum(isum, few_rows);
        if constexpr (NW > 1) {
            if (lane == 0) red_i[wave] = isum;
            __syncthreads();
            isum = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) isum += red_i[w];
        }
        if (tid == 0) code_sum[row] = isum;
    }
    if (tid == 0) s_dequant[row] = s_d;
}

}  // namespace
}  // namespace hbl
