// Weight set-up kernels: the per-tensor absmean ternary quantiser (Eq. 1-2) and the
// 2-bit packing of its codes into the streaming layout the GEMM kernels read.
//
// Packed layout (one form, 2 bits per weight, read by every GEMM kernel).  The [N, K] code matrix is cut into
// tiles of 32 output rows x 128 input features, stored K-block-major (all row tiles of features 0..127, then
// all of 128..255, ...):
//   tile(nt, kb) at byte ((kb * (N/32) + nt) * 1024), nt = o / 32, kb = k / 128,
// so that a prefill workgroup's stage (16 row tiles of one K-block) is one contiguous 16 KiB piece and the waves
// of a small-batch launch, each walking the K range of its own row tile, together sweep memory linearly.
// A tile is 64 lanes x 4 dwords (lane-major, 16 bytes per lane).  Lane l, dword j holds the 16 weights of
// row 32*nt + (l & 31) at features
//   k = 128*kb + 64*(j >> 1) + 32*(l >> 5) + 16*(j & 1) + i,  i = 0..15,
// i.e. dwords 2s, 2s+1 are one lane's share of the A operand of a 32x32x64 fp6/fp4 MFMA for K-step s, and
// dword j one lane's share of a 32x32x32 int8 MFMA operand.  A weight is a (sign, magnitude) bit pair:
// weight i < 8 has its magnitude at bit 4*i + 1 and its sign at bit 4*i + 3, weight i >= 8 its magnitude at
// bit 4*(i-8) and its sign at bit 4*(i-8) + 2.  Then
//   p & 0xAAAAAAAA  and  (p << 1) & 0xAAAAAAAA
// are eight fp4 (e2m1) values each (+-1.0 = s010, 0 = 0000), and (p >> {0,1,4,5}) & 0x05050505 are four
// weights each as byte values {0, 1, 5} that one byte-permute look-up turns into int8 {0, +1, -1}.
// After the N*K/4 bytes of tiles come N int32 row sums sum_k c[o][k] (the epilogue of the int8 path needs
// them when activation codes are stored with an offset).
#include "hbl_internal.h"

namespace hbl {
namespace {

constexpr int kSumBlock = 256;
constexpr int kSumItems = 16;       // floats per thread and chunk
constexpr int kChunk = kSumBlock * kSumItems;
constexpr int kSumGrid = 2048;      // most workgroups of the sum = most partial sums

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Floats [4q, 4q + 4) of W.  VEC: W is 16-byte aligned; else four 4-byte loads of the same floats.  Only whole quads.
template <bool VEC>
__device__ __forceinline__ f32x4 load_quad(const float* __restrict__ W, int64_t q) {
    if constexpr (VEC) return reinterpret_cast<const f32x4*>(W)[q];
    else return f32x4{W[4 * q], W[4 * q + 1], W[4 * q + 2], W[4 * q + 3]};
}

// Sum of one fp64 value per thread over the workgroup, in a fixed order; every thread gets it.  `red`: a double per wave.
__device__ __forceinline__ double workgroup_sum(double s, double* red) {
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) s += __shfl_xor(s, sft, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int w = 1; w < kSumBlock / 64; ++w) t += red[w];
    return t;
}

// Eq. 1: partial sums of |W| in fp64, one per workgroup, in an order that depends on the sizes alone.  Bound by the
// read of W: a thread keeps four 16-byte loads in flight and walks chunks of 4096 floats (4096 x 16384 weights: 46 us =
// 5.8 TB/s; with 4-byte loads and a workgroup per chunk it was 80 us, and one more launch of 17 us added 16384 sums).
template <bool VEC>
__global__ __launch_bounds__(kSumBlock) void abs_sum_partial_kernel(const float* __restrict__ W, int64_t count,
                                                                    double* __restrict__ partial) {
    __shared__ double red[kSumBlock / 64];
    double s = 0.0;
    const int64_t chunks = count / kChunk;
    for (int64_t c = blockIdx.x; c < chunks; c += gridDim.x) {
        f32x4 w[kSumItems / 4];
#pragma unroll
        for (int i = 0; i < kSumItems / 4; ++i) w[i] = load_quad<VEC>(W, c * (kChunk / 4) + i * kSumBlock + threadIdx.x);
#pragma unroll
        for (int i = 0; i < kSumItems / 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) s += (double)fabsf(w[i][e]);
    }
    if (blockIdx.x == 0)   // the floats beyond the last whole chunk
        for (int64_t i = chunks * kChunk + threadIdx.x; i < count; i += kSumBlock) s += (double)fabsf(W[i]);
    s = workgroup_sum(s, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Code of one weight: RoundClip(w / denom, -1, 1).  For a normal denom the rounded quotient fl(w / denom) exceeds 1/2
// exactly when w > denom / 2: the next float above denom / 2 already lies more than half an ulp(1/2) of quotient
// above 1/2, and 1/2 itself rounds to the even 0.  So two compares stand for the IEEE division, the rounding and
// the clip.  (denom tiny, zero, negative, infinite or NaN: `divide`, the formula itself.)
__device__ __forceinline__ uint32_t ternary_code(float w, float denom, float half, bool divide) {
    if (divide) {
        const float r = fminf(fmaxf(rintf(w / denom), -1.0f), 1.0f);
        return (uint32_t)(uint8_t)(int8_t)(int)r;
    }
    return w > half ? 0x01u : (w < -half ? 0xFFu : 0x00u);
}

// Eq. 1-2: alpha = mean |W| from the partial sums (each workgroup adds all of them, in one fixed order, so no launch
// of its own is needed; at most 16 KiB out of L2), then codes = RoundClip(W / (alpha + eps), -1, 1).  The chunks are
// walked from the end: the memory-side cache still holds the last ones that the sum has read (1 % of the three
// launches).  4096 x 16384 weights: 55 us = 6.1 TB/s; one weight per step with a division and a byte store was 85 us.
// VEC: W is 16-byte and codes 4-byte aligned.
template <bool VEC>
__global__ __launch_bounds__(kSumBlock) void ternarize_kernel(const float* __restrict__ W, int64_t count,
                                                              const double* __restrict__ partial, int nparts, float eps,
                                                              float* __restrict__ alpha, int8_t* __restrict__ codes) {
    __shared__ double red[kSumBlock / 64];
    double s = 0.0;
    for (int i = threadIdx.x; i < nparts; i += kSumBlock) s += partial[i];
    const float mean = (float)(workgroup_sum(s, red) / (double)count);
    if (blockIdx.x == 0 && threadIdx.x == 0) *alpha = mean;
    const float denom = mean + eps, half = 0.5f * denom;
    const bool divide = !(denom >= 0x1p-100f && denom <= 0x1p100f);   // uniform
    const int64_t chunks = count / kChunk;
    for (int64_t c = chunks - 1 - blockIdx.x; c >= 0; c -= gridDim.x) {
        f32x4 w[kSumItems / 4];
#pragma unroll
        for (int i = 0; i < kSumItems / 4; ++i) w[i] = load_quad<VEC>(W, c * (kChunk / 4) + i * kSumBlock + threadIdx.x);
#pragma unroll
        for (int i = 0; i < kSumItems / 4; ++i) {
            const int64_t q = c * (kChunk / 4) + i * kSumBlock + threadIdx.x;
            uint32_t b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = ternary_code(w[i][e], denom, half, divide);
            if constexpr (VEC) {
                reinterpret_cast<uint32_t*>(codes)[q] = b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) codes[4 * q + e] = (int8_t)b[e];
            }
        }
    }
    if (blockIdx.x == gridDim.x - 1)
        for (int64_t i = chunks * kChunk + threadIdx.x; i < count; i += kSumBlock)
            codes[i] = (int8_t)ternary_code(W[i], denom, half, divide);
}

// dword d of the packed stream -> (row, first feature) of its 16 weights
__device__ __forceinline__ void packed_dword_origin(int64_t d, int64_t N, int64_t* row, int64_t* k0) {
    const int64_t ntiles = N / 32;
    const int dd = (int)(d & 3);
    const int lane = (int)((d >> 2) & 63);
    const int64_t tile = d >> 8;
    const int64_t kb = tile / ntiles, nt = tile % ntiles;
    *row = nt * 32 + (lane & 31);
    *k0 = kb * 128 + (dd >> 1) * 64 + (lane >> 5) * 32 + (dd & 1) * 16;
}

__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t* __restrict__ packed, int64_t N, int64_t K,
                                                     int8_t* __restrict__ codes) {
    const int64_t total = (N / 32) * (K / 128) * 256;
    const int64_t d = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (d >= total) return;
    int64_t row, k0;
    packed_dword_origin(d, N, &row, &k0);
    const uint32_t p = packed[d];
    uint4 raw;
    int8_t* c = reinterpret_cast<int8_t*>(&raw);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
        const int ma = (p >> (4 * n + 1)) & 1, sa = (p >> (4 * n + 3)) & 1;
        const int mb = (p >> (4 * n)) & 1, sb = (p >> (4 * n + 2)) & 1;
        c[n] = (int8_t)(sa ? -ma : ma);
        c[8 + n] = (int8_t)(sb ? -mb : mb);
    }
    *reinterpret_cast<uint4*>(codes + row * K + k0) = raw;
}

// Four codes (one byte each) -> their four nibbles: magnitude (code != 0) at bit 1, sign (code < 0) at bit 3.
__device__ __forceinline__ uint32_t weight_nibbles(uint32_t c) {
    const uint32_t nonzero = (((c & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | c) & 0x80808080u;
    uint32_t v = (nonzero >> 6) | ((c & 0x80808080u) >> 4);
    v = (v | (v >> 4)) & 0x00FF00FFu;
    return (v | (v >> 8)) & 0xFFFFu;
}

// Packs eight output rows and adds up their codes.  A wave reads 8 rows x 128 features per load (eight whole
// 128-byte lines), a lane's 16 codes are one packed dword, and the wave's store is two pieces of 128 bytes of the
// tile; the waves of the workgroup take the K-blocks in turn.  The row sums sum_k c[o][k] come from the same read.
// Bound by the read of the codes: 16 us for 4096 x 16384 (5.2 TB/s; 8 loads in flight measured the same); with
// scattered 16-byte loads and a launch of its own for the row sums it was 22 + 13 us.
constexpr int kPackRows = 8, kPackWaves = 8, kPackAhead = 4;   // rows per workgroup, most waves, loads in flight per wave
__global__ __launch_bounds__(64 * kPackWaves) void pack_kernel(const int8_t* __restrict__ codes, int64_t N, int64_t K,
                                                               uint32_t* __restrict__ packed,
                                                               int32_t* __restrict__ row_sum) {
    __shared__ int red[kPackWaves][kPackRows];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int nkb = (int)(K / 128);
    const int64_t row = (int64_t)blockIdx.x * kPackRows + (lane >> 3);
    const int chunk = lane & 7;   // 16 features
    // dword j of tile lane l covers features 64 (j >> 1) + 32 (l >> 5) + 16 (j & 1) + 0..15 of row l & 31
    const int dword = ((int)(row & 31) + 32 * ((chunk >> 1) & 1)) * 4 + 2 * (chunk >> 2) + (chunk & 1);
    const int8_t* src = codes + row * K + chunk * 16;
    uint32_t* dst = packed + (row / 32) * 256 + dword;
    const int64_t kb_stride = (N / 32) * 256;
    int sum = 0;
    for (int kb = wave; kb < nkb; kb += waves * kPackAhead) {
        uint4 c[kPackAhead];
#pragma unroll
        for (int u = 0; u < kPackAhead; ++u) {
            c[u] = make_uint4(0, 0, 0, 0);
            if (kb + u * waves < nkb) c[u] = *reinterpret_cast<const uint4*>(src + (int64_t)(kb + u * waves) * 128);
        }
#pragma unroll
        for (int u = 0; u < kPackAhead; ++u) {
            sum = __builtin_amdgcn_sdot4((int)c[u].x, 0x01010101, sum, false);
            sum = __builtin_amdgcn_sdot4((int)c[u].y, 0x01010101, sum, false);
            sum = __builtin_amdgcn_sdot4((int)c[u].z, 0x01010101, sum, false);
            sum = __builtin_amdgcn_sdot4((int)c[u].w, 0x01010101, sum, false);
            // weights 0..7 of the dword at bits 1 and 3 of a nibble, weights 8..15 at bits 0 and 2
            const uint32_t a = weight_nibbles(c[u].x) | (weight_nibbles(c[u].y) << 16);
            const uint32_t b = weight_nibbles(c[u].z) | (weight_nibbles(c[u].w) << 16);
            if (kb + u * waves < nkb) dst[(int64_t)(kb + u * waves) * kb_stride] = a | (b >> 1);
        }
    }
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) sum += __shfl_xor(sum, m, 64);
    if (chunk == 0) red[wave][lane >> 3] = sum;
    __syncthreads();
    if (threadIdx.x < kPackRows) {
        int t = 0;
        for (int w = 0; w < waves; ++w) t += red[w][threadIdx.x];
        row_sum[(int64_t)blockIdx.x * kPackRows + threadIdx.x] = t;
    }
}

// Workgroups (= partial sums) of the absolute sum.
int64_t sum_blocks(int64_t count) {
    const int64_t chunks = (count + kChunk - 1) / kChunk;
    return chunks < kSumGrid ? chunks : kSumGrid;
}

}  // namespace

size_t ternarize_workspace_bytes(int64_t count) { return round_up((size_t)sum_blocks(count) * sizeof(double), 256); }

int launch_ternarize(const float* W, int64_t count, float eps, int8_t* codes, float* alpha, void* workspace,
                     hipStream_t stream) {
    double* partial = static_cast<double*>(workspace);
    const int nb = (int)sum_blocks(count);
    // any float-aligned W and any codes pointer are taken; the wide accesses need 16 and 4 bytes
    const bool wide_in = aligned16(W), wide = wide_in && (reinterpret_cast<uintptr_t>(codes) & 3u) == 0;
    if (wide_in) launch_kernel("abs_sum_partial_kernel", abs_sum_partial_kernel<true>, dim3(nb), dim3(kSumBlock), 0, stream, W, count, partial);
    else launch_kernel("abs_sum_partial_kernel", abs_sum_partial_kernel<false>, dim3(nb), dim3(kSumBlock), 0, stream, W, count, partial);
    const int rc = after_launch();
    if (rc != HBL_OK) return rc;
    if (wide) launch_kernel("ternarize_kernel", ternarize_kernel<true>, dim3(nb), dim3(kSumBlock), 0, stream, W, count, partial, nb, eps, alpha, codes);
    else launch_kernel("ternarize_kernel", ternarize_kernel<false>, dim3(nb), dim3(kSumBlock), 0, stream, W, count, partial, nb, eps, alpha, codes);
    return after_launch();
}

int launch_pack(const int8_t* codes, int64_t N, int64_t K, void* packed, hipStream_t stream) {
    int32_t* row_sum = reinterpret_cast<int32_t*>(static_cast<char*>(packed) + packed_tile_bytes(N, K));
    const int64_t nkb = K / 128;
    const int waves = nkb < kPackWaves ? (int)nkb : kPackWaves;
    launch_kernel("pack_kernel", pack_kernel, dim3((unsigned)(N / kPackRows)), dim3(64 * waves), 0, stream, codes, N, K,
                  static_cast<uint32_t*>(packed), row_sum);
    return after_launch();
}

int launch_unpack(const void* packed, int64_t N, int64_t K, int8_t* codes, hipStream_t stream) {
    const int64_t total = (N / 32) * (K / 128) * 256;
    launch_kernel("unpack_kernel", unpack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const uint32_t*>(packed), N, K, codes);
    return after_launch();
}

}  // namespace hbl
