// One-launch form of the forward pass for short rows and up to 16 tokens (K <= 3584, both widths, with or without the transform
// and the norm; fused_small.hip is asked first).
//
// Such a projection is two launches of 2.2 to 2.9 us each, nearly all of it start-up and drain, and on the host two launches
// where one takes as long as the rest of the call.  Here every workgroup (32 output rows) requests its weights, quantises all
// rows for itself - one wave per row, side by side, with the bodies of the quantiser launches - into bytes in LDS, and
// multiplies them on the int8 matrix cores.  The sums are the same integers as on the other paths.
//
// Bound: one serial chain - launch, a row's loads, transform and two reductions across the wave, LDS, MFMA, a sum over the waves.
// 16 fp32 rows of 256 against 256 output rows, transformed: 3.5 us of GPU time for 5.2 with two launches, 5.3 us for 9.3 called
// one after another from the host.
#include "quant_bodies.h"

namespace hbl {
namespace {

using gemm::lds_dma16;
using gemm::v4i;

constexpr int kFusedTokens = 16, kFusedLength = 3584;

struct FusedBytesArgs {
    const void* x;
    const uint32_t* packed;
    const float* w_scales;
    uint16_t* y;
    int T, K, N;
    int rows_per_group;
    RowParams rp;
};

// Bytes of a token's codes in LDS: 16 more than the row, so that 16 tokens' reads start in different banks.
constexpr int code_row_bytes(int K) { return K + 16; }

// LOG2K: transformed rows of 2^LOG2K (7..11); 0: plain rows of up to 512 * MAXC.  WAVES >= T.
template <int LOG2K, int MAXC, int BITS, bool BF16, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void fused_bytes_kernel(const FusedBytesArgs a) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ float s_d[WAVES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = LOG2K ? 1 << LOG2K : a.K;
    const int nkb = K / 128, row_bytes = code_row_bytes(K);
    char* const weights = lds;                              // nkb tiles of 1 KiB, later the waves' sums
    char* const codes = lds + (nkb > WAVES ? nkb : WAVES) * 1024;

    // 1. the weights of this workgroup's 32 rows
    const size_t wstride = (size_t)(a.N / 32) * 1024;
    const char* const w0 = reinterpret_cast<const char*>(a.packed) + (size_t)blockIdx.x * 1024;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)weights;
    for (int kb = wave; kb < nkb; kb += WAVES) lds_dma16(lds0 + kb * 1024, w0 + kb * wstride, lane * 16);

    // 2. a row per wave (no barrier inside: one-wave bodies)
    if (wave < a.T) {
        const void* x = static_cast<const char*>(a.x) + (size_t)wave * K * (BF16 ? 2 : 4);
        int8_t* dst = reinterpret_cast<int8_t*>(codes + wave * row_bytes);
        if constexpr (LOG2K != 0) fwht_quant_body<LOG2K, 1, BITS, BF16, true>(0, lane, x, dst, s_d + wave, nullptr, a.rp, 0);
        else quant_generic_body<BITS, BF16, MAXC, kRecordBlockBytes, 1>(0, lane, x, K, dst, s_d + wave, nullptr, a.rp, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wave's weights have landed
    __syncthreads();

    // 3. 16x16x64 MFMAs: wave w multiplies half w & 1 of the 32 rows, K-blocks w >> 1, (w >> 1) + WAVES / 2, ...; lane = (token
    // lane & 15, group g = lane >> 4 of 16 features of a 64-feature step)
    const int g = lane >> 4, r = lane & 15, half = wave & 1;
    const char* const crow = codes + (r < a.T ? r : 0) * row_bytes + 16 * g;
    const char* const wrow = weights + ((r + 16 * half + 32 * (g >> 1)) * 4 + (g & 1)) * 4;
    v4i acc = {0, 0, 0, 0};
    for (int kb = wave >> 1; kb < nkb; kb += WAVES / 2)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const v4i c = *reinterpret_cast<const v4i*>(crow + kb * 128 + s * 64);
            const uint32_t p = *reinterpret_cast<const uint32_t*>(wrow + kb * 1024 + s * 8);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(gemm::expand_weights_i8(p), c, acc, 0, 0, 0);
        }
    __syncthreads();                                        // every wave is done with the weights
    v4i* const sums = reinterpret_cast<v4i*>(weights);
    if (wave >= 2) sums[wave * 64 + lane] = acc;
    __syncthreads();
    if (wave >= 2 || r >= a.T) return;
#pragma unroll
    for (int w = 2; w < WAVES; w += 2) acc += sums[(w + half) * 64 + lane];
    const int n = blockIdx.x * 32 + half * 16 + 4 * g;
    *reinterpret_cast<uint2*>(a.y + (size_t)r * a.N + n) = gemm::dequant_quad(acc, s_d[r], a.w_scales[n / a.rows_per_group], 0, nullptr);
}

template <int LOG2K, int MAXC, int BITS, bool BF16, int WAVES>
int launch_cfg(const FusedBytesArgs& a, hipStream_t stream) {
    const int nkb = a.K / 128;
    const size_t lds = (size_t)(nkb > WAVES ? nkb : WAVES) * 1024 + (size_t)a.T * code_row_bytes(a.K);   // at most 85 KiB
    constexpr auto kern = fused_bytes_kernel<LOG2K, MAXC, BITS, BF16, WAVES>;
    constexpr int longest = LOG2K ? 1 << LOG2K : 512 * MAXC;   // (16 rows of 2048 are 256 bytes beyond 48 KiB)
    constexpr size_t most = (longest / 128 > WAVES ? longest / 128 : WAVES) * 1024 + WAVES * code_row_bytes(longest);
    if (const int rc = allow_dynamic_lds<kern, most>(); rc != HBL_OK) return rc;
    launch_kernel("fused_bytes_kernel", kern, dim3((unsigned)(a.N / 32)), dim3(64 * WAVES), lds, stream, a);
    return after_launch();
}
template <int LOG2K, int MAXC, int BITS, bool BF16>
int launch_waves(const FusedBytesArgs& a, hipStream_t stream) {
    if (a.T <= 4) return launch_cfg<LOG2K, MAXC, BITS, BF16, 4>(a, stream);
    if (a.T <= 8) return launch_cfg<LOG2K, MAXC, BITS, BF16, 8>(a, stream);
    return launch_cfg<LOG2K, MAXC, BITS, BF16, 16>(a, stream);
}
template <int BITS, bool BF16>
int launch_rows(const FusedBytesArgs& a, bool hadamard, hipStream_t stream) {
    if (!hadamard) {
        switch ((a.K + 511) / 512) {
            case 1: return launch_waves<0, 1, BITS, BF16>(a, stream);
            case 2: return launch_waves<0, 2, BITS, BF16>(a, stream);
            case 3: return launch_waves<0, 3, BITS, BF16>(a, stream);
            case 4: return launch_waves<0, 4, BITS, BF16>(a, stream);
            case 5: return launch_waves<0, 5, BITS, BF16>(a, stream);
            case 6: return launch_waves<0, 6, BITS, BF16>(a, stream);
            case 7: return launch_waves<0, 7, BITS, BF16>(a, stream);
            default: return HBL_E_SHAPE;
        }
    }
    switch (a.K) {
        case 128: return launch_waves<7, 0, BITS, BF16>(a, stream);
        case 256: return launch_waves<8, 0, BITS, BF16>(a, stream);
        case 512: return launch_waves<9, 0, BITS, BF16>(a, stream);
        case 1024: return launch_waves<10, 0, BITS, BF16>(a, stream);
        case 2048: return launch_waves<11, 0, BITS, BF16>(a, stream);
        default: return HBL_E_SHAPE;
    }
}

}  // namespace

// Every workgroup quantises all rows, so what one launch costs grows with the workgroups a CU runs one after another and with
// the waves of each; the second launch that it saves costs the same throughout.  The line: 1024 workgroups of 4 waves, 512 of 8
// or 256 of 16 (each 4 waves a SIMD).  One launch against two, INT4 and INT8, transformed and plain, K 128 to 1024, on the near
// side of it: 0.47 to 0.95 of the time (us: T = 1, K = 1024, N = 4096, INT8 transformed 3.74 for 7.19; T = 16 5.25 for 7.33;
// INT4 K = 256, T = 4, N = 8192 3.08 for 5.62; T = 8, K = 1024, N = 16384 6.09 for 6.43).  Beyond it: T = 4, N = 65536 0.80 to
// 1.12, T = 8, N = 32768 0.80 to 1.41, T = 16, N = 16384 0.75 to 1.31.  Rows of records (INT4, K >= 512) have the faster second
// launch: four of 1024 against N = 32768 take 6.73 for 6.36, three 5.83 for 6.32.  One to four of them that fused_small.hip
// takes are its.
// Rows of 1152 to 2048: plain ones 0.46 to 0.98 on the near side (INT8, K = 1536, T = 16, N = 4096 4.11 for 7.79; INT4, K = 1920,
// T = 8, N = 8192 4.36 for 6.66), beyond it T = 4 1.00 to 1.14 (INT4; INT8 0.71 to 0.81 at N = 32768, taken), T = 8 0.87 to 1.34,
// T = 16 0.75 to 1.39.  A transform of 2048 in one wave is the longer chain: up to 8 rows and 256 workgroups 0.71 to 0.96,
// 16 rows 0.95 to 1.30, N = 16384 0.79 to 1.43.
// Plain rows of 2176 to 3584 (up to 56 values a lane): 0.56 to 0.95 on the near side (INT8, K = 3072, T = 8, N = 8192 4.91 for
// 7.89; INT4 5.17 for 6.72), beyond it INT4 T = 5 to 8 0.91 to 1.07, T = 16 1.39 to 1.58, INT8 T = 16 1.09 to 1.23.  Rows of 4096:
// INT4, T = 16 1.05 to 1.13 and spills; they stay two launches.
// The norm (double-precision squares, a reduction and the gains' loads) is repeated in every workgroup too.  With it, 2800 sizes: INT4
// by values in all rows, 16 x 1536 0.80 to 0.88, 12 x 2560 0.89 to 0.96;  up to 4096 output rows and 8192, 9 x 3584 0.95 to 0.98 and 1.02,
// 16 x 2048 0.97 to 1.02 and 1.06, 12 x 3072 0.94 to 0.98 and 1.03, 16 x 3072 1.02 to 1.11 and 1.15;  five to eight rows against 8224 to 16384 output rows, INT4: 1536 0.85 to 0.96, 2048 1.00 to 1.15,
// transformed 1024 7 x 0.97, 8 x 1.03, INT8: 8 x 2560 0.93 to 0.97, 8 x 3072 1.00 to 1.03, 8 x 3584 1.04 to 1.08;  transformed rows of
// 2048, INT4, five to eight: up to 4096 output rows 0.95 to 1.00, 8192 1.02 to 1.05.
bool fused_bytes_preferred(int64_t T, int64_t K, int64_t N, int bits, bool hadamard, bool norm) {
    if (T > kFusedTokens || K > kFusedLength) return false;
    const int64_t values = T * K;
    if (norm && bits == 4 && (values > (N > 4096 ? 31744 : 36864) || (hadamard && K > 1024 && T > 4 && N > 4096))) return false;
    const bool heavy = norm && (bits == 8 ? values > 23552 : K > 1536 || (hadamard && values > 7168));
    const int64_t eight = heavy ? 256 : 512;   // workgroups for five to eight rows
    if (K > 2048) return !hadamard && N / 32 <= (T <= 8 && bits == 8 ? eight : 256);
    if (K > 1024) return hadamard ? T <= 8 && N / 32 <= 256 : N / 32 <= (T <= 4 ? (bits == 8 ? 1024 : 512) : T <= 8 ? eight : 256);
    const int few = bits == 4 && K >= 512 && values >= 4096 ? 3 : 4;
    return N / 32 <= (T <= few ? 1024 : T <= 4 ? 512 : T <= 8 ? eight : 256);
}

int launch_fused_bytes(const void* x, int x_dtype, int64_t T, int64_t K, const void* packed, int64_t N, const float* w_scales,
                       int64_t groups, int bits, float eps, bool hadamard, const float* ln_gain, float ln_eps, void* y,
                       hipStream_t stream) {
    FusedBytesArgs a = {};
    a.x = x;
    a.packed = static_cast<const uint32_t*>(packed);
    a.w_scales = w_scales;
    a.y = static_cast<uint16_t*>(y);
    a.T = (int)T;
    a.K = (int)K;
    a.N = (int)N;
    a.rows_per_group = (int)(N / groups);
    a.rp = RowParams{eps, ln_gain, ln_eps, 1};
    const bool bf = x_dtype == HBL_BF16;
    if (bits == 8) return bf ? launch_rows<8, true>(a, hadamard, stream) : launch_rows<8, false>(a, hadamard, stream);
    return bf ? launch_rows<4, true>(a, hadamard, stream) : launch_rows<4, false>(a, hadamard, stream);
}

}  // namespace hbl
