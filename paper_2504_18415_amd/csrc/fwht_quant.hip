// Activation front end of H-BitLinear (Section 2.1): online Hadamard transform
// (Eq. 3-4) fused with the per-token INT8 absmax / INT4 absmean quantiser
// (Eq. 5-6).  One workgroup owns one token row; the row never leaves registers
// / LDS between the load of x and the store of the int8 codes.
//
// Arithmetic contract (what makes the codes reproducible bit for bit):
//   - butterflies are single fp32 adds / subtracts, stages in ascending stride
//     order 1,2,4,...,K/2 - which stage runs in registers, across lanes or
//     through LDS does not change any value;
//   - one multiply by c_n = (float)(1/sqrt(K)) after the last stage;
//   - gamma = max|x_r| (exact); beta = (float)(sum|x_r| in fp64 / K);
//   - gain = 127/(gamma+eps) or sqrt7/(beta+eps) with IEEE fp32 division,
//     code = RoundClip(gain * x_r) with round-half-to-even.
//
// Index bits of a row of K = CH*64*R*W elements, low to high:
//   [e: log2 CH in-thread][lane: 6][r: log2 R in-thread chunks][wave: log2 W]
// so that every global access is one contiguous CH-element piece per lane and
// the stage order e -> lane -> r -> wave is ascending.  The wave stages swap
// the wave bits with the low r bits through LDS once, then run in registers.
#include <atomic>

#include "quant_bodies.h"

namespace hbl {
namespace {

template <int LOG2K, int W, int BITS, bool BF16, bool HADAMARD>
__global__ __launch_bounds__(64 * W) void fwht_quant_kernel(const void* __restrict__ x, int8_t* __restrict__ codes,
                                                            float* __restrict__ s_dequant,
                                                            int32_t* __restrict__ code_sum, RowParams rp, int code_offset) {
    fwht_quant_body<LOG2K, W, BITS, BF16, HADAMARD>(blockIdx.x, threadIdx.x, x, codes, s_dequant, code_sum, rp,
                                                    code_offset);
}

template <int LOG2K, int W, int BITS, bool BF16, bool HADAMARD>
int launch_one(const void* x, int64_t T, int8_t* codes, float* s_dequant, int32_t* code_sum, RowParams rp,
               int code_offset, hipStream_t stream) {
    constexpr int K = 1 << LOG2K;
    const size_t lds = (HADAMARD && W > 1) ? sizeof(float) * K : 0;
    auto kern = fwht_quant_kernel<LOG2K, W, BITS, BF16, HADAMARD>;
    static std::atomic<uint64_t> lds_allowed{0};   // per instantiation: devices already set up
    if (const int rc = allow_dynamic_lds(kern, lds, lds_allowed); rc != HBL_OK) return rc;
    launch_kernel("fwht_quant_kernel", kern, dim3((unsigned)T), dim3(64 * W), lds, stream, x, codes, s_dequant, code_sum, rp, code_offset);
    return after_launch();
}

template <int BITS, bool BF16, int MAXC>
__global__ __launch_bounds__(256) void quant_generic_kernel(const void* __restrict__ x, int K,
                                                            int8_t* __restrict__ codes,
                                                            float* __restrict__ s_dequant,
                                                            int32_t* __restrict__ code_sum, RowParams rp, int code_offset) {
    quant_generic_body<BITS, BF16, MAXC>(blockIdx.x, threadIdx.x, x, K, codes, s_dequant, code_sum, rp, code_offset);
}

template <int BITS, bool BF16>
void launch_generic_slots(const void* x, int64_t T, int64_t K, RowParams rp, int8_t* codes, float* s_dequant,
                          int32_t* code_sum, int code_offset, hipStream_t stream) {
    const dim3 grid((unsigned)T), block(256);
    const int64_t per_thread = (K / 8 + 255) / 256;   // 8-element chunks per thread
#define HBL_GENERIC(MAXC)                                                                                     \
    launch_kernel("quant_generic_kernel", (quant_generic_kernel<BITS, BF16, MAXC>), grid, block, 0, stream, x, (int)K, codes, s_dequant, \
                       code_sum, rp, code_offset)
    if (per_thread <= 1) HBL_GENERIC(1);
    else if (per_thread <= 2) HBL_GENERIC(2);
    else if (per_thread <= 4) HBL_GENERIC(4);
    else HBL_GENERIC(8);
#undef HBL_GENERIC
}

int launch_generic(const void* x, int x_dtype, int64_t T, int64_t K, int bits, RowParams rp, int8_t* codes,
                   float* s_dequant, int32_t* code_sum, int code_offset, hipStream_t stream) {
    const bool bf = x_dtype == HBL_BF16;
    if (bits == 8) {
        if (bf) launch_generic_slots<8, true>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
        else    launch_generic_slots<8, false>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
    } else {
        if (bf) launch_generic_slots<4, true>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
        else    launch_generic_slots<4, false>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
    }
    return after_launch();
}


// ---------------------------------------------------------------------------------------------

// Each workgroup walks rows blockIdx.x, blockIdx.x + gridDim.x, ...; the grid is sized to what the chip holds
// at once (the LDS row buffer allows only a few workgroups per CU), and the next row's loads are issued
// under the tail of the current row's arithmetic so that their latency is not exposed once per row.  The
// compiler also moves the ~100 per-thread LDS and global address computations out of the row loop and keeps
// them in registers (about 200 VGPRs in all): measured 7-20 % faster than recomputing them per row, and the
// LDS row buffer limits the workgroups per CU before the registers do.
// FEW: at most kFewRows rows - one row per workgroup and the short-latency reductions.
template <int LOG2K, int BITS, bool BF16, bool BF6OUT, bool NORM, bool FEW>
__global__ __launch_bounds__((1 << LOG2K) / 64, 2) void fwht_quant_bigrow_kernel(
    const void* __restrict__ x, int64_t T, int8_t* __restrict__ codes, float* __restrict__ s_dequant,
    int32_t* __restrict__ code_sum, RowParams rp, int code_offset) {
    int64_t row = blockIdx.x;
    BigRowRaw<BF16> cur;
    extern __shared__ __attribute__((aligned(16))) float row_lds[];   // K floats
    if constexpr (FEW && kRowThroughLds<LOG2K, BF16>) {
        bigrow_load_lds<LOG2K, BF16>(x, row, threadIdx.x, reinterpret_cast<char*>(row_lds), cur);
    } else {
        bigrow_load<LOG2K, BF16>(x, row, threadIdx.x, cur);
    }
    if constexpr (BITS == 0 || FEW) {   // (transform only: the row loop would cost it registers it lacks)
        fwht_quant_bigrow_body<LOG2K, BITS, BF16, BF6OUT, NORM>(row, threadIdx.x, cur, row_lds, codes, s_dequant, code_sum, rp,
                                                                code_offset);
        return;
    }
    for (;;) {
        const int64_t next = row + gridDim.x;
        BigRowRaw<BF16> ahead;
        const uint32_t tid = threadIdx.x;
        fwht_quant_bigrow_body<LOG2K, BITS, BF16, BF6OUT, NORM, true>(
            row, tid, cur, row_lds, codes, s_dequant, code_sum, rp, code_offset,
            [&]() { if (next < T) bigrow_load<LOG2K, BF16>(x, next, tid, ahead); });
        if (next >= T) break;
        cur = ahead;
        row = next;
    }
}

template <int LOG2K, int BITS, bool BF16, bool BF6OUT, bool NORM, bool FEW>
int launch_bigrow_form(const void* x, int64_t T, int8_t* codes, float* s_dequant, int32_t* code_sum, RowParams rp,
                       int code_offset, hipStream_t stream);

template <int LOG2K, int BITS, bool BF16, bool BF6OUT = false>
int launch_bigrow(const void* x, int64_t T, int8_t* codes, float* s_dequant, int32_t* code_sum, RowParams rp,
                  int code_offset, hipStream_t stream) {
    if constexpr (BITS != 0) {
        const bool norm = rp.ln_gain != nullptr;
        if (rp.few_rows)
            return norm ? launch_bigrow_form<LOG2K, BITS, BF16, BF6OUT, true, true>(x, T, codes, s_dequant, code_sum, rp,
                                                                                    code_offset, stream)
                        : launch_bigrow_form<LOG2K, BITS, BF16, BF6OUT, false, true>(x, T, codes, s_dequant, code_sum, rp,
                                                                                     code_offset, stream);
        if (norm)
            return launch_bigrow_form<LOG2K, BITS, BF16, BF6OUT, true, false>(x, T, codes, s_dequant, code_sum, rp,
                                                                              code_offset, stream);
    }
    return launch_bigrow_form<LOG2K, BITS, BF16, BF6OUT, false, false>(x, T, codes, s_dequant, code_sum, rp, code_offset,
                                                                       stream);
}

template <int LOG2K, int BITS, bool BF16, bool BF6OUT, bool NORM, bool FEW>
int launch_bigrow_form(const void* x, int64_t T, int8_t* codes, float* s_dequant, int32_t* code_sum, RowParams rp,
                       int code_offset, hipStream_t stream) {
    constexpr int K = 1 << LOG2K;
    constexpr size_t lds = sizeof(float) * K;
    auto kern = fwht_quant_bigrow_kernel<LOG2K, BITS, BF16, BF6OUT, NORM, FEW>;
    static std::atomic<uint64_t> lds_allowed{0};   // per instantiation: devices already set up
    if (const int rc = allow_dynamic_lds(kern, lds, lds_allowed); rc != HBL_OK) return rc;
    int grid = (int)T;   // one row per workgroup ...
    if constexpr (BITS != 0 && !FEW) {   // ... or as many workgroups as the chip holds at once, walking the rows
        static std::atomic<int> resident[64];
        if (const int rc = resident_workgroups(kern, K / 64, lds, resident, &grid); rc != HBL_OK) return rc;
        if ((int64_t)grid > T) grid = (int)T;
    }
    launch_kernel("fwht_quant_bigrow_kernel", kern, dim3((unsigned)grid), dim3(K / 64), lds, stream, x, T, codes, s_dequant, code_sum, rp,
                       code_offset);
    return after_launch();
}

template <int LOG2K>
int dispatch_bigrow(const void* x, int x_dtype, int64_t T, int bits, RowParams rp, int8_t* codes, float* s_dequant,
                    int32_t* code_sum, int code_offset, hipStream_t stream) {
    const bool bf = x_dtype == HBL_BF16;
    if (code_offset == kCodesBf6)
        return bf ? launch_bigrow<LOG2K, 4, true, true>(x, T, codes, s_dequant, code_sum, rp, 8, stream)
                  : launch_bigrow<LOG2K, 4, false, true>(x, T, codes, s_dequant, code_sum, rp, 8, stream);
    if (bits == 8) return bf ? launch_bigrow<LOG2K, 8, true>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream)
                             : launch_bigrow<LOG2K, 8, false>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
    return bf ? launch_bigrow<LOG2K, 4, true>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream)
              : launch_bigrow<LOG2K, 4, false>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
}

// WITH_H = false: rows of 4096 and more, whose transform belongs to the all-register kernel above - only the
// plain quantiser is compiled from this body for them.
template <int LOG2K, int W, bool WITH_H = true>
int dispatch(const void* x, int x_dtype, int64_t T, int bits, RowParams rp, bool hadamard, int8_t* codes,
             float* s_dequant, int32_t* code_sum, int code_offset, hipStream_t stream) {
    const bool bf = x_dtype == HBL_BF16;
    if constexpr (!WITH_H) {
        if (hadamard) return HBL_E_SHAPE;
    } else if (hadamard) {
        if (bits == 8) return bf ? launch_one<LOG2K, W, 8, true, true>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream)
                                 : launch_one<LOG2K, W, 8, false, true>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
        return bf ? launch_one<LOG2K, W, 4, true, true>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream)
                  : launch_one<LOG2K, W, 4, false, true>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
    }
    if (bits == 8) return bf ? launch_one<LOG2K, W, 8, true, false>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream)
                             : launch_one<LOG2K, W, 8, false, false>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
    return bf ? launch_one<LOG2K, W, 4, true, false>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream)
              : launch_one<LOG2K, W, 4, false, false>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
}

// Rows of several projections in one grid (small-batch path): workgroup -> (problem, row), then the
// body the stand-alone launch would run for that problem.  A body that needs fewer than 256 threads
// runs on the first waves only; the other waves end at once, and a workgroup barrier waits only for
// waves that have not ended.
template <int BITS, bool BF16>
__global__ __launch_bounds__(256) void quant_grouped_kernel(const QuantGroupArgs a) {
    extern __shared__ __attribute__((aligned(16))) float row_lds[];
    const QuantProblem p = a.p[group_index_of(a.row_begin, a.n, (int)blockIdx.x)];
    const int64_t row = (int)blockIdx.x - p.row_begin;
    const int tid = threadIdx.x;
    if (!p.hadamard) {
        quant_generic_body<BITS, BF16>(row, tid, p.x, p.K, p.codes, p.s_dequant, p.code_sum, RowParams{a.eps, p.ln_gain, p.ln_eps, 1}, p.code_offset);
        return;
    }
#define HBL_SMALL_ROW(L2K)                                                                                    \
    case 1 << L2K:                                                                                            \
        if (tid < 64)                                                                                         \
            fwht_quant_body<L2K, 1, BITS, BF16, true>(row, tid, p.x, p.codes, p.s_dequant, p.code_sum, RowParams{a.eps, p.ln_gain, p.ln_eps, 1}, \
                                                      p.code_offset);                                         \
        return;
#define HBL_BIG_ROW(L2K)                                                                                      \
    case 1 << L2K:                                                                                            \
        if (tid < (1 << L2K) / 64) {                                                                          \
            BigRowRaw<BF16> raw;                                                                              \
            if constexpr (kRowThroughLds<L2K, BF16>)                                                          \
                bigrow_load_lds<L2K, BF16>(p.x, row, tid, reinterpret_cast<char*>(row_lds), raw);             \
            else                                                                                              \
                bigrow_load<L2K, BF16>(p.x, row, tid, raw);                                                       \
            const RowParams rp{a.eps, p.ln_gain, p.ln_eps, 1};                                                \
            if constexpr (BITS == 4) {                                                                        \
                if (p.code_offset == kCodesBf6) {                                                             \
                    fwht_quant_bigrow_body<L2K, 4, BF16, true, true>(row, tid, raw, row_lds, p.codes, p.s_dequant, p.code_sum, rp, 8); \
                    return;                                                                                   \
                }                                                                                             \
            }                                                                                                 \
            fwht_quant_bigrow_body<L2K, BITS, BF16, false, true>(row, tid, raw, row_lds, p.codes, p.s_dequant, p.code_sum, rp, \
                                                                 p.code_offset);                              \
        }                                                                                                     \
        return;
    switch (p.K) {
        HBL_SMALL_ROW(7)
        HBL_SMALL_ROW(8)
        HBL_SMALL_ROW(9)
        HBL_SMALL_ROW(10)
        HBL_SMALL_ROW(11)
        HBL_BIG_ROW(12)
        HBL_BIG_ROW(13)
        HBL_BIG_ROW(14)
        default: return;
    }
#undef HBL_SMALL_ROW
#undef HBL_BIG_ROW
}

}  // namespace

int launch_quant_grouped(const QuantGroupArgs& args, int bits, int x_dtype, hipStream_t stream) {
    int rows = 0;
    size_t lds = 0;
    for (int i = 0; i < args.n; ++i) {
        rows += args.p[i].T;
        if (args.p[i].hadamard && args.p[i].K >= 4096 && sizeof(float) * (size_t)args.p[i].K > lds)
            lds = sizeof(float) * (size_t)args.p[i].K;
    }
    if (rows == 0) return HBL_OK;
    const bool bf = x_dtype == HBL_BF16;
    auto launch = [&](auto kern) -> int {
        static std::atomic<uint64_t> lds_allowed{0};   // per instantiation: devices already set up
        if (const int rc = allow_dynamic_lds(kern, 64 * 1024, lds_allowed); rc != HBL_OK) return rc;
        launch_kernel("quant_grouped_kernel", kern, dim3((unsigned)rows), dim3(256), lds, stream, args);
        return after_launch();
    };
    if (bits == 8) return bf ? launch(quant_grouped_kernel<8, true>) : launch(quant_grouped_kernel<8, false>);
    return bf ? launch(quant_grouped_kernel<4, true>) : launch(quant_grouped_kernel<4, false>);
}

int launch_fwht_only(const void* x, int x_dtype, int64_t T, int64_t K, void* out, int out_dtype, hipStream_t stream) {
    if (T == 0) return HBL_OK;
    const bool bf = x_dtype == HBL_BF16;
    int8_t* o = static_cast<int8_t*>(out);
#define HBL_SMALL(L2K)                                                                                           \
    case 1 << L2K:                                                                                               \
        return bf ? launch_one<L2K, 1, 0, true, true>(x, T, o, nullptr, nullptr, RowParams{0.0f, nullptr, 0.0f, 0}, out_dtype, stream)        \
                  : launch_one<L2K, 1, 0, false, true>(x, T, o, nullptr, nullptr, RowParams{0.0f, nullptr, 0.0f, 0}, out_dtype, stream);
#define HBL_BIG(L2K)                                                                                             \
    case 1 << L2K:                                                                                               \
        return bf ? launch_bigrow<L2K, 0, true, false>(x, T, o, nullptr, nullptr, RowParams{0.0f, nullptr, 0.0f, 0}, out_dtype, stream)       \
                  : launch_bigrow<L2K, 0, false, false>(x, T, o, nullptr, nullptr, RowParams{0.0f, nullptr, 0.0f, 0}, out_dtype, stream);
    switch (K) {
        HBL_SMALL(7)
        HBL_SMALL(8)
        HBL_SMALL(9)
        HBL_SMALL(10)
        HBL_SMALL(11)
        HBL_BIG(12)
        HBL_BIG(13)
        HBL_BIG(14)
        default: return HBL_E_SHAPE;
    }
#undef HBL_SMALL
#undef HBL_BIG
}

// Large Hadamard rows: up to here one row per workgroup with the short-latency reductions, the row loop beyond.  Time of the
// former against the latter (both input types and widths, with the norm and without): up to 320 rows 0.79 to 1.01 at every K.
// K = 16384, of which two workgroups share a CU, 0.81 to 1.03 up to 512 rows, INT4 codes 1.01 to 1.11 from 576 on; K = 8192 0.85 to
// 1.01 up to 1024 rows, 1.00 to 1.07 at 1536; K = 4096 0.94 to 1.00 up to 1536.  One line for all, below the first loss.
constexpr int64_t kFewRows = 320;
// The one-row-per-workgroup kernels: the short-latency form of the reductions up to here, the six shuffle rounds beyond.  Against
// the latter: up to 4096 rows 0.85 to 1.01 (transformed rows of 2048 1.04 at 4096); at 5120 to 16384 rows still 0.82 to 1.00
// for most lengths, but 0.98 to 1.04 for transformed rows of 1024 and 2048.
constexpr int64_t kShortReductionRows = 4096;

int launch_fwht_quant(const void* x, int x_dtype, int64_t T, int64_t K, int bits, float eps, bool hadamard,
                      int8_t* codes, float* s_dequant, int32_t* code_sum, int code_offset, hipStream_t stream,
                      const float* ln_gain, float ln_eps) {
    if (T == 0) return HBL_OK;
    const RowParams rp = {eps, ln_gain, ln_eps, T <= kFewRows ? 1 : 0};
    if (code_offset == kCodesBf6 && (bits != 4 || K < 512)) return HBL_E_SHAPE;   // records need 8-element chunks
    const RowParams row_rp = {eps, ln_gain, ln_eps, T <= kShortReductionRows ? 1 : 0};
    if (!hadamard && !is_pow2(K)) return launch_generic(x, x_dtype, T, K, bits, row_rp, codes, s_dequant, code_sum, code_offset, stream);
    if (hadamard) {
        if (K == 4096) return dispatch_bigrow<12>(x, x_dtype, T, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
        if (K == 8192) return dispatch_bigrow<13>(x, x_dtype, T, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
        if (K == 16384) return dispatch_bigrow<14>(x, x_dtype, T, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
    }
    switch (K) {
        case 128:   return dispatch<7, 1>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 256:   return dispatch<8, 1>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 512:   return dispatch<9, 1>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 1024:  return dispatch<10, 1>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 2048:  return dispatch<11, 1>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 4096:  return dispatch<12, 2, false>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 8192:  return dispatch<13, 4, false>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 16384: return dispatch<14, 4, false>(x, x_dtype, T, bits, row_rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        default:    return HBL_E_SHAPE;
    }
}

}  // namespace hbl
