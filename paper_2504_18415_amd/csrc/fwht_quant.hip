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
// Index bits of a transformed row of K = CH*64*R < 2048 elements, by one wave (from 2048 on: large_rows.h), low to high:
//   [e: log2 CH in-thread][lane: 6][r: log2 R in-thread chunks]
// so that every global access is one contiguous CH-element piece per lane and
// the stage order e -> lane -> r is ascending.
#include "large_rows.h"

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
    launch_kernel("fwht_quant_kernel", (fwht_quant_kernel<LOG2K, W, BITS, BF16, HADAMARD>), dim3((unsigned)T), dim3(64 * W), 0, stream, x,
                  codes, s_dequant, code_sum, rp, code_offset);
    return after_launch();
}

template <int BITS, bool BF16, int MAXC, int NW>
__global__ __launch_bounds__(64 * NW) void quant_generic_kernel(const void* __restrict__ x, int K,
                                                               int8_t* __restrict__ codes,
                                                               float* __restrict__ s_dequant,
                                                               int32_t* __restrict__ code_sum, RowParams rp, int code_offset) {
    quant_generic_body<BITS, BF16, MAXC, kRecordBlockBytes, NW>(blockIdx.x, threadIdx.x, x, K, codes, s_dequant, code_sum, rp, code_offset);
}

template <int BITS, bool BF16, int NW>
void launch_generic_slots(const void* x, int64_t T, int64_t K, RowParams rp, int8_t* codes, float* s_dequant,
                          int32_t* code_sum, int code_offset, hipStream_t stream) {
    const dim3 grid((unsigned)T), block(64 * NW);
#define HBL_GENERIC(MAXC)                                                                                     \
    case MAXC:                                                                                                \
        if constexpr (512 * NW * (MAXC - 1) < 16384)                                                          \
            launch_kernel("quant_generic_kernel", (quant_generic_kernel<BITS, BF16, MAXC, NW>), grid, block, 0, stream, x, (int)K, \
                          codes, s_dequant, code_sum, rp, code_offset);                                       \
        break;
    switch ((K / 8 + 64 * NW - 1) / (64 * NW)) {   // 8-element chunks per thread
        HBL_GENERIC(1)
        HBL_GENERIC(2)
        HBL_GENERIC(3)
        HBL_GENERIC(4)
        HBL_GENERIC(5)
        HBL_GENERIC(6)
        HBL_GENERIC(7)
        HBL_GENERIC(8)
    }
#undef HBL_GENERIC
}
// Waves per row.  Few rows: many waves of few values finish a row sooner.  Many rows: the reductions, the divisions and the norm's
// square root are the same work for every wave, so fewer waves of more values do it less often.  Time against four waves (bf16,
// records; without / with the norm):
//   64 rows:    16 waves: 3072 0.98 / 1.03  5504 0.95 / 1.01  11008 0.91 / 0.96  16256 0.87 / 0.91;  1 wave: 384 0.98 / 0.94  640 1.07
//   512 rows:   16 waves: 11008 1.05 / 1.16  16256 0.99 / 1.06;  2 waves: 640 0.99  1920 1.10
//   1024 rows:  2 waves: 640 0.92 / 0.86  1152 0.94 / 0.89  1920 0.96 / 0.91  3072 0.95 / 0.88;  1 wave: 0.95 / 0.86  0.97 / 0.89  1.03 / 0.94  1.04 / 0.97
//   3001 rows:  1 wave: 640 0.84 / 0.75  1152 0.87 / 0.77  1920 0.92 / 0.81  3072 0.93 / 0.83 (2 waves 0.93 / 0.86);  2 waves: 5504 1.04 / 0.99
//   8192 rows:  1 wave: 384 0.60 / 0.50  1152 0.74 / 0.65  3072 0.95 / 0.81;  2 waves: 5504 1.00 / 0.95  8064 1.03 / 1.02
// Long rows and a finer look at the number of rows (2100 sizes; mean over 3 lengths each):
//   INT4, 2048 to 2500 rows: 1792 to 3072 1 wave 0.97 to 1.05 (2 waves 0.93 to 0.98), 3200 to 3584 0.98 to 1.09 (0.98 to 1.02),
//     3712 to 3968 1.03 to 1.14 (1.00 to 1.03);  2600 rows and more: 1792 to 3072 0.83 to 0.98, 3200 and above 0.98 to 1.10 (0.96 to 1.03)
//   INT4, 1024 to 2000 rows, 2 waves: up to 3072 0.92 to 1.04, 3200 and above 0.98 to 1.12
//   INT8 bf16 0.82 to 1.03 by 1 wave, from 2048 rows on, and by 2 waves before;  fp32, 3200 and above, 1.00 to 1.06
//   with the norm, from 2048 rows on, 1 wave: INT8 0.60 to 1.00;  INT4 up to 3584 0.65 to 0.99, above 0.92 to 1.05 (2 waves 0.90 to 0.98)
//   INT4, fp32 rows, whose chunks are two loads each, 1792 to 3072: 2 waves 0.92 to 1.00, 1.03 at 8192 rows
template <int BITS>
int generic_waves(int64_t T, int64_t K, bool bf16, bool norm) {
    if (K > 4096) return T <= 256 ? 16 : 4;
    if (K <= 512) return 1;
    const bool records = BITS == 4 && !norm;   // (few other instructions to share, and more of them per value)
    if (!norm && K > 3072 && (BITS == 4 || !bf16)) return 4;
    if (T >= (records && K > 1536 ? 2560 : 2048) && (bf16 || K <= (records ? 1536 : 2048))) return BITS == 4 && K > 3584 ? 2 : 1;
    return T >= 1024 ? 2 : 4;
}
template <int BITS, bool BF16>
void launch_generic_waves(const void* x, int64_t T, int64_t K, RowParams rp, int8_t* codes, float* s_dequant,
                          int32_t* code_sum, int code_offset, hipStream_t stream) {
    switch (generic_waves<BITS>(T, K, BF16, rp.ln_gain != nullptr)) {
        case 1: return launch_generic_slots<BITS, BF16, 1>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
        case 2: return launch_generic_slots<BITS, BF16, 2>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
        case 4: return launch_generic_slots<BITS, BF16, 4>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
        default: return launch_generic_slots<BITS, BF16, 16>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
    }
}

int launch_generic(const void* x, int x_dtype, int64_t T, int64_t K, int bits, RowParams rp, int8_t* codes,
                   float* s_dequant, int32_t* code_sum, int code_offset, hipStream_t stream) {
    const bool bf = x_dtype == HBL_BF16;
    if (bits == 8) {
        if (bf) launch_generic_waves<8, true>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
        else    launch_generic_waves<8, false>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
    } else {
        if (bf) launch_generic_waves<4, true>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
        else    launch_generic_waves<4, false>(x, T, K, rp, codes, s_dequant, code_sum, code_offset, stream);
    }
    return after_launch();
}


// ---------------------------------------------------------------------------------------------

// Rows of 8192 and 16384: 16 values per thread up to here, 32 beyond.  While every row has a CU to itself, twice the waves finish
// it sooner, although one or two more stages run between lanes (64 rows, INT4 records: 8192 4.3 -> 4.0 us, 16384 5.35 ->
// 5.25); from 257 rows on the fewer instructions count (257 rows of 16384 with the norm 9.4 -> 8.9; 512 of 8192 5.9 -> 5.8).
constexpr int64_t kSixteenValueRows = 256;

// Transformed rows of 2048 features and more (large_rows.h): one row per workgroup.
template <int LOG2K, int R, int BITS, bool BF16, bool BF6OUT, bool NORM>
__global__ __launch_bounds__((1 << LOG2K) >> R) void fwht_quant_bigrow_kernel(
    const void* __restrict__ x, int64_t first_row, int8_t* __restrict__ codes, float* __restrict__ s_dequant,
    int32_t* __restrict__ code_sum, RowParams rp, int code_offset) {
    extern __shared__ __attribute__((aligned(16))) float row_lds[];   // K floats
    const int64_t row = first_row + blockIdx.x;
    LargeRowRaw<R, BF16> raw;
    large_row_load<LOG2K, R, BF16>(x, row, threadIdx.x, raw);
    large_row_body<LOG2K, R, BITS, BF16, BF6OUT, NORM>(row, threadIdx.x, raw, row_lds, codes, s_dequant, code_sum, rp, code_offset);
}

template <int LOG2K, int R, int BITS, bool BF16, bool BF6OUT, bool NORM>
int launch_bigrow_form(const void* x, int64_t T, int8_t* codes, float* s_dequant, int32_t* code_sum, RowParams rp,
                       int code_offset, hipStream_t stream) {
    using L = LargeRow<LOG2K, R>;
    constexpr size_t lds = sizeof(float) * L::K;
    constexpr auto kern = fwht_quant_bigrow_kernel<LOG2K, R, BITS, BF16, BF6OUT, NORM>;
    if (const int rc = allow_dynamic_lds<kern, lds>(); rc != HBL_OK) return rc;
    constexpr int64_t most = (int64_t)1 << 22;   // rows per launch: a grid has fewer than 2^32 threads
    for (int64_t first = 0; first < T; first += most)
        launch_kernel("fwht_quant_bigrow_kernel", kern, dim3((unsigned)(T - first < most ? T - first : most)), dim3(L::NT), lds, stream,
                      x, first, codes, s_dequant, code_sum, rp, code_offset);
    return after_launch();
}

template <int LOG2K, int BITS, bool BF16, bool BF6OUT = false>
int launch_bigrow(const void* x, int64_t T, int8_t* codes, float* s_dequant, int32_t* code_sum, RowParams rp,
                  int code_offset, hipStream_t stream) {
    auto launch = [&](auto r_tag) {
        constexpr int R = decltype(r_tag)::value;
        if constexpr (BITS != 0) {
            if (rp.ln_gain != nullptr)
                return launch_bigrow_form<LOG2K, R, BITS, BF16, BF6OUT, true>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
        }
        return launch_bigrow_form<LOG2K, R, BITS, BF16, BF6OUT, false>(x, T, codes, s_dequant, code_sum, rp, code_offset, stream);
    };
    if constexpr (LOG2K >= 13) {
        if (T > kSixteenValueRows) return launch(std::integral_constant<int, 5>{});
    }
    return launch(std::integral_constant<int, 4>{});
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

// WITH_H = false: rows of 2048 and more, whose transform belongs to the kernel above - only the plain quantiser is compiled from this body for them.
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

// Rows of several projections in one grid (small-batch path): workgroup -> (problem, row), then the body the stand-alone launch
// would run for that problem.  A body that needs fewer threads than the workgroup has runs on the first waves only; the other
// waves end at once, and a workgroup barrier waits only for waves that have not ended.
// MANY: more than 256 rows of more than 4096 features, so that a CU gets more than one of them: fewer waves of more values, as in the
// stand-alone launches - 32 values a thread for transformed rows of 8192 and 16384, four waves (eight beyond 8192) for plain rows.
// Time against the other form, whole calls (bf16 and fp32, with the norm and without): 257 to 512 plain rows of 4224 to 8192
// 0.82 to 0.99, of 11008 to 16384 0.87 to 1.01; transformed rows of 16384 INT4 0.88 to 0.95, INT8 0.97 to 1.02, of 8192 0.96 to 1.03.
// Up to 256 such rows 0.95 to 1.03; with short rows beside them up to 1.07.
constexpr int64_t kManyGroupedRows = 256;

constexpr int grouped_row_threads(int64_t K, bool hadamard, bool many) {
    if (many) return K <= 8192 ? 256 : 512;
    return K <= 4096 ? 256 : (hadamard && K == 8192 ? 512 : 1024);
}

template <int BITS, bool BF16, bool MANY>
__global__ __launch_bounds__(MANY ? 512 : 1024, 4) void quant_grouped_kernel(const QuantGroupArgs a) {
    extern __shared__ __attribute__((aligned(16))) float row_lds[];
    const QuantProblem p = a.p[group_index_of(a.row_begin, a.n, (int)blockIdx.x)];
    const int64_t row = (int)blockIdx.x - p.row_begin;
    const int tid = threadIdx.x;
    const RowParams rp{a.eps, p.ln_gain, p.ln_eps, 1};
    if (!p.hadamard) {
#define HBL_PLAIN_ROW(MAXC, NW) \
    quant_generic_body<BITS, BF16, MAXC, kRecordBlockBytes, NW>(row, tid, p.x, p.K, p.codes, p.s_dequant, p.code_sum, rp, p.code_offset)
        if (p.K > 8192) {
            if constexpr (MANY) {
                if (p.K > 12288) HBL_PLAIN_ROW(4, 8);
                else HBL_PLAIN_ROW(3, 8);
            } else {
                HBL_PLAIN_ROW(2, 16);
            }
        } else if (p.K > 4096) {
            if constexpr (MANY) {
                if (tid < 256) {
                    if (p.K > 6144) HBL_PLAIN_ROW(4, 4);
                    else HBL_PLAIN_ROW(3, 4);
                }
            } else {
                HBL_PLAIN_ROW(1, 16);
            }
        } else if (tid < 256) {
            if (p.K > 2048) HBL_PLAIN_ROW(2, 4);
            else HBL_PLAIN_ROW(1, 4);
        }
#undef HBL_PLAIN_ROW
        return;
    }
#define HBL_SMALL_ROW(L2K)                                                                                    \
    case 1 << L2K:                                                                                            \
        if (tid < 64)                                                                                         \
            fwht_quant_body<L2K, 1, BITS, BF16, true>(row, tid, p.x, p.codes, p.s_dequant, p.code_sum, rp, p.code_offset); \
        return;
#define HBL_BIG_ROW(L2K, R)                                                                                   \
    case 1 << L2K:                                                                                            \
        if (tid < LargeRow<L2K, R>::NT) {                                                                     \
            LargeRowRaw<R, BF16> raw;                                                                         \
            large_row_load<L2K, R, BF16>(p.x, row, tid, raw);                                                 \
            if constexpr (BITS == 4) {                                                                        \
                if (p.code_offset == kCodesBf6) {                                                             \
                    large_row_body<L2K, R, 4, BF16, true, true>(row, tid, raw, row_lds, p.codes, p.s_dequant, p.code_sum, rp, 8); \
                    return;                                                                                   \
                }                                                                                             \
            }                                                                                                 \
            large_row_body<L2K, R, BITS, BF16, false, true>(row, tid, raw, row_lds, p.codes, p.s_dequant, p.code_sum, rp, p.code_offset); \
        }                                                                                                     \
        return;
    switch (p.K) {
        HBL_SMALL_ROW(7)
        HBL_SMALL_ROW(8)
        HBL_SMALL_ROW(9)
        HBL_SMALL_ROW(10)
        HBL_BIG_ROW(11, 4)
        HBL_BIG_ROW(12, 4)
        HBL_BIG_ROW(13, (MANY ? 5 : 4))
        HBL_BIG_ROW(14, (MANY ? 5 : 4))
        default: return;
    }
#undef HBL_SMALL_ROW
#undef HBL_BIG_ROW
}

template <int BITS, bool BF16, bool MANY>
int launch_grouped_kernel(const QuantGroupArgs& args, int rows, int threads, size_t lds, hipStream_t stream) {
    constexpr auto kern = quant_grouped_kernel<BITS, BF16, MANY>;
    if (const int rc = allow_dynamic_lds<kern, 64 * 1024>(); rc != HBL_OK) return rc;
    launch_kernel("quant_grouped_kernel", kern, dim3((unsigned)rows), dim3((unsigned)threads), lds, stream, args);
    return after_launch();
}
template <int BITS, bool BF16>
int launch_grouped_rows(const QuantGroupArgs& args, hipStream_t stream) {
    int rows = 0, large = 0, threads = 256;
    size_t lds = 0;
    for (int i = 0; i < args.n; ++i) {
        rows += args.p[i].T;
        if (args.p[i].K > 4096) large += args.p[i].T;
    }
    const bool many = large > kManyGroupedRows;
    for (int i = 0; i < args.n; ++i) {
        const QuantProblem& p = args.p[i];
        if (p.hadamard && p.K >= 2048 && sizeof(float) * (size_t)p.K > lds) lds = sizeof(float) * (size_t)p.K;
        const int need = grouped_row_threads(p.K, p.hadamard != 0, many);
        if (need > threads) threads = need;
    }
    if (rows == 0) return HBL_OK;
    return many ? launch_grouped_kernel<BITS, BF16, true>(args, rows, threads, lds, stream)
                : launch_grouped_kernel<BITS, BF16, false>(args, rows, threads, lds, stream);
}

}  // namespace

int launch_quant_grouped(const QuantGroupArgs& args, int bits, int x_dtype, hipStream_t stream) {
    const bool bf = x_dtype == HBL_BF16;
    if (bits == 8) return bf ? launch_grouped_rows<8, true>(args, stream) : launch_grouped_rows<8, false>(args, stream);
    return bf ? launch_grouped_rows<4, true>(args, stream) : launch_grouped_rows<4, false>(args, stream);
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
        return bf ? launch_bigrow<L2K, 0, true>(x, T, o, nullptr, nullptr, RowParams{0.0f, nullptr, 0.0f, 0}, out_dtype, stream)        \
                  : launch_bigrow<L2K, 0, false>(x, T, o, nullptr, nullptr, RowParams{0.0f, nullptr, 0.0f, 0}, out_dtype, stream);
    switch (K) {
        HBL_SMALL(7)
        HBL_SMALL(8)
        HBL_SMALL(9)
        HBL_SMALL(10)
        HBL_BIG(11)
        HBL_BIG(12)
        HBL_BIG(13)
        HBL_BIG(14)
        default: return HBL_E_SHAPE;
    }
#undef HBL_SMALL
#undef HBL_BIG
}

// The kernels of one wave or more per row (transformed rows of up to 1024, plain rows): the short-latency form of the reductions
// up to here, the six shuffle rounds beyond.  Against the latter: up to 4096 rows 0.85 to 1.01; at 5120 to 16384 rows still
// 0.82 to 1.00 for most lengths, but 0.98 to 1.04 for transformed rows of 1024.
constexpr int64_t kShortReductionRows = 4096;

constexpr int64_t kFewPlainRows = 512;

int launch_fwht_quant(const void* x, int x_dtype, int64_t T, int64_t K, int bits, float eps, bool hadamard,
                      int8_t* codes, float* s_dequant, int32_t* code_sum, int code_offset, hipStream_t stream,
                      const float* ln_gain, float ln_eps) {
    if (T == 0) return HBL_OK;
    if (code_offset == kCodesBf6 && (bits != 4 || K < 512)) return HBL_E_SHAPE;   // records need 8-element chunks
    const RowParams rp = {eps, ln_gain, ln_eps, T <= kShortReductionRows ? 1 : 0};
    // Plain rows that are a power of two have a kernel without any test for the row's end, one or two waves up to 4096; few rows
    // of 2048 and 4096 are faster by four waves (64 rows 0.87 and 0.91 of the time, 512 rows 0.91 and 0.87; 1024 rows 1.05; INT8
    // rows of 2048 1.02 to 1.07).
    if (!hadamard && (!is_pow2(K) || (T <= kFewPlainRows && (K == 4096 || (K == 2048 && bits == 4))))) return launch_generic(x, x_dtype, T, K, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
    if (hadamard) {
        if (K == 2048) return dispatch_bigrow<11>(x, x_dtype, T, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
        if (K == 4096) return dispatch_bigrow<12>(x, x_dtype, T, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
        if (K == 8192) return dispatch_bigrow<13>(x, x_dtype, T, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
        if (K == 16384) return dispatch_bigrow<14>(x, x_dtype, T, bits, rp, codes, s_dequant, code_sum, code_offset, stream);
    }
    switch (K) {
        case 128:   return dispatch<7, 1>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 256:   return dispatch<8, 1>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 512:   return dispatch<9, 1>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 1024:  return dispatch<10, 1>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 2048:  return dispatch<11, 1, false>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 4096:  return dispatch<12, 2, false>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 8192:  return dispatch<13, 4, false>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        case 16384: return dispatch<14, 4, false>(x, x_dtype, T, bits, rp, hadamard, codes, s_dequant, code_sum, code_offset, stream);
        default:    return HBL_E_SHAPE;
    }
}

}  // namespace hbl
