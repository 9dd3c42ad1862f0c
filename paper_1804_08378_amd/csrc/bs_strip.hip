// One 3 x 3 (row-major: or 2 x 2 / 2) pooling step, or a 3 x 3 / 1 / 1 step and a 3 x 3 maximum behind it, without LDS: strip_kernel.
//
// A lane owns one channel (two with 16-bit storage measured slower) of a strip of QO output columns and walks down a chunk of
// output rows with the rows of its windows in registers.  The columns a strip's windows share with the next strip are read
// and computed by both lanes (they come from the caches): no lane waits for another one, any width, any channel count.
//   Channels-last tensors: the lanes of a wave are neighbouring channels (then neighbouring strips), so every access is
//   contiguous.  Work-groups are numbered so that an XCD gets one contiguous part of the tensor (xcd_contiguous).
//   Row-major tensors, rows that are no whole vectors: the lanes are neighbouring strips of a row; a lane reads its columns as
//   vectors at whatever address they begin (16 bytes of own columns per lane and row, so that a wave's load has no gaps).
//
// Arithmetic and order of the other kernels: every layer rounds to the storage type, averages add row-major from
// +0, the first maximum wins.  Where no index is asked for, an average in front of a maximum is rounded behind it (rounding
// never decreases, so it commutes with the maximum).
//
// What bounds it on MI355X (back to back; single launches take 3 to 7 us more): halo_stress float32 53 us = 4.9 TB/s of input and output
// (memory, with vector instructions close behind), bfloat16 38 us = 3.4 TB/s (vector instructions, 27 per cell: conversions and the
// nine additions per average and its halo); one step with indices 4.9 TB/s (ResNet stem bfloat16, 37 us).  Row-major 32 x 64 x 147 x 147
// / 2 binary16: 28 us = 3.9 TB/s (one wave's rows at a time in flight).  The kernels it takes over from: bs_plan.cpp has both sides.
#include <algorithm>

#include "bs_nhwc_device.h"
#include "bs_strip_device.h"

#include "bs_internal.h"

namespace bs {
namespace {

// Element-wise list on N pixels of V channels (pixel-major).  CODE >= 0: kinds compiled in, the parameters read once per lane by
// load(); -1: kinds and parameters read at every use (holding the first four operations' parameters measured 2 to 20 % slower here).
template <int DT, int V, int CODE>
struct FwdList {
    static constexpr int L = CODE > 0 ? ew_code_len(CODE) : 0;
    HeldParams<V> held[L ? L : 1];

    BS_DEV void load(const StripK &k, const EwOp *ew, int32_t n, int32_t c)
    {
#pragma unroll
        for (int q = 0; q < L; ++q)
            if (CODE == BN_RELU && q == 0 && n == 1) held[q].identity();  // ReLU alone
            else held[q].load(k.params, ew_code_kind(CODE, q), ew[q].arg, c, k.C);
    }
    template <int N, typename P>
    BS_DEV static void one(int32_t kind, const P &p, float (&x)[N])
    {
        if (kind == OP_BN) {
            float a[V], b[V];
            p.bn(a, b);
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = __builtin_fmaf(x[i], a[i % V], b[i % V]);
            round_store_all<DT, N>(x);
        } else if (kind == OP_RELU) {
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = __builtin_fmaxf(x[i], 0.0f);  // NaN, -0 -> +0
        } else if (kind == OP_LEAKY) {
            const float slope = p.first();
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = round_store<DT>(x[i] > 0.0f ? x[i] : x[i] * slope);
        } else {  // OP_CLAMP
            const float lo = p.first(), hi = p.second();
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = round_store<DT>(__builtin_fminf(__builtin_fmaxf(x[i], lo), hi));
        }
    }
    template <int N>
    BS_DEV void apply(const StripK &k, const EwOp *ew, int32_t n, int32_t c, float (&x)[N]) const
    {
        if constexpr (CODE >= 0) {
#pragma unroll
            for (int q = 0; q < L; ++q) one<N>(ew_code_kind(CODE, q), held[q], x);
        } else {
#pragma clang loop unroll(disable)
            for (int32_t q = 0; q < n; ++q) one<N>(ew[q].kind, ReadParams<V>{k.params, ew[q].arg, c, k.C}, x);
        }
    }
};

// CL: channels-last tensors -- the lanes of a wave are channels, a column is one pixel further on.  Otherwise row-major -- the lanes
// are neighbouring strips of a row, a lane's columns are consecutive elements, read as vectors that need no alignment.
// K1: the first pooling (OP_MAXPOOL, OP_AVGSUM; 0: one pooling step only), 3 x 3, stride 1, padding 1; K2: the second (only) one,
// K x K, stride S, padding P.  IDX: the second one's picks are written.  PRE, POST: codes of the lists, or -1 (then the list
// between the poolings is read at run time, too, and averages may have any divisor; otherwise there is none and they divide by nine).
template <int DT, bool CL, int QO, int K1, int K2, int K, int S, int P, bool IDX, int PRE, int POST, typename OFF>
__global__ __launch_bounds__(256) void strip_kernel(const StripK k)
{
    static_assert((K == 3 && (S == 1 || S == 2) && (P == 0 || P == 1) && (K1 == 0 || P == 1)) || (K == 2 && S == 2 && P == 0 && K1 == 0),
                  "compiled windows");
    constexpr int V = 1;                              // channels per lane
    constexpr int CA = (QO - 1) * S + K;              // columns of the plane the second pooling reads
    constexpr int CX = K1 ? CA + 2 : CA;              // columns of the input
    constexpr int ES = elem_bytes<DT>(), KEEP = K - S, KEPT = KEEP ? KEEP : 1;
    constexpr bool MAX2 = K2 == OP_MAXPOOL, GENERAL = PRE < 0;
    constexpr bool DEFER = K1 == OP_AVGSUM && MAX2 && !IDX && !GENERAL;  // the average is rounded behind the maximum
    // Non-temporal stores (a wave writes whole cache lines of channels; float32 indices plainly) where the output is hardly ever the next launch's input:
    // training, and the average-maximum pair.  Measured, us, plain / non-temporal: ResNet stem with indices 64 x 64 x 112 x 112 bfloat16 39.5 / 31.9, float32 62.2 / 60.9;
    // 32 x 192 x 71 x 71 / 2 with indices binary16 23.7 / 18.8, float32 36.9 / 31.6; halo_stress float32 56.3 / 52.7, bfloat16 40.3 / 38.6, with indices 50.9 / 44.8, 33 x 40
    // x 17 x 55 (0.7 MB) 6.8 / 7.1.  Two maxima between two launches, 32 x 64 x 56 x 56 float32, four blocks: 29.7 / 31.6 (plain).  float32 indices, forward and backward:
    // 146.8 / 149.6 (plain).  A flag read in the loop instead: stem 37.4.
    constexpr bool STREAMED = CL && (IDX || K1 == OP_AVGSUM);
    constexpr float PAD1 = K1 == OP_MAXPOOL ? -INFINITY : 0.0f, PAD2 = MAX2 ? -INFINITY : 0.0f;
    uint32_t i0 = xcd_contiguous(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
    const bool live = i0 < k.total;
    i0 = live ? i0 : 0u;
    // channels-last: (image, chunk, strip, channel), row-major: (image, channel, chunk, strip), the last one fastest
    uint32_t n, plane = 0;
    int32_t c0, ow0, chunk;
    if constexpr (CL) {
        const uint32_t u0 = fdiv(i0, k.div_c);
        c0 = (int32_t)(i0 - u0 * k.div_c.d);
        const uint32_t v0 = fdiv(u0, k.div_strips);
        ow0 = (int32_t)(u0 - v0 * k.div_strips.d) * QO;
        n = fdiv(v0, k.div_chunks);
        chunk = (int32_t)(v0 - n * k.div_chunks.d);
    } else {
        const uint32_t u0 = fdiv(i0, k.div_strips);
        ow0 = (int32_t)(i0 - u0 * k.div_strips.d) * QO;
        plane = fdiv(u0, k.div_chunks);
        chunk = (int32_t)(u0 - plane * k.div_chunks.d);
        n = fdiv(plane, k.div_c);
        c0 = (int32_t)(plane - n * k.div_c.d);
    }

    const int32_t a0 = ow0 * S - P, x0 = K1 ? a0 - 1 : a0;
    const OFF pa = CL ? (OFF)(k.C + k.in_xp) * ES : (OFF)ES, po = CL ? (OFF)(k.C + k.out_xp) * ES : (OFF)ES, arow = (OFF)k.W * pa;
    OFF col[CX];
#pragma unroll
    for (int j = 0; j < CX; ++j) col[j] = (OFF)min(max(x0 + j, 0), k.W - 1) * pa;  // outside the plane: a safe column, replaced below
    const bool inside = x0 >= 0 && x0 + CX <= k.W, whole = ow0 + QO <= k.Wo, lead = P == 1 && ow0 == 0;

    FwdList<DT, V, PRE> pre;
    FwdList<DT, V, POST> post;
    pre.load(k, k.pre, k.n_pre, c0);
    post.load(k, k.post, k.n_post, c0);
    const FwdList<DT, V, -1> mid{};

    const int32_t oh0 = chunk * k.rc, oh_end = min(oh0 + k.rc, k.Ho);
    // input rows are requested in order: `next`, at byte offset `at` (clamped to the plane)
    int32_t next = K1 ? oh0 * S - P - 1 : oh0 * S - P;
    OFF at = (CL ? (OFF)(n * (uint32_t)(k.H * k.W)) * pa + (OFF)c0 * ES : ((OFF)(plane * (uint32_t)(k.H * k.W)) + (OFF)n * k.in_xp) * ES) +
             (OFF)min(max(next, 0), k.H - 1) * arow;
    // row-major: a run of CX elements that begins here at the latest lies inside the tensor (columns beside the plane are other
    // rows' elements then, replaced below)
    const bool run_fits = k.in_bytes >= (uint64_t)CX * ES;
    const OFF last_run = run_fits ? (OFF)(k.in_bytes - (uint64_t)CX * ES) : (OFF)0;
    int32_t row1 = oh0 * S - P;  // the next row of the plane the second pooling reads
    float y[2][CX * V];          // K1: the two newest input rows after the leading list

    // the next N input rows -> after the leading list, padding in place
    auto input_rows = [&](auto n_tag, float (&r)[decltype(n_tag)::value][CX * V]) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value;
        float x[N * CX * V];
        uint32_t w[N][CL ? CX : run_words<DT, CX>()];  // requested for all rows before the first is used
        bool ok[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            ok[j] = next >= 0 && next < k.H;
            if constexpr (CL) {
#pragma unroll
                for (int c = 0; c < CX; ++c) {
                    uint32_t e[1];
                    load_run<DT, 1>(static_cast<const char *>(k.in) + (OFF)(at + col[c]), e);
                    w[j][c] = e[0];
                }
            } else {
                const OFF from = at + (OFF)x0 * (OFF)ES;
                if (run_fits && from <= last_run) {
                    load_run<DT, CX>(static_cast<const char *>(k.in) + from, w[j]);
                } else {  // at the tensor's ends: one by one
#pragma unroll
                    for (int c = 0; c < CX; ++c) {
                        uint32_t e[1];
                        load_run<DT, 1>(static_cast<const char *>(k.in) + (OFF)(at + col[c]), e);
                        if constexpr (DT == DT_F32) w[j][c] = e[0];
                        else w[j][c / 2] = c % 2 ? w[j][c / 2] | e[0] << 16 : e[0];
                    }
                }
            }
            at += next >= 0 && next < k.H - 1 ? arow : (OFF)0;
            ++next;
        }
#pragma unroll
        for (int j = 0; j < N; ++j)
#pragma unroll
            for (int c = 0; c < CX; ++c) x[j * CX + c] = CL ? run_element<DT>(&w[j][c], 0) : run_element<DT>(w[j], c);
        pre.template apply<N * CX * V>(k, k.pre, k.n_pre, c0, x);
#pragma unroll
        for (int j = 0; j < N; ++j) {
#pragma unroll
            for (int i = 0; i < CX * V; ++i) r[j][i] = x[j * CX * V + i];
            if (!(inside && ok[j])) {
#pragma unroll
                for (int i = 0; i < CX * V; ++i) {
                    const int32_t c = x0 + i / V;
                    r[j][i] = ok[j] && c >= 0 && c < k.W ? r[j][i] : K1 ? PAD1 : PAD2;
                }
            }
        }
    };
    // sum of a window, row-major from +0; r[d]: its rows
    auto window_sum = [&](auto n_tag, const float *const (&r)[decltype(n_tag)::value]) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value;
        // a list that ends in a ReLU has no -0, so the sum may start with the first cell instead of +0
        float t = ends_in_relu(PRE) ? r[0][0] : 0.0f + r[0][0];
#pragma unroll
        for (int d = 0; d < N; ++d)
#pragma unroll
            for (int e = 0; e < N; ++e)
                if (d + e > 0) t = t + r[d][e];
        return t;
    };
    auto divisor = [&](const PoolK &p, int32_t oh, int32_t ow) __attribute__((always_inline)) {
        if constexpr (!GENERAL) return p.inv_kk;
        const int32_t h = oh * p.sh - p.ph, w = ow * p.sw - p.pw;
        return avg_inv(p, p.kh, p.kw, k.H, k.W, h, w, max(h, 0), min(h + p.kh, k.H), max(w, 0), min(w + p.kw, k.W));
    };
    // row `row1` of the plane between the poolings from three rows of the input
    auto first_pool = [&](const float (&ra)[CX * V], const float (&rb)[CX * V], const float (&rc)[CX * V], float (&a)[CA * V])
                          __attribute__((always_inline)) {
        if constexpr (K1 == OP_MAXPOOL) {
            float m[CX * V];
#pragma unroll
            for (int i = 0; i < CX * V; ++i) m[i] = __builtin_fmaxf(__builtin_fmaxf(ra[i], rb[i]), rc[i]);
#pragma unroll
            for (int i = 0; i < CA * V; ++i) a[i] = __builtin_fmaxf(__builtin_fmaxf(m[i], m[i + V]), m[i + 2 * V]);
        } else {
#pragma unroll
            for (int i = 0; i < CA * V; ++i) {
                const float *const r[3] = {ra + i, rb + i, rc + i};
                a[i] = window_sum(std::integral_constant<int, 3>{}, r) * divisor(k.pool1, row1, a0 + i / V);
            }
            if constexpr (!DEFER) round_store_all<DT, CA * V>(a);
        }
        if constexpr (GENERAL) mid.template apply<CA * V>(k, k.mid, k.n_mid, c0, a);
        const bool ok = row1 >= 0 && row1 < k.H;
        if (!(inside && ok)) {
#pragma unroll
            for (int i = 0; i < CA * V; ++i) {
                const int32_t c = a0 + i / V;
                a[i] = ok && c >= 0 && c < k.W ? a[i] : PAD2;
            }
        }
    };
    // the next N rows of the plane the second pooling reads
    auto rows = [&](auto n_tag, float (&a)[decltype(n_tag)::value][CA * V]) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value;
        if constexpr (K1 == 0) {
            input_rows(n_tag, a);
            row1 += N;
        } else {
            float r[N][CX * V];
            input_rows(n_tag, r);
            each_of(std::make_integer_sequence<int, N>{}, [&](auto j_tag) __attribute__((always_inline)) {
                constexpr int j = decltype(j_tag)::value;
                first_pool(y[0], y[1], r[j], a[j]);
                ++row1;
#pragma unroll
                for (int i = 0; i < CX * V; ++i) {
                    y[0][i] = y[1][i];
                    y[1][i] = r[j][i];
                }
            });
        }
    };
    // what is kept of the KEEP rows that the next output row reads again: maximum -- the windows' row maxima (and their cells);
    // average -- the rows
    float m[KEPT][QO * V], w[KEPT][CA * V];
    int32_t cell[KEPT][QO * V];
    auto row_max = [&](const float (&a)[CA * V], int32_t row, float (&mx)[QO * V], int32_t (&ix)[QO * V]) __attribute__((always_inline)) {
        if constexpr (IDX) {
            if constexpr (K == 3) {
                row_maxima<V, S, QO, CA, 0, P == 1 ? 0 : -1, ends_in_relu(PRE)>(a, lead, mx, ix);
            } else {
#pragma unroll
                for (int i = 0; i < QO; ++i) {
                    mx[i] = ends_in_relu(PRE) ? a[i * S] : __builtin_fmaxf(a[i * S], -INFINITY);
                    ix[i] = 0;
                    take_if_more(a[i * S + 1], 1, mx[i], ix[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < QO * V; ++i) ix[i] += row * k.W + a0 + (i / V) * S;
        } else {
#pragma unroll
            for (int i = 0; i < QO * V; ++i) {
                const float *p = a + (i / V) * S * V + i % V;
                mx[i] = __builtin_fmaxf(p[0], p[V]);
                if constexpr (K == 3) mx[i] = __builtin_fmaxf(mx[i], p[2 * V]);
            }
        }
    };
    if constexpr (KEEP > 0) {
        if constexpr (K1 != 0) input_rows(std::integral_constant<int, 2>{}, y);
        float a[KEEP][CA * V];
        const int32_t first = row1;
        rows(std::integral_constant<int, KEEP>{}, a);
#pragma unroll
        for (int j = 0; j < KEEP; ++j) {
            if constexpr (MAX2) row_max(a[j], first + j, m[j], cell[j]);
            else
#pragma unroll
                for (int i = 0; i < CA * V; ++i) w[j][i] = a[j][i];
        }
    }

    const uint32_t opix0 = CL ? (n * (uint32_t)k.Ho + (uint32_t)oh0) * (uint32_t)k.Wo + (uint32_t)ow0
                              : (plane * (uint32_t)k.Ho + (uint32_t)oh0) * (uint32_t)k.Wo + (uint32_t)ow0;
    int32_t oh = oh0;
    OFF oat = CL ? (OFF)opix0 * po + (OFF)c0 * ES : ((OFF)opix0 + (OFF)n * k.out_xp) * ES;
    uint32_t iat = CL ? opix0 * (uint32_t)k.C + (uint32_t)c0 : opix0;  // IDX: the first output's place among the indices
    auto step = [&]() __attribute__((always_inline)) {
        float a[S][CA * V], o[QO * V];
        const int32_t first = row1;  // the first new row
        rows(std::integral_constant<int, S>{}, a);
        int32_t pick[QO * V];
        if constexpr (MAX2) {
            float mn[S][QO * V];
            int32_t cn[S][QO * V];
#pragma unroll
            for (int j = 0; j < S; ++j) row_max(a[j], first + j, mn[j], cn[j]);
            // the window's rows: the KEEP kept ones, then the new ones
#pragma unroll
            for (int i = 0; i < QO * V; ++i) {
                o[i] = KEEP ? m[0][i] : mn[0][i];
                if constexpr (IDX) {
                    // the first window row lies above the plane (padding): never picked
                    const int32_t first_cell = KEEP ? cell[0][i] : cn[0][i], second_cell = KEEP == 2 ? cell[KEPT - 1][i] : cn[KEEP ? 0 : S - 1][i];
                    pick[i] = P == 1 && oh == 0 ? second_cell : first_cell;
                }
#pragma unroll
                for (int d = 1; d < K; ++d) {
                    const float v = d < KEEP ? m[d < KEEP ? d : 0][i] : mn[d < KEEP ? 0 : d - KEEP][i];
                    if constexpr (IDX) take_if_more(v, d < KEEP ? cell[d < KEEP ? d : 0][i] : cn[d < KEEP ? 0 : d - KEEP][i], o[i], pick[i]);
                    else o[i] = __builtin_fmaxf(o[i], v);
                }
            }
            if constexpr (DEFER) round_store_all<DT, QO * V>(o);
#pragma unroll
            for (int j = 0; j < KEEP; ++j)
#pragma unroll
                for (int i = 0; i < QO * V; ++i) {
                    m[j][i] = KEEP == 2 && j == 0 ? m[KEPT - 1][i] : mn[S - 1][i];
                    if constexpr (IDX) cell[j][i] = KEEP == 2 && j == 0 ? cell[KEPT - 1][i] : cn[S - 1][i];
                }
        } else {
#pragma unroll
            for (int i = 0; i < QO * V; ++i) {
                const int j = (i / V) * S * V + i % V;
                const float *r[K];
#pragma unroll
                for (int d = 0; d < K; ++d) r[d] = (d < KEEP ? w[d < KEEP ? d : 0] : a[d < KEEP ? 0 : d - KEEP]) + j;
                o[i] = window_sum(std::integral_constant<int, K>{}, r) * divisor(k.pool2, oh, ow0 + i / V);
            }
            round_store_all<DT, QO * V>(o);
#pragma unroll
            for (int j = 0; j < KEEP; ++j)
#pragma unroll
                for (int i = 0; i < CA * V; ++i) w[j][i] = KEEP == 2 && j == 0 ? w[KEPT - 1][i] : a[S - 1][i];
        }
        post.template apply<QO * V>(k, k.post, k.n_post, c0, o);
        if (live) {
            char *out = static_cast<char *>(k.out) + oat;
            if (!CL && whole) {
                store_run<DT, QO>(out, o);
                if constexpr (IDX) __builtin_memcpy(k.idx + iat, pick, 4 * QO);
            } else if constexpr (STREAMED) {
#pragma unroll
                for (int j = 0; j < QO; ++j)
                    if (whole || ow0 + j < k.Wo) {
                        store_elems<DT, 1>(NonTemporal{}, out + (OFF)j * po, o + j);
                        if constexpr (IDX) {
                            int32_t *at = k.idx + (iat + (uint32_t)j * (uint32_t)k.C);
                            if constexpr (DT == DT_F32) *at = pick[j];
                            else __builtin_nontemporal_store(pick[j], at);
                        }
                    }
            } else {
#pragma unroll
                for (int j = 0; j < QO; ++j)
                    if (whole || ow0 + j < k.Wo) {
                        const float t[1] = {o[j]};
                        store_elems<DT, 1>(out + (OFF)j * po, 0, t);
                        if constexpr (IDX) k.idx[iat + (uint32_t)j * (CL ? (uint32_t)k.C : 1u)] = pick[j];
                    }
            }
        }
        oat += (OFF)k.Wo * po;
        iat += (uint32_t)k.Wo * (CL ? (uint32_t)k.C : 1u);
        ++oh;
    };
    // twice per iteration: the rows that stay and the new ones change registers without moves.  Chunks are not empty.
    for (;;) {
        step();
        if (oh >= oh_end) break;
        step();
        if (oh >= oh_end) break;
    }
}

constexpr int BN_RELU_TWICE = BN_RELU + BN_RELU * K_EW_BASE * K_EW_BASE;

// The lists of the common networks are compiled in; in front of a maximum without indices they have moved behind it.
constexpr bool lists_lead(int K1, int K2, bool idx) { return K1 == OP_AVGSUM || (K1 == 0 && (K2 == OP_AVGSUM || idx)); }
constexpr int common_pre(int K1, int K2, bool idx) { return lists_lead(K1, K2, idx) ? BN_RELU : 0; }
constexpr int common_post(int K1, int K2, bool idx) { return K1 == OP_AVGSUM || !lists_lead(K1, K2, idx) ? BN_RELU : 0; }

enum class Lists { RUN_TIME, COMMON, TWICE, BARE };

Lists lists_of(const StripK &k, bool idx)
{
    const int K1 = k.pool1.kind, K2 = k.pool2.kind;
    if (k.n_mid > 0 || (K1 == OP_AVGSUM && k.pool1.count_include_pad != 1) || (K2 == OP_AVGSUM && k.pool2.count_include_pad != 1))
        return Lists::RUN_TIME;
    const int32_t pre = strip_list_code(k.pre, k.n_pre), post = strip_list_code(k.post, k.n_post);
    if (pre == common_pre(K1, K2, idx) && post == common_post(K1, K2, idx)) return Lists::COMMON;
    if (k.nhwc && K1 == OP_MAXPOOL && !idx && pre == 0 && post == BN_RELU_TWICE) return Lists::TWICE;  // two blocks of the stacked pooling
    if (K1 != OP_MAXPOOL && k.pool2.kh == 3 && pre == 0 && post == 0) return Lists::BARE;  // the pooling branch and the reductions of Inception modules
    return Lists::RUN_TIME;
}

template <int DT, bool CL, int K1, int K2, int K, int S, int P, bool IDX>
void launch_lists(const StripK &k, bool wide, dim3 g, hipStream_t st)
{
    constexpr int QO = strip_columns(CL, DT, S), PRE = common_pre(K1, K2, IDX), POST = common_post(K1, K2, IDX);
    const Lists lists = wide ? Lists::RUN_TIME : lists_of(k, IDX);
    if (lists == Lists::COMMON) {
        strip_kernel<DT, CL, QO, K1, K2, K, S, P, IDX, PRE, POST, uint32_t><<<g, 256, 0, st>>>(k);
        return;
    }
    if constexpr (CL && K1 == OP_MAXPOOL && !IDX)
        if (lists == Lists::TWICE) {
            strip_kernel<DT, CL, QO, K1, K2, K, S, P, IDX, 0, BN_RELU_TWICE, uint32_t><<<g, 256, 0, st>>>(k);
            return;
        }
    if constexpr (K == 3 && K1 != OP_MAXPOOL)
        if (lists == Lists::BARE) {
            strip_kernel<DT, CL, QO, K1, K2, K, S, P, IDX, 0, 0, uint32_t><<<g, 256, 0, st>>>(k);
            return;
        }
    if constexpr (!(K1 == OP_AVGSUM && S == 2))  // the planner takes no such pair (strips_lists_compiled): one instance for any offsets
        if (!wide) {
            strip_kernel<DT, CL, QO, K1, K2, K, S, P, IDX, -1, -1, uint32_t><<<g, 256, 0, st>>>(k);
            return;
        }
    strip_kernel<DT, CL, QO, K1, K2, K, S, P, IDX, -1, -1, uint64_t><<<g, 256, 0, st>>>(k);
}

template <int DT, bool CL, int K1, int K2>
void launch_windows(const StripK &k, bool wide, dim3 g, hipStream_t st)
{
    const PoolK &p = k.pool2;
    constexpr bool MAX2 = K2 == OP_MAXPOOL;
#define BS_STRIP(K, S, P)                                                                      \
    do {                                                                                       \
        if (MAX2 && k.idx) launch_lists<DT, CL, K1, K2, K, S, P, MAX2>(k, wide, g, st);        \
        else launch_lists<DT, CL, K1, K2, K, S, P, false>(k, wide, g, st);                     \
    } while (0)
    if constexpr (K1 == 0 && !CL) {
        if (p.kh == 2) {
            BS_STRIP(2, 2, 0);
            return;
        }
    }
    if (p.sh == 2 && p.ph == 1) BS_STRIP(3, 2, 1);
    else if (p.sh == 1 && p.ph == 1) BS_STRIP(3, 1, 1);
    else if constexpr (K1 == 0) {
        if (p.sh == 2) BS_STRIP(3, 2, 0);
        else BS_STRIP(3, 1, 0);
    }
#undef BS_STRIP
}

template <int DT, bool CL>
void launch_kinds(const StripK &k, bool wide, dim3 g, hipStream_t st)
{
    if (k.pool1.kind == OP_AVGSUM) launch_windows<DT, CL, OP_AVGSUM, OP_MAXPOOL>(k, wide, g, st);
    else if (k.pool1.kind == OP_MAXPOOL) launch_windows<DT, CL, OP_MAXPOOL, OP_MAXPOOL>(k, wide, g, st);
    else if (k.pool2.kind == OP_MAXPOOL) launch_windows<DT, CL, 0, OP_MAXPOOL>(k, wide, g, st);
    else launch_windows<DT, CL, 0, OP_AVGSUM>(k, wide, g, st);
}

}  // namespace

bool strips_supported(const StripK &k)
{
    const PoolK &p = k.pool1, &q = k.pool2;
    auto is3 = [](const PoolK &w) {
        return (w.kind == OP_MAXPOOL || w.kind == OP_AVGSUM) && w.kh == 3 && w.kw == 3 && w.sh == w.sw && w.ph == w.pw && (w.sh == 1 || w.sh == 2) &&
               w.ph >= 0 && w.ph <= 1;
    };
    const bool two = !k.nhwc && p.kind == 0 && (q.kind == OP_MAXPOOL || q.kind == OP_AVGSUM) && q.kh == 2 && q.kw == 2 && q.sh == 2 && q.sw == 2 &&
                     q.ph == 0 && q.pw == 0;
    if (!is3(q) && !two) return false;
    if (p.kind != 0 && (!is3(p) || p.sh != 1 || p.ph != 1 || q.ph != 1 || q.kind != OP_MAXPOOL)) return false;
    const EwOp *lists[3] = {k.pre, k.mid, k.post};
    const int32_t counts[3] = {k.n_pre, k.n_mid, k.n_post};
    for (int l = 0; l < 3; ++l)
        for (int32_t j = 0; j < counts[l]; ++j)
            if (lists[l][j].kind == OP_ADD) return false;  // strips do not read residual operands
    return true;
}

bool strips_lists_compiled(const StripK &k) { return lists_of(k, k.pool2.kind == OP_MAXPOOL && k.pool2.idx_slot >= 0) != Lists::RUN_TIME; }

bs_status launch_strips(const StripK &arg, int32_t dtype, int64_t grid, void *stream)
{
    StripK k = arg;
    const int32_t qo = strip_columns(k.nhwc != 0, dtype, k.pool2.sh);
    // what the kernel assumes: the windows and lists above, strips and chunks that cover the output, no empty chunk, the divisors
    // of the lane numbering
    if (!strips_supported(k) || grid < 1 || grid > 0x7fffffffll || (uint64_t)grid * 256 < k.total || (int64_t)k.div_c.d != k.C ||
        k.strips != (k.Wo + qo - 1) / qo || (int64_t)k.div_strips.d != k.strips || (int64_t)k.div_chunks.d != k.chunks ||
        k.rc < 1 || (int64_t)k.chunks * k.rc < k.Ho || (int64_t)(k.chunks - 1) * k.rc >= k.Ho ||
        k.total % ((uint64_t)k.strips * k.chunks * k.C) != 0)
        return BS_ERR_UNSUPPORTED;
    // elements from the first to the last one of each tensor; 32-bit byte offsets where both end below 4 GiB
    const uint64_t images = k.total / ((uint64_t)k.strips * k.chunks * k.C), es = dtype == BS_F32 ? 4 : 2;
    const uint64_t in_px = (uint64_t)k.H * k.W, out_px = (uint64_t)k.Ho * k.Wo;
    const uint64_t in_n = k.nhwc ? images * in_px * (k.C + (uint64_t)k.in_xp) : images * in_px * k.C + (images - 1) * k.in_xp;
    const uint64_t out_n = k.nhwc ? images * out_px * (k.C + (uint64_t)k.out_xp) : images * out_px * k.C + (images - 1) * k.out_xp;
    k.in_bytes = in_n * es;
    const bool wide = std::max(in_n, out_n) * es > 0xffffffffull;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 g((uint32_t)grid);
#define BS_STRIPS(DT)                                                \
    do {                                                             \
        if (k.nhwc) launch_kinds<DT, true>(k, wide, g, st);          \
        else launch_kinds<DT, false>(k, wide, g, st);                \
    } while (0)
    if (dtype == BS_F32) BS_STRIPS(DT_F32);
    else if (dtype == BS_BF16) BS_STRIPS(DT_BF16);
    else if (dtype == BS_F16) BS_STRIPS(DT_F16);
    else return BS_ERR_UNSUPPORTED;
#undef BS_STRIPS
    return BS_OK;
}

}  // namespace bs
