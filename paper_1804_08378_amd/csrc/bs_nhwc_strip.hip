// Channels-last tensors, one 3 x 3 pooling step, or a 3 x 3 / 1 / 1 step and a 3 x 3 maximum behind it, without LDS:
// nhwc_strip_kernel.
//
// A lane owns V channels (one: two with 16-bit storage measured slower) of a strip of QO output columns and walks down a chunk of output rows with the rows of its windows in
// registers; the lanes of a wave are neighbouring channels (then neighbouring strips), so every access is contiguous.  The
// columns a strip's windows share with the next strip are read and computed by both lanes (they come from the caches):
// no lane waits for another one, any width, any channel count.  Work-groups are numbered so that an XCD gets one contiguous
// part of the tensor (xcd_contiguous).
//
// Arithmetic and order of the other channels-last kernels: every layer rounds to the storage type, averages add row-major from
// +0, the first maximum wins.  Where no index is asked for, an average in front of a maximum is rounded behind it (rounding
// never decreases, so it commutes with the maximum).
//
// What bounds it on MI355X: halo_stress float32 53 us = 4.9 TB/s of input and output (memory, with vector instructions close
// behind), bfloat16 42 us = 3.1 TB/s (vector instructions: conversions and the nine additions per average and its halo); one
// step with indices 4.9 TB/s (ResNet stem bfloat16, 37 us).  The kernels it takes over from: bs_plan.cpp has both sides.
#include <algorithm>

#include "bs_nhwc_device.h"
#include "bs_strip_device.h"

#include "bs_internal.h"

namespace bs {
namespace {

// Element-wise list on N pixels of V channels (pixel-major).  CODE >= 0: kinds compiled in, BatchNorm's parameters read once
// by load(); -1: kinds and parameters read at every use.
template <int DT, int V, int CODE>
struct FwdList {
    static constexpr int L = CODE > 0 ? ew_code_len(CODE) : 0;
    float sc[L ? L : 1][V], sh[L ? L : 1][V];

    BS_DEV void load(const StripK &k, const EwOp *ew, int32_t c)
    {
#pragma unroll
        for (int q = 0; q < L; ++q)
            if (ew_code_kind(CODE, q) == OP_BN)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    sc[q][e] = k.params[ew[q].arg + c + e];
                    sh[q][e] = k.params[ew[q].arg + k.C + c + e];
                }
    }
    template <int N>
    BS_DEV void one(const StripK &k, int32_t kind, int32_t arg, const float (&a)[V], const float (&b)[V], float (&x)[N]) const
    {
        if (kind == OP_BN) {
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = __builtin_fmaf(x[i], a[i % V], b[i % V]);
            round_store_all<DT, N>(x);
        } else if (kind == OP_RELU) {
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = relu(x[i]);
        } else if (kind == OP_LEAKY) {
            const float slope = k.params[arg];
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = round_store<DT>(x[i] > 0.0f ? x[i] : x[i] * slope);
        } else {  // OP_CLAMP
            const float lo = k.params[arg], hi = k.params[arg + 1];
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = round_store<DT>(__builtin_fminf(__builtin_fmaxf(x[i], lo), hi));
        }
    }
    template <int N>
    BS_DEV void apply(const StripK &k, const EwOp *ew, int32_t n, int32_t c, float (&x)[N]) const
    {
        if constexpr (CODE >= 0) {
#pragma unroll
            for (int q = 0; q < L; ++q) one<N>(k, ew_code_kind(CODE, q), ew[q].arg, sc[q], sh[q], x);
        } else {
#pragma clang loop unroll(disable)
            for (int32_t q = 0; q < n; ++q) {
                float a[V] = {}, b[V] = {};
                if (ew[q].kind == OP_BN)
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        a[e] = k.params[ew[q].arg + c + e];
                        b[e] = k.params[ew[q].arg + k.C + c + e];
                    }
                one<N>(k, ew[q].kind, ew[q].arg, a, b, x);
            }
        }
    }
};

// K1: the first pooling (OP_MAXPOOL, OP_AVGSUM; 0: one pooling step only), 3 x 3, stride 1, padding 1; K2: the second (only) one,
// 3 x 3, stride S, padding P.  IDX: the second one's picks are written.  PRE, POST: codes of the lists, or -1 (then the list
// between the poolings is read at run time, too, and averages may have any divisor; otherwise there is none and they divide by nine).
template <int DT, int V, int QO, int K1, int K2, int S, int P, bool IDX, int PRE, int POST, typename OFF>
__global__ __launch_bounds__(256) void nhwc_strip_kernel(const StripK k)
{
    static_assert((S == 1 || S == 2) && (P == 0 || P == 1) && (K1 == 0 || P == 1), "compiled windows");
    constexpr int CA = (QO - 1) * S + 3;              // columns of the plane the second pooling reads
    constexpr int CX = K1 ? CA + 2 : CA;              // columns of the input
    constexpr int ES = elem_bytes<DT>(), KEEP = 3 - S;
    constexpr bool MAX2 = K2 == OP_MAXPOOL, GENERAL = PRE < 0;
    constexpr bool DEFER = K1 == OP_AVGSUM && MAX2 && !IDX && !GENERAL;  // the average is rounded behind the maximum
    constexpr float PAD1 = K1 == OP_MAXPOOL ? -INFINITY : 0.0f, PAD2 = MAX2 ? -INFINITY : 0.0f;
    uint32_t i0 = xcd_contiguous(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
    const bool live = i0 < k.total;
    i0 = live ? i0 : 0u;
    const uint32_t u0 = fdiv(i0, k.div_c);
    const int32_t c0 = (int32_t)(i0 - u0 * k.div_c.d) * V;
    const uint32_t v0 = fdiv(u0, k.div_strips);
    const int32_t ow0 = (int32_t)(u0 - v0 * k.div_strips.d) * QO;
    const uint32_t n = fdiv(v0, k.div_chunks);
    const int32_t chunk = (int32_t)(v0 - n * k.div_chunks.d);

    const int32_t a0 = ow0 * S - P, x0 = K1 ? a0 - 1 : a0;
    const OFF pa = (OFF)(k.C + k.in_xp) * ES, po = (OFF)(k.C + k.out_xp) * ES, arow = (OFF)k.W * pa;
    OFF col[CX];
#pragma unroll
    for (int j = 0; j < CX; ++j) col[j] = (OFF)min(max(x0 + j, 0), k.W - 1) * pa;  // outside the plane: a safe column, replaced below
    const bool inside = x0 >= 0 && x0 + CX <= k.W, whole = ow0 + QO <= k.Wo, lead = P == 1 && ow0 == 0;

    FwdList<DT, V, PRE> pre;
    FwdList<DT, V, POST> post;
    pre.load(k, k.pre, c0);
    post.load(k, k.post, c0);
    const FwdList<DT, V, -1> mid{};

    const int32_t oh0 = chunk * k.rc, oh_end = min(oh0 + k.rc, k.Ho);
    // input rows are requested in order: `next`, at byte offset `at` (clamped to the plane)
    int32_t next = K1 ? oh0 * S - P - 1 : oh0 * S - P;
    OFF at = (OFF)(n * (uint32_t)(k.H * k.W)) * pa + (OFF)c0 * ES + (OFF)min(max(next, 0), k.H - 1) * arow;
    int32_t row1 = oh0 * S - P;  // the next row of the plane the second pooling reads
    float y[2][CX * V];          // K1: the two newest input rows after the leading list

    // the next N input rows -> after the leading list, padding in place
    auto input_rows = [&](auto n_tag, float (&r)[decltype(n_tag)::value][CX * V]) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value;
        float x[N * CX * V];
        bool ok[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            ok[j] = next >= 0 && next < k.H;
#pragma unroll
            for (int c = 0; c < CX; ++c) {
                Raw<DT, V> raw;
                raw.q = *reinterpret_cast<const typename Raw<DT, V>::type *>(static_cast<const char *>(k.in) + (OFF)(at + col[c]));
                float t[V];
                unpack<DT, V>(raw, t);
#pragma unroll
                for (int e = 0; e < V; ++e) x[(j * CX + c) * V + e] = t[e];
            }
            at += next >= 0 && next < k.H - 1 ? arow : (OFF)0;
            ++next;
        }
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
    // one window row of a 3 x 3 average: sum, row-major from +0
    auto sum9 = [&](const float *ra, const float *rb, const float *rc) __attribute__((always_inline)) {
        // a list that ends in a ReLU has no -0, so the sum may start with the first cell instead of +0
        float t = ends_in_relu(PRE) ? ra[0] : 0.0f + ra[0];
        t = t + ra[V];
        t = t + ra[2 * V];
#pragma unroll
        for (int d = 0; d < 3; ++d) t = t + rb[d * V];
#pragma unroll
        for (int d = 0; d < 3; ++d) t = t + rc[d * V];
        return t;
    };
    auto divisor = [&](const PoolK &p, int32_t oh, int32_t ow) __attribute__((always_inline)) {
        if constexpr (!GENERAL) return p.inv_kk;
        const int32_t h = oh * p.sh - p.ph, w = ow * p.sw - p.pw;
        return avg_inv(p, 3, 3, k.H, k.W, h, w, max(h, 0), min(h + 3, k.H), max(w, 0), min(w + 3, k.W));
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
            for (int i = 0; i < CA * V; ++i) a[i] = sum9(ra + i, rb + i, rc + i) * divisor(k.pool1, row1, a0 + i / V);
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
    float m[KEEP][QO * V], w[KEEP][CA * V];
    int32_t cell[KEEP][QO * V];
    auto row_max = [&](const float (&a)[CA * V], int32_t row, float (&mx)[QO * V], int32_t (&ix)[QO * V]) __attribute__((always_inline)) {
        if constexpr (IDX) {
            row_maxima<V, S, QO, CA, 0, P == 1 ? 0 : -1, ends_in_relu(PRE)>(a, lead, mx, ix);
#pragma unroll
            for (int i = 0; i < QO * V; ++i) ix[i] += row * k.W + a0 + (i / V) * S;
        } else {
#pragma unroll
            for (int i = 0; i < QO * V; ++i) {
                const float *p = a + (i / V) * S * V + i % V;
                mx[i] = __builtin_fmaxf(__builtin_fmaxf(p[0], p[V]), p[2 * V]);
            }
        }
    };
    {
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

    const OFF obase = ((OFF)(n * (uint32_t)(k.Ho * k.Wo)) + (OFF)ow0) * po + (OFF)c0 * ES;
    int32_t oh = oh0;
    OFF oat = obase + (OFF)(uint32_t)(oh0 * k.Wo) * po;
    uint32_t iat = (n * (uint32_t)k.Ho + (uint32_t)oh0) * (uint32_t)k.Wo + (uint32_t)ow0;  // IDX: output pixel
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
            const float(&m0)[QO * V] = m[0];
            const float(&m1)[QO * V] = KEEP == 2 ? m[KEEP - 1] : mn[0];
            const float(&m2)[QO * V] = mn[S - 1];
            if constexpr (IDX) {
                const int32_t(&i0)[QO * V] = cell[0];
                const int32_t(&i1)[QO * V] = KEEP == 2 ? cell[KEEP - 1] : cn[0];
                const int32_t(&i2)[QO * V] = cn[S - 1];
                const bool top = P == 1 && oh == 0;  // the first window row lies above the plane: never picked
#pragma unroll
                for (int i = 0; i < QO * V; ++i) {
                    o[i] = m0[i];
                    pick[i] = top ? i1[i] : i0[i];
                    take_if_more(m1[i], i1[i], o[i], pick[i]);
                    take_if_more(m2[i], i2[i], o[i], pick[i]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < QO * V; ++i) o[i] = __builtin_fmaxf(__builtin_fmaxf(m0[i], m1[i]), m2[i]);
            }
            if constexpr (DEFER) round_store_all<DT, QO * V>(o);
#pragma unroll
            for (int j = 0; j < KEEP; ++j)
#pragma unroll
                for (int i = 0; i < QO * V; ++i) {
                    m[j][i] = KEEP == 2 && j == 0 ? m[KEEP - 1][i] : mn[S - 1][i];
                    cell[j][i] = KEEP == 2 && j == 0 ? cell[KEEP - 1][i] : cn[S - 1][i];
                }
        } else {
            const float(&w0)[CA * V] = w[0];
            const float(&w1)[CA * V] = KEEP == 2 ? w[KEEP - 1] : a[0];
            const float(&w2)[CA * V] = a[S - 1];
#pragma unroll
            for (int i = 0; i < QO * V; ++i) {
                const int j = (i / V) * S * V + i % V;
                o[i] = sum9(w0 + j, w1 + j, w2 + j) * divisor(k.pool2, oh, ow0 + i / V);
            }
            round_store_all<DT, QO * V>(o);
#pragma unroll
            for (int j = 0; j < KEEP; ++j)
#pragma unroll
                for (int i = 0; i < CA * V; ++i) w[j][i] = KEEP == 2 && j == 0 ? w[KEEP - 1][i] : a[S - 1][i];
        }
        post.template apply<QO * V>(k, k.post, k.n_post, c0, o);
        if (live) {
            auto put = [&](int j) __attribute__((always_inline)) {
                float t[V];
                int32_t p[V];
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    t[e] = o[j * V + e];
                    p[e] = IDX ? pick[j * V + e] : 0;
                }
                store_elems<DT, V>(static_cast<char *>(k.out) + (OFF)(oat + (OFF)j * po), 0, t);
                if constexpr (IDX) store_indices<V>(k.idx + (iat + (uint32_t)j) * (uint32_t)k.C + (uint32_t)c0, p);
            };
            if (whole) {
#pragma unroll
                for (int j = 0; j < QO; ++j) put(j);
            } else {
#pragma unroll
                for (int j = 0; j < QO; ++j)
                    if (ow0 + j < k.Wo) put(j);
            }
        }
        oat += (OFF)k.Wo * po;
        iat += (uint32_t)k.Wo;
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

constexpr int BN_RELU = OP_BN + OP_RELU * K_EW_BASE;
constexpr int BN_RELU_TWICE = BN_RELU + BN_RELU * K_EW_BASE * K_EW_BASE;

int32_t list_code(const EwOp *ew, int32_t n)
{
    int32_t c = 0, digit = 1;
    if (n > 6) return -1;
    for (int32_t j = 0; j < n; ++j, digit *= K_EW_BASE) c += ew[j].kind * digit;
    return c;
}

template <int DT, int K1, int K2, int S, int P, bool IDX>
void launch_lists(const StripK &k, bool wide, dim3 g, hipStream_t st)
{
    constexpr int V = 1, QO = K_STRIP_QO;
    const int32_t pre = list_code(k.pre, k.n_pre), post = list_code(k.post, k.n_post);
    const bool plain = k.n_mid == 0 && (K1 != OP_AVGSUM || k.pool1.count_include_pad == 1) && (K2 != OP_AVGSUM || k.pool2.count_include_pad == 1);
    if (wide) {
        nhwc_strip_kernel<DT, V, QO, K1, K2, S, P, IDX, -1, -1, uint64_t><<<g, 256, 0, st>>>(k);
        return;
    }
    // the lists of the common networks compiled in; in front of a maximum without indices they have moved behind it
    constexpr bool AVG = K1 == OP_AVGSUM || (K1 == 0 && K2 == OP_AVGSUM);
    constexpr int PRE = AVG || (IDX && K1 == 0) ? BN_RELU : 0, POST = K1 == OP_AVGSUM || (!AVG && !(IDX && K1 == 0)) ? BN_RELU : 0;
    if (plain && pre == PRE && post == POST) {
        nhwc_strip_kernel<DT, V, QO, K1, K2, S, P, IDX, PRE, POST, uint32_t><<<g, 256, 0, st>>>(k);
        return;
    }
    if constexpr (K1 == OP_MAXPOOL && !IDX)  // two blocks of the stacked pooling
        if (plain && pre == 0 && post == BN_RELU_TWICE) {
            nhwc_strip_kernel<DT, V, QO, K1, K2, S, P, IDX, 0, BN_RELU_TWICE, uint32_t><<<g, 256, 0, st>>>(k);
            return;
        }
    if constexpr (K1 == 0 && K2 == OP_AVGSUM)  // the pooling branch of an Inception module
        if (plain && pre == 0 && post == 0) {
            nhwc_strip_kernel<DT, V, QO, K1, K2, S, P, IDX, 0, 0, uint32_t><<<g, 256, 0, st>>>(k);
            return;
        }
    nhwc_strip_kernel<DT, V, QO, K1, K2, S, P, IDX, -1, -1, uint32_t><<<g, 256, 0, st>>>(k);
}

template <int DT, int K1, int K2>
void launch_windows(const StripK &k, bool wide, dim3 g, hipStream_t st)
{
    const PoolK &p = k.pool2;
    constexpr bool MAX2 = K2 == OP_MAXPOOL;
#define BS_STRIP(S, P)                                                                    \
    do {                                                                                  \
        if (MAX2 && k.idx) launch_lists<DT, K1, K2, S, P, MAX2>(k, wide, g, st);       \
        else launch_lists<DT, K1, K2, S, P, false>(k, wide, g, st);                    \
    } while (0)
    if (p.sh == 2 && p.ph == 1) BS_STRIP(2, 1);
    else if (p.sh == 1 && p.ph == 1) BS_STRIP(1, 1);
    else if constexpr (K1 == 0) {
        if (p.sh == 2) BS_STRIP(2, 0);
        else BS_STRIP(1, 0);
    }
#undef BS_STRIP
}

template <int DT>
void launch_kinds(const StripK &k, bool wide, dim3 g, hipStream_t st)
{
    if (k.pool1.kind == OP_AVGSUM) launch_windows<DT, OP_AVGSUM, OP_MAXPOOL>(k, wide, g, st);
    else if (k.pool1.kind == OP_MAXPOOL) launch_windows<DT, OP_MAXPOOL, OP_MAXPOOL>(k, wide, g, st);
    else if (k.pool2.kind == OP_MAXPOOL) launch_windows<DT, 0, OP_MAXPOOL>(k, wide, g, st);
    else launch_windows<DT, 0, OP_AVGSUM>(k, wide, g, st);
}

}  // namespace

bool nhwc_strips_supported(const StripK &k)
{
    const PoolK &p = k.pool1, &q = k.pool2;
    auto is3 = [](const PoolK &w) {
        return (w.kind == OP_MAXPOOL || w.kind == OP_AVGSUM) && w.kh == 3 && w.kw == 3 && w.sh == w.sw && w.ph == w.pw && (w.sh == 1 || w.sh == 2) &&
               w.ph >= 0 && w.ph <= 1;
    };
    if (!is3(q)) return false;
    if (p.kind != 0 && (!is3(p) || p.sh != 1 || p.ph != 1 || q.ph != 1 || q.kind != OP_MAXPOOL)) return false;
    const EwOp *lists[3] = {k.pre, k.mid, k.post};
    const int32_t counts[3] = {k.n_pre, k.n_mid, k.n_post};
    for (int l = 0; l < 3; ++l)
        for (int32_t j = 0; j < counts[l]; ++j)
            if (lists[l][j].kind == OP_ADD) return false;  // strips do not read residual operands
    return true;
}

bs_status launch_nhwc_strips(const StripK &k, int32_t dtype, int64_t grid, void *stream)
{
    const int32_t qo = K_STRIP_QO;
    // what the kernel assumes: the windows and lists above, strips and chunks that cover the output, no empty chunk, the divisors
    // of the lane numbering
    if (!nhwc_strips_supported(k) || grid < 1 || grid > 0x7fffffffll || (uint64_t)grid * 256 < k.total ||
        (int64_t)k.div_c.d != k.C || k.strips != (k.Wo + qo - 1) / qo || (int64_t)k.div_strips.d != k.strips ||
        (int64_t)k.div_chunks.d != k.chunks || k.rc < 1 || (int64_t)k.chunks * k.rc < k.Ho || (int64_t)(k.chunks - 1) * k.rc >= k.Ho ||
        k.total % ((uint64_t)k.strips * k.chunks * k.div_c.d) != 0)
        return BS_ERR_UNSUPPORTED;
    // 32-bit byte offsets where every tensor ends below 4 GiB
    const uint64_t images = k.total / ((uint64_t)k.strips * k.chunks * k.div_c.d), es = dtype == BS_F32 ? 4 : 2;
    const uint64_t far = std::max(images * k.H * k.W * ((uint64_t)k.C + k.in_xp), images * k.Ho * k.Wo * ((uint64_t)k.C + k.out_xp)) * es;
    const bool wide = far > 0xffffffffull;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 g((uint32_t)grid);
    if (dtype == BS_F32) launch_kinds<DT_F32>(k, wide, g, st);
    else if (dtype == BS_BF16) launch_kinds<DT_BF16>(k, wide, g, st);
    else if (dtype == BS_F16) launch_kinds<DT_F16>(k, wide, g, st);
    else return BS_ERR_UNSUPPORTED;
    return BS_OK;
}

}  // namespace bs
