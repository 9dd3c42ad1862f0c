// Backward kernels of stages with overlapping 3 x 3 pooling windows whose lanes walk strips of columns: no recorded picks, no
// recomputation pass, nothing through the workspace.
//
// A lane owns one channel of a strip of Q columns and walks down a chunk of rows; the columns a strip's windows reach into
// beside it are read and computed by the lane itself -- they come from the caches, and no lane waits for another one: no LDS,
// no barrier, no lane exchange, any width and any channel count.  (Two channels per lane, 16-bit storage, measured the same in
// the one-level kernel and spill in the two-level one.)
//   Channels-last tensors (CL): the lanes of a wave are neighbouring channels, then neighbouring strips; every access is contiguous.
//   Row-major tensors: the lanes are neighbouring strips of a row; a lane reads and writes its columns as vectors at whatever
//   address they begin.
// Work-groups are numbered so that each XCD gets one contiguous part of the tensor (xcd_contiguous): the strips that share
// columns find them in one L2.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bs_bwd_device.h"
#include "bs_strip_device.h"
#include "bs_internal.h"

namespace bs {
namespace {

// OFF: the type of byte offsets -- uint32_t where every tensor of the launch ends below 4 GiB (one address addition per access:
// the base stays in scalar registers), else uint64_t.  Byte offset `off` of n elements, checked in audit builds.
template <int DT, typename OFF>
BS_DEV OFF audited_bytes(const BwdK &k, int which, int site, OFF off, uint32_t n)
{
#if defined(BS_BWD_AUDIT)
    return audited<OFF>(k, which, site, off / elem_bytes<DT>(), n) * elem_bytes<DT>();
#else
    return off;
#endif
}

// One element at byte offset `off`, as it lies in memory.
// (V = 2: two 16-bit elements in one word, at a multiple of four bytes)
template <int DT, typename OFF, int V = 1>
BS_DEV uint32_t load_at(const BwdK &k, int which, int site, const void *base, OFF off)
{
    uint32_t w[1];
    load_run<DT, V>(static_cast<const char *>(base) + audited_bytes<DT, OFF>(k, which, site, off, V), w);
    return w[0];
}

// Non-temporal: the input gradient is written once.  Measured, channels-last backward (bwd_keys_kernel), us, plain / non-temporal: ResNet stem bfloat16
// 50.2 / 46.2, float32 100.9 / 94; 32 x 192 x 71 x 71 bfloat16 38.3 / 35.2.
template <int DT, typename OFF, int V = 1>
BS_DEV void store_at(const BwdK &k, int site, void *base, OFF off, const float *v)
{
    store_elems<DT, V>(NonTemporal{}, static_cast<char *>(base) + audited_bytes<DT, OFF>(k, 2, site, off, V), v);
}

// Words that hold N columns of a row: channels-last one per column, row-major the run as it lies in memory.
template <int DT, bool CL, int N>
constexpr int row_words() { return CL ? N : run_words<DT, N>(); }

// N columns of a row at byte offset `row`, column j at + col[j] (outside the plane: a safe column, the caller replaces it).
// Row-major: the run from column `first` is read whole if it begins at `last` at the latest (so that it ends inside the tensor;
// columns beside the plane are other rows' elements then), else one by one.
template <int DT, bool CL, int N, typename OFF, int V = 1>
BS_DEV void load_row(const BwdK &k, int which, int site, const void *base, OFF row, const OFF (&col)[N], int32_t first, bool fits, OFF last,
                     uint32_t (&w)[row_words<DT, CL, N>()])
{
    if constexpr (CL) {
#pragma unroll
        for (int j = 0; j < N; ++j) w[j] = load_at<DT, OFF, V>(k, which, site, base, row + col[j]);
    } else {
        const OFF from = row + (OFF)first * (OFF)elem_bytes<DT>();
        if (fits && from <= last) {
            load_run<DT, N>(static_cast<const char *>(base) + audited_bytes<DT, OFF>(k, which, site, from, N), w);
        } else {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const uint32_t e = load_at<DT, OFF>(k, which, site, base, row + col[j]);
                if constexpr (DT == DT_F32) w[j] = e;
                else w[j / 2] = j % 2 ? w[j / 2] | e << 16 : e;
            }
        }
    }
}
template <int DT, bool CL, int N, int V = 1>
BS_DEV void unpack_row(const uint32_t (&w)[row_words<DT, CL, N>()], float *v)
{
#pragma unroll
    for (int j = 0; j < N * V; ++j) v[j] = V == 2 ? run_element<DT>(&w[j / V], j % V) : CL ? run_element<DT>(&w[CL ? j : 0], 0) : run_element<DT>(w, j);
}

// N columns of a row of the input gradient, `pitch` bytes apart; whole: all of them lie in the plane.
template <int DT, bool CL, int N, typename OFF, int V = 1>
BS_DEV void store_row(const BwdK &k, int site, OFF at, int32_t first, int32_t width, OFF pitch, bool whole, const float (&v)[N * V])
{
    if constexpr (!CL) {
        if (whole) {
            store_run<DT, N>(static_cast<char *>(k.g_in) + audited_bytes<DT, OFF>(k, 2, site, at, N), v);
            return;
        }
    }
    if (whole) {
#pragma unroll
        for (int j = 0; j < N; ++j) store_at<DT, OFF, V>(k, site, k.g_in, at + (OFF)j * pitch, v + j * V);
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (first + j < width) store_at<DT, OFF, V>(k, site, k.g_in, at + (OFF)j * pitch, v + j * V);
    }
}

// The lane's place.  Channels-last: (image, chunk, strip, V channels), row-major: (image, channel, chunk, strip), the last one fastest.
struct StripLane {
    bool live;
    uint32_t n, plane;
    int32_t chunk, q0, c0;
};

template <bool CL, int Q, int V = 1>
BS_DEV StripLane strip_lane(const BwdK &k)
{
    StripLane L;
    uint32_t i = xcd_contiguous(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
    L.live = i < k.total;
    i = L.live ? i : 0u;
    uint32_t v = i;
    L.plane = 0;
    if constexpr (CL) {
        v = fdiv(i, k.div_wv);
        L.c0 = (int32_t)(i - v * k.div_wv.d) * V;
    }
    const uint32_t u = fdiv(v, k.div_cbs);
    L.q0 = (int32_t)(v - u * k.div_cbs.d) * Q;
    const uint32_t p = fdiv(u, k.div_chunks);
    L.chunk = (int32_t)(u - p * k.div_chunks.d);
    L.n = p;
    if constexpr (!CL) {
        L.plane = p;
        L.n = fdiv(p, k.div_c);
        L.c0 = (int32_t)(p - L.n * k.div_c.d);
    }
    return L;
}

// Where the lane's rows begin and how far columns and rows lie apart (bytes).
template <int DT, bool CL, typename OFF>
struct StripPlaces {
    OFF pa, pg, pi, abase, gbase, ibase, arow, grow, irow;
    BS_DEV StripPlaces(const BwdK &k, const StripLane &L)
    {
        constexpr int ES = elem_bytes<DT>();
        pa = CL ? (OFF)(k.C + k.a_extra) * ES : (OFF)ES;
        pg = CL ? (OFF)(k.C + k.gout_extra) * ES : (OFF)ES;
        pi = CL ? (OFF)(k.C + k.gin_extra) * ES : (OFF)ES;
        const uint32_t in_px = (uint32_t)(k.H * k.W), out_px = (uint32_t)(k.Ho * k.Wo);
        abase = CL ? (OFF)(L.n * in_px) * pa + (OFF)L.c0 * ES : ((OFF)(L.plane * in_px) + (OFF)L.n * k.a_extra) * ES;
        gbase = CL ? (OFF)(L.n * out_px) * pg + (OFF)L.c0 * ES : ((OFF)(L.plane * out_px) + (OFF)L.n * k.gout_extra) * ES;
        ibase = (CL ? (OFF)(L.n * in_px) * pi + (OFF)L.c0 * ES : ((OFF)(L.plane * in_px) + (OFF)L.n * k.gin_extra) * ES) + (OFF)L.q0 * pi;
        arow = (OFF)k.W * pa;
        grow = (OFF)k.Wo * pg;
        irow = (OFF)k.W * pi;
    }
};

// at == AT: sum += g
template <int AT, bool FIRST>
BS_DEV void add_if_at(int32_t at, float g, float &sum)
{
    const float t = at == AT ? g : 0.0f;
    sum = FIRST ? t : sum + t;  // FIRST: nothing there yet
}

// An element-wise list on N pixels of V channels (pixel-major), with the product t of its derivatives: float32, rounded
// to the storage type after every layer, as the forward kernels compute it.  CODE >= 0: the kinds are compile-time
// (base-K_EW_BASE digits) and load() reads the parameters of the lane's channels once, in front of the row loop; -1: kinds and
// parameters are read at every use -- HOLD: those of the first HELD operations once per lane (two levels, 64 x 64 x 55 x 55 row-major
// float32 with leaky ReLU 100 -> 75 us; one level: 4 % faster in float32, up to 6 % slower with 16-bit storage, so read at every use).
template <int DT, int V, int CODE, bool HOLD>
struct StripList {
    static constexpr int HELD = HOLD ? 4 : 0, L = CODE > 0 ? ew_code_len(CODE) : CODE == 0 ? 0 : HELD;
    HeldParams<V> held[L ? L : 1];
    uint32_t kinds;  // HOLD: K_EW_BASE digits
    int32_t first, count, c0;

    BS_DEV void load(const BwdK &k, int32_t c, int32_t f, int32_t n)
    {
        first = f;
        count = n;
        c0 = c;
        kinds = 0;
#pragma unroll
        for (int q = 0; q < L; ++q) {
            if constexpr (CODE >= 0) {
                if (CODE == BN_RELU && q == 0 && n == 1) held[q].identity();  // ReLU alone
                else held[q].load(k.params, ew_code_kind(CODE, q), k.ew[f + q].arg, c, k.C);
            } else {
                const bool there = q < n;
                const int32_t kind = there ? k.ew[f + q].kind : (int32_t)OP_RELU;
                kinds |= (uint32_t)kind << (4 * q);
                held[q].load(k.params, kind, there ? k.ew[f + q].arg : 0, c, k.C);
            }
        }
    }

    template <int N, typename P>
    BS_DEV static void one(int32_t kind, const P &p, float (&x)[N], float (&t)[N])
    {
        if (kind == OP_BN) {
            float a[V], b[V];
            p.bn(a, b);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                x[i] = __builtin_fmaf(x[i], a[i % V], b[i % V]);
                t[i] *= a[i % V];
            }
            round_store_all<DT, N>(x);
        } else if (kind == OP_RELU) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                t[i] = x[i] > 0.0f ? t[i] : 0.0f;
                x[i] = __builtin_fmaxf(x[i], 0.0f);  // NaN, -0 -> +0
            }
        } else if (kind == OP_LEAKY) {
            const float slope = p.first();
#pragma unroll
            for (int i = 0; i < N; ++i) {
                t[i] *= x[i] > 0.0f ? 1.0f : slope;
                x[i] = round_store<DT>(x[i] > 0.0f ? x[i] : x[i] * slope);
            }
        } else {  // OP_CLAMP: the gradient passes where lo <= x <= hi
            const float lo = p.first(), hi = p.second();
#pragma unroll
            for (int i = 0; i < N; ++i) {
                t[i] = x[i] >= lo && x[i] <= hi ? t[i] : 0.0f;
                x[i] = round_store<DT>(__builtin_fminf(__builtin_fmaxf(x[i], lo), hi));
            }
        }
    }

    template <int N>
    BS_DEV void apply(const BwdK &k, float (&x)[N], float (&t)[N]) const
    {
        static_assert(N % V == 0, "whole pixels");
#pragma unroll
        for (int i = 0; i < N; ++i) t[i] = 1.0f;
        if constexpr (CODE >= 0) {
#pragma unroll
            for (int q = 0; q < L; ++q) one<N>(ew_code_kind(CODE, q), held[q], x, t);
        } else {
#pragma clang loop unroll(disable)
            for (int32_t q = first; q < first + count; ++q) {
                if constexpr (HOLD) {
                    const int32_t i = q - first;
                    HeldParams<V> p;
                    int32_t kind = k.ew[q].kind;
                    if (i < HELD) {
                        kind = (int32_t)(kinds >> (4 * i) & 15u);
#pragma unroll
                        for (int e = 0; e < V; ++e) {
                            p.a[e] = one_of(i, held[0].a[e], held[1].a[e], held[2].a[e], held[3].a[e]);
                            p.b[e] = one_of(i, held[0].b[e], held[1].b[e], held[2].b[e], held[3].b[e]);
                        }
                    } else {
                        p.load(k.params, kind, k.ew[q].arg, c0, k.C);
                    }
                    one<N>(kind, p, x, t);
                } else {
                    one<N>(k.ew[q].kind, ReadParams<V>{k.params, k.ew[q].arg, c0, k.C}, x, t);
                }
            }
        }
    }
};
static_assert(K_EW_BASE == 16, "a digit of `kinds` is four bits");

// The windows' picks from the row maxima of their three rows.  top: the first window row lies above the plane (padding, all
// -infinity) and must not be picked, not even by a window of nothing but -infinity.
template <int N, bool BY_MAX>
BS_DEV void combine_rows(const float (&m0)[N], const int32_t (&code0)[N], const float (&m1)[N], const int32_t (&code1)[N], const float (&m2)[N],
                         const int32_t (&code2)[N], bool top, float (&best)[N], int32_t (&pick)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        best[i] = m0[i];
        pick[i] = top ? code1[i] : code0[i];
        if constexpr (BY_MAX) {
            max_if_more(m1[i], code1[i], best[i], pick[i]);
            max_if_more(m2[i], code2[i], best[i], pick[i]);
        } else {
            take_if_more(m1[i], code1[i], best[i], pick[i]);
            take_if_more(m2[i], code2[i], best[i], pick[i]);
        }
    }
}

// sum[window row][column] += the gradients of the windows that picked the cell, left windows first: window b begins at column
// X0 + b * S of the strip's G columns.  Rows FRESH, FRESH + 1 ... hold nothing yet: their first window writes.
// KEYS: picks are codes of keys, (2 - row) * 16 + 15 - strip column; else 3 * row + window column.
template <int V, int S, int N, int X0, int G, int FRESH, bool KEYS = false>
BS_DEV void scatter(const int32_t (&pick)[N * V], const float (&g)[N * V], float (&sum0)[G * V], float (&sum1)[G * V], float (&sum2)[G * V])
{
    auto cell = [&](auto dh_tag, auto dw_tag, auto b_tag) __attribute__((always_inline)) {
        constexpr int dh = decltype(dh_tag)::value, dw = decltype(dw_tag)::value, b = decltype(b_tag)::value, col = X0 + b * S + dw;
        // the first window over this column: the smallest b with X0 + b * S + 2 >= col
        constexpr int b0 = col - 2 - X0 <= 0 ? 0 : (col - 2 - X0 + S - 1) / S;
        if constexpr (col >= 0 && col < G) {
#pragma unroll
            for (int e = 0; e < V; ++e)
                add_if_at<KEYS ? (2 - dh) * 16 + 15 - (b * S + dw) : 3 * dh + dw, (dh >= FRESH && b == b0)>(pick[b * V + e], g[b * V + e],
                                                                 (dh == 0 ? sum0 : dh == 1 ? sum1 : sum2)[col * V + e]);
        }
    };
    auto window = [&](auto dh_tag, auto b_tag) __attribute__((always_inline)) {
        cell(dh_tag, std::integral_constant<int, 0>{}, b_tag);
        cell(dh_tag, std::integral_constant<int, 1>{}, b_tag);
        cell(dh_tag, std::integral_constant<int, 2>{}, b_tag);
    };
    auto row = [&](auto dh_tag) __attribute__((always_inline)) {
        each_of(std::make_integer_sequence<int, N>{}, [&](auto b_tag) __attribute__((always_inline)) { window(dh_tag, b_tag); });
    };
    row(std::integral_constant<int, 0>{});
    row(std::integral_constant<int, 1>{});
    row(std::integral_constant<int, 2>{});
}

// =============================================================================
// bwd_strip_kernel: [list, max pooling 3 x 3 with stride S = 1 or 2 and padding P = 0 or 1, list] (the ResNet and Inception
// stems, the pools of SqueezeNet and AlexNet).  Per window row the lane reads S new input rows, finds the row maxima
// of its windows in each (a row two window rows share is scanned once), combines three of them into the windows' picks,
// adds the windows' gradients -- times the trailing list's derivative at the maximum -- to the picked cells and writes
// the S rows no later window reaches.  A cell sums its windows in row-major window order.
// PRE, POST: codes of the lists, or -1 (small stages with such lists gather kept picks instead: bs_backward.cpp).  BatchNorm -> ReLU or ReLU
// alone in front and nothing behind: bwd_keys_kernel.
// Measured on MI355X with BatchNorm -> ReLU in front (before bwd_keys_kernel took that list over), us of a call with the caller's picks at
// hand, gathering kernel -> this one: ResNet stem 64 x 64 x 112 x 112 float32 105 -> 98 (waits for memory), bfloat16 87 -> 60 (vector
// instructions: 36 per cell, 70 % of the time); without kept picks the gathering kernel needs a forward pass on top (row-major 64 x 64 x 111 x
// 111 / 2 float32 385 -> 145; whole vectors without padding, 32 x 64 x 112 x 112 / 2, 180 -> 72).
// =============================================================================
template <int DT, bool CL, int Q, int S, int P, int PRE, int POST, typename OFF>
__global__ __launch_bounds__(256) void bwd_strip_kernel(const BwdK k)
{
    static_assert(Q % S == 0 && (S == 1 || S == 2) && (P == 0 || P == 1), "compiled windows");
    static_assert(PRE == 0 || PRE == -1, "BatchNorm, ReLU in front and nothing behind: bwd_keys_kernel");
    constexpr int OW0 = -((2 - P) / S);            // first window over the strip: q0 / S + OW0 = ceil((q0 + P - 2) / S)
    constexpr int NW = (Q + 1) / S + 1;            // windows over the strip
    constexpr int X0 = OW0 * S - P;                // their first column, from q0
    constexpr int CW = (NW - 1) * S + 3;           // their columns
    constexpr int KEEP = 3 - S, V = 1, ES = elem_bytes<DT>();
    constexpr int OEND = (P + S - 1) / S;
    const StripLane L = strip_lane<CL, Q>(k);
    const StripPlaces<DT, CL, OFF> at0(k, L);
    const OFF pa = at0.pa, pg = at0.pg, pi = at0.pi, arow = at0.arow, grow = at0.grow, irow = at0.irow;

    const int32_t x0 = L.q0 + X0, ow0 = L.q0 / S + OW0;
    constexpr int LEAD = P == 1 ? -OW0 : -1;
    const bool lead = L.q0 == 0;
    OFF acol[CW], gcol[NW];
    bool win[NW];
#pragma unroll
    for (int j = 0; j < CW; ++j) acol[j] = (OFF)min(max(x0 + j, 0), k.W - 1) * pa;  // outside the plane: a safe column, replaced below
#pragma unroll
    for (int b = 0; b < NW; ++b) {
        win[b] = ow0 + b >= 0 && ow0 + b < k.Wo;
        gcol[b] = (OFF)min(max(ow0 + b, 0), k.Wo - 1) * pg;
    }
    const bool a_fits = k.a_bytes >= (uint64_t)CW * ES, g_fits = k.g_bytes >= (uint64_t)NW * ES;
    const OFF a_last = a_fits ? (OFF)(k.a_bytes - (uint64_t)CW * ES) : (OFF)0, g_last = g_fits ? (OFF)(k.g_bytes - (uint64_t)NW * ES) : (OFF)0;
    const bool inside = x0 >= 0 && x0 + CW <= k.W, whole = L.q0 + Q <= k.W;

    StripList<DT, V, PRE, false> pre;
    StripList<DT, V, POST, false> post;
    pre.load(k, L.c0, 0, k.n_ew);
    post.load(k, L.c0, k.n_ew, k.n_post);

    const int32_t r_lo = L.chunk * k.rc * S, r_hi = min(r_lo + k.rc * S, k.H);  // rows this chunk writes
    const int32_t oh_first = L.chunk * k.rc + OW0;
    float m[3][NW * V], s[3][Q * V], t[3][Q * V];
    int32_t code[3][NW * V];
    // rows are requested in order, `at` = the offset of row `next` (clamped to the plane)
    int32_t next = oh_first * S - P;
    OFF at = at0.abase + (OFF)min(max(next, 0), k.H - 1) * arow;
    OFF gat = at0.gbase + (OFF)min(max(oh_first, 0), k.Ho - 1) * grow;
    OFF iat = at0.ibase + (OFF)r_lo * irow;
    // the next N rows -> ring slots slots(0) .. slots(N - 1), scanned as window rows DH0, DH0 + 1 ...
    auto take_rows = [&](auto n_tag, auto dh_tag, auto slot_of) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value, DH0 = decltype(dh_tag)::value;
        float x[N * CW * V], d[N * CW * V];
        uint32_t w[N][row_words<DT, CL, CW>()];  // requested for all rows before the first is used
        bool ok[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            ok[j] = next >= 0 && next < k.H;
            load_row<DT, CL, CW, OFF>(k, 0, 40, k.a, at, acol, x0, a_fits, a_last, w[j]);
            at += next >= 0 && next < k.H - 1 ? arow : (OFF)0;
            ++next;
        }
#pragma unroll
        for (int j = 0; j < N; ++j) unpack_row<DT, CL, CW>(w[j], &x[j * CW]);
        pre.template apply<N * CW * V>(k, x, d);
        each_of(std::make_integer_sequence<int, N>{}, [&](auto j_tag) __attribute__((always_inline)) {
            constexpr int j = decltype(j_tag)::value, dh = DH0 + j;
            const int slot = slot_of(j);
            float y[CW * V];
#pragma unroll
            for (int i = 0; i < CW * V; ++i) y[i] = x[j * CW * V + i];
            if (!(inside && ok[j])) {
#pragma unroll
                for (int i = 0; i < CW * V; ++i) {
                    const int32_t c = x0 + i / V;
                    y[i] = ok[j] && c >= 0 && c < k.W ? y[i] : -INFINITY;
                }
            }
            row_maxima<V, S, NW, CW, dh, LEAD, false>(y, lead, m[slot], code[slot]);
#pragma unroll
            for (int i = 0; i < Q * V; ++i) {
                t[slot][i] = d[(j * CW - X0) * V + i];
                if (dh < KEEP) s[slot][i] = 0.0f;
            }
        });
    };
    if constexpr (KEEP > 0) take_rows(std::integral_constant<int, KEEP>{}, std::integral_constant<int, 0>{}, [](int j) { return j; });

    int32_t oh = oh_first;
    // one window row; its three rows are in ring slots R0 (stride 2: two rows are new, the third's slot and the first's change
    // roles from one window row to the next; stride 1: the rows move up)
    auto step = [&](auto par) __attribute__((always_inline)) {
        constexpr int R0 = decltype(par)::value ? 2 : 0, R2 = 2 - R0;
        const int32_t hA = oh * S - P;
        const bool row_ok = oh >= 0 && oh < k.Ho;
        float g[NW * V];
        uint32_t gw[row_words<DT, CL, NW>()];
        load_row<DT, CL, NW, OFF>(k, 1, 41, k.g_out, gat, gcol, ow0, g_fits, g_last, gw);
        gat += oh >= 0 && oh < k.Ho - 1 ? grow : (OFF)0;
        take_rows(std::integral_constant<int, S>{}, std::integral_constant<int, KEEP>{}, [](int j) { return KEEP + j == 2 ? R2 : KEEP + j; });
        unpack_row<DT, CL, NW>(gw, g);
        float best[NW * V];
        int32_t pick[NW * V];
        combine_rows<NW * V, false>(m[R0], code[R0], m[1], code[1], m[R2], code[R2], hA < 0, best, pick);
#pragma unroll
        for (int i = 0; i < NW * V; ++i) g[i] = row_ok && win[i / V] ? g[i] : 0.0f;  // windows that do not exist give nothing
        if constexpr (POST != 0) {
            float tp[NW * V];
            post.template apply<NW * V>(k, best, tp);
#pragma unroll
            for (int i = 0; i < NW * V; ++i) g[i] *= tp[i];
        }
        scatter<V, S, NW, X0, Q, KEEP>(pick, g, s[R0], s[1], s[R2]);
        // the S rows no later window row holds are complete
#pragma unroll
        for (int d = 0; d < S; ++d) {
            const int32_t row = hA + d;
            const int slot = d == 0 ? R0 : 1;
            if (L.live && row >= r_lo && row < r_hi) {
                float v[Q * V];
#pragma unroll
                for (int i = 0; i < Q * V; ++i) v[i] = s[slot][i] * t[slot][i];
                store_row<DT, CL, Q, OFF>(k, 42, iat, L.q0, k.W, pi, whole, v);
                iat += irow;
            }
        }
        if constexpr (S == 2) {
#pragma unroll
            for (int i = 0; i < NW * V; ++i) code[R2][i] -= 6;
        } else {
#pragma unroll
            for (int d = 0; d < KEEP; ++d) {
#pragma unroll
                for (int i = 0; i < NW * V; ++i) {
                    m[d][i] = m[d + 1][i];
                    code[d][i] = code[d + 1][i] - 3;
                }
#pragma unroll
                for (int i = 0; i < Q * V; ++i) {
                    s[d][i] = s[d + 1][i];
                    t[d][i] = t[d + 1][i];
                }
            }
        }
        ++oh;
    };
    const int32_t oh_end = oh_first + k.rc + OEND - OW0;  // as many window rows for every lane
    for (;;) {
        step(std::integral_constant<int, 0>{});
        if (oh == oh_end) break;
        if constexpr (S == 2) {
            step(std::integral_constant<int, 1>{});
            if (oh == oh_end) break;
        }
    }
}

// =============================================================================
// bwd_strip2_kernel: [list, average pooling 3 x 3 / 1 / 1] and [max pooling 3 x 3 / 2 / 1, list] in one kernel; the plane
// between the poolings and its gradient (float32) stay in registers.  Per window row `oh` of the max pooling a lane
//   1. reads the input rows 2 oh + 1, 2 oh + 2 and applies the leading list (values y, derivatives T),
//   2. forms rows 2 oh, 2 oh + 1 of the average's output in the forward kernels' arithmetic (row-major sum from +0, times
//      the divisor's reciprocal, rounded to storage) and their windows' row maxima,
//   3. combines rows 2 oh - 1 .. 2 oh + 1 into the picks and adds the upstream gradients, scaled by the trailing list's
//      derivative at the maximum, to the picked cells,
//   4. average rows 2 oh - 1, 2 oh can get nothing more: their gradients times the divisor's reciprocal, summed over the
//      three windows of the row that hold a cell (rows of hs),
//   5. writes the input gradient of rows 2 oh - 2, 2 oh - 1: hs of the rows above, at and below, times T.
// Q columns need Q + 2 of the average's gradient, Q / 2 + 2 windows, Q + 5 averages and Q + 7 inputs.
// INC: every divisor is 9 (count_include_pad, nothing overhangs).
// Measured on MI355X (halo_stress, us of a call): three stages with two forward passes through the workspace -> this kernel:
// float32 510 -> 106, bfloat16 390 -> 101; row-major, 64 x 64 x 55 x 55 float32 291 -> 65, binary16 287 -> 43.  Bound by vector
// instructions (the 18 additions per average and their halo, the scans); two waves per SIMD with 8 columns beat four with 4
// columns, which compute 9 averages per 4 columns instead of 13 per 8.
// Lists read at run time (PRE, POST -1): 4 columns, so that nothing lies in scratch memory; three stages / 8 columns with scratch / 4
// columns, 64 x 64 x 55 x 55 channels-last: BatchNorm, leaky ReLU, average, maximum, BatchNorm, leaky ReLU float32 143 / 65 / 63, bfloat16
// 117 / 69 / 74; halo_stress's lists without padding counted float32 147 / 180 / 94, bfloat16 116 / 170 / 100; 8 x 64 x 28 x 28 27 / 53 / 25.
// =============================================================================
// Waves per SIMD: what the registers of an instance allow without scratch memory.
constexpr int strip2_waves(int Q, int PRE, int off_bytes) { return off_bytes == 8 ? 1 : Q == 8 || PRE < 0 ? 2 : 3; }

template <int DT, bool CL, int Q, bool INC, int PRE, int POST, typename OFF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(strip2_waves(Q, PRE, sizeof(OFF)), strip2_waves(Q, PRE, sizeof(OFF)))))
void bwd_strip2_kernel(const BwdK k)
{
    static_assert(Q % 2 == 0, "whole windows");
    constexpr int NW = Q / 2 + 2, CA = Q + 5, CX = Q + 7, CG = Q + 2, V = 1, ES = elem_bytes<DT>();
    const StripLane L = strip_lane<CL, Q>(k);
    const StripPlaces<DT, CL, OFF> at0(k, L);
    const OFF pa = at0.pa, pg = at0.pg, pi = at0.pi, arow = at0.arow, grow = at0.grow, irow = at0.irow;

    const int32_t x0 = L.q0 - 4, ow0 = L.q0 / 2 - 1;
    const bool lead = L.q0 == 0;
    OFF acol[CX], gcol[NW];
    bool win[NW];
#pragma unroll
    for (int j = 0; j < CX; ++j) acol[j] = (OFF)min(max(x0 + j, 0), k.W - 1) * pa;  // outside the plane: a safe column, replaced below
#pragma unroll
    for (int b = 0; b < NW; ++b) {
        win[b] = ow0 + b >= 0 && ow0 + b < k.Wo;
        gcol[b] = (OFF)min(max(ow0 + b, 0), k.Wo - 1) * pg;
    }
    const bool a_fits = k.a_bytes >= (uint64_t)CX * ES, g_fits = k.g_bytes >= (uint64_t)NW * ES;
    const OFF a_last = a_fits ? (OFF)(k.a_bytes - (uint64_t)CX * ES) : (OFF)0, g_last = g_fits ? (OFF)(k.g_bytes - (uint64_t)NW * ES) : (OFF)0;
    const bool inside = x0 >= 0 && x0 + CX <= k.W, whole = L.q0 + Q <= k.W;

    StripList<DT, V, PRE, true> pre;
    StripList<DT, V, POST, true> post;
    pre.load(k, L.c0, 0, k.n_ew);
    post.load(k, L.c0, k.n_ew, k.n_post);

    const int32_t r_lo = L.chunk * k.rc * 2, r_hi = min(r_lo + k.rc * 2, k.H);
    const int32_t oh_first = L.chunk * k.rc - 1;

    // KEYS: averages of values that are not negative, 16-bit storage -- window maxima as keys of value and place (PickKey; a code is
    // (2 - window row) * 16 + 15 - column).  halo_stress, us, compares / keys: bfloat16 116 / 101, binary16 102 / 98; float32 106 / 116 (its keys are doubles).
    constexpr bool KEYS = ends_in_relu(PRE) && DT != DT_F32;
    static_assert(CA <= 15, "a code holds four bits of column");
    using Key = PickKey<DT>;
    float y[4][CX * V], T[5][Q * V], m[3][KEYS ? 1 : NW * V], gt[3][CG * V], hs[4][Q * V];
    int32_t code[3][KEYS ? 1 : NW * V];
    Key km[3][KEYS ? NW * V : 1];
    // rows are requested in order, `at` = the offset of row `next` (clamped to the plane)
    int32_t next = oh_first * 2 - 2;
    OFF at = at0.abase + (OFF)min(max(next, 0), k.H - 1) * arow;
    OFF gat = at0.gbase + (OFF)min(max(oh_first, 0), k.Ho - 1) * grow;
    OFF iat = at0.ibase + (OFF)r_lo * irow;
    // the next N rows: leading list -> y (outside the plane +0, the average's padding), derivatives -> T
    auto take_rows = [&](auto n_tag, int slot, int tslot) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value;
        float x[N * CX * V], d[N * CX * V];
        uint32_t w[N][row_words<DT, CL, CX>()];  // requested for all rows before the first is used
        bool ok[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            ok[j] = next >= 0 && next < k.H;
            load_row<DT, CL, CX, OFF>(k, 0, 43, k.a, at, acol, x0, a_fits, a_last, w[j]);
            at += next >= 0 && next < k.H - 1 ? arow : (OFF)0;
            ++next;
        }
#pragma unroll
        for (int j = 0; j < N; ++j) unpack_row<DT, CL, CX>(w[j], &x[j * CX]);
        pre.template apply<N * CX * V>(k, x, d);
#pragma unroll
        for (int j = 0; j < N; ++j) {
#pragma unroll
            for (int i = 0; i < CX * V; ++i) y[slot + j][i] = x[j * CX * V + i];
            if (!(inside && ok[j])) {
#pragma unroll
                for (int i = 0; i < CX * V; ++i) {
                    const int32_t c = x0 + i / V;
                    y[slot + j][i] = ok[j] && c >= 0 && c < k.W ? y[slot + j][i] : 0.0f;
                }
            }
#pragma unroll
            for (int i = 0; i < Q * V; ++i) T[tslot + j][i] = d[(j * CX + 4) * V + i];
        }
    };
    // times the divisors' reciprocals of the average's windows around N cells of row `row`, from column `col` on (outside the
    // plane: any).  A strip whose windows all lie inside the plane has one divisor: no division per cell.
    auto scale = [&](auto n_tag, int32_t row, int32_t col, float *v) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value;
        if (INC || k.pool.count_include_pad == 1 || (inside && row >= 1 && row < k.H - 1)) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] *= k.pool.inv_kk;
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] *= bwd_avg_inv(k.pool, k.H, k.W, row, min(max(col + i / V, 0), k.W - 1));
        }
    };
    // row `row` of the average's output from three rows of y -> row maxima of the windows (outside the plane: -infinity),
    // scanned as window row DH
    auto average_row = [&](const float (&ya)[CX * V], const float (&yb)[CX * V], const float (&yc)[CX * V], auto dh_tag, int mslot, int32_t row) __attribute__((always_inline)) {
        float a[CA * V];
#pragma unroll
        for (int i = 0; i < CA * V; ++i) {
            // a list that ends in a ReLU has no -0, so the sum may start with the first cell instead of +0
            float sum = ends_in_relu(PRE) ? ya[i] : 0.0f + ya[i];
            sum = sum + ya[i + V];
            sum = sum + ya[i + 2 * V];
#pragma unroll
            for (int dw = 0; dw < 3; ++dw) sum = sum + yb[i + dw * V];
#pragma unroll
            for (int dw = 0; dw < 3; ++dw) sum = sum + yc[i + dw * V];
            a[i] = sum;
        }
        scale(std::integral_constant<int, CA * V>{}, row, L.q0 - 3, a);
        const bool ok = row >= 0 && row < k.H;
        if constexpr (KEYS) {
            Key key[CA * V];
            column_keys<DT, V, CA>(a, (uint32_t)((2 - decltype(dh_tag)::value) * 16 + 15), key);
            if (!(inside && ok)) {
#pragma unroll
                for (int i = 0; i < CA * V; ++i) {
                    const int32_t c = L.q0 - 3 + i / V;
                    key[i] = Key::choose(ok && c >= 0 && c < k.W, key[i], Key::none());
                }
            }
#pragma unroll
            for (int b = 0; b < NW; ++b) km[mslot][b] = Key::max(Key::max(key[2 * b], key[2 * b + 1]), key[2 * b + 2]);
        }
        if constexpr (!KEYS) {
            round_store_all<DT, CA * V>(a);
            if (!(inside && ok)) {
#pragma unroll
                for (int i = 0; i < CA * V; ++i) {
                    const int32_t c = L.q0 - 3 + i / V;
                    a[i] = ok && c >= 0 && c < k.W ? a[i] : -INFINITY;
                }
            }
            row_maxima<V, 2, NW, CA, decltype(dh_tag)::value, 1, ends_in_relu(PRE), true>(a, lead, m[mslot], code[mslot]);
        }
    };

#pragma unroll
    for (int i = 0; i < CG * V; ++i) gt[0][i] = 0.0f;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int i = 0; i < Q * V; ++i) hs[d][i] = 0.0f;
    // y rows 2 oh - 2 .. 2 oh of the first window row -> average row 2 oh - 1; y rows 2 oh - 1, 2 oh stay
    take_rows(std::integral_constant<int, 3>{}, 1, 0);
    average_row(y[1], y[2], y[3], std::integral_constant<int, 0>{}, 0, oh_first * 2 - 1);
#pragma unroll
    for (int i = 0; i < CX * V; ++i) {
        y[0][i] = y[2][i];
        y[1][i] = y[3][i];
    }

    int32_t oh = oh_first;
    // one window row of the max pooling.  The rows that stay (two of y, one of the average's windows and gradient sums, two of
    // hs) and the new ones change roles from one window row to the next: PAR.
    auto step = [&](auto par) __attribute__((always_inline)) {
        constexpr int PAR = decltype(par)::value, K0 = 2 * PAR, N0 = 2 - K0, R0 = 2 * PAR, R2 = 2 - R0;
        const int32_t hA = oh * 2 - 1;  // average rows hA .. hA + 2 under this window row
        const bool row_ok = oh >= 0 && oh < k.Ho;
        float g[NW * V];
        uint32_t gw[row_words<DT, CL, NW>()];
        load_row<DT, CL, NW, OFF>(k, 1, 44, k.g_out, gat, gcol, ow0, g_fits, g_last, gw);
        gat += oh >= 0 && oh < k.Ho - 1 ? grow : (OFF)0;
        take_rows(std::integral_constant<int, 2>{}, N0, 3);
        average_row(y[K0], y[K0 + 1], y[N0], std::integral_constant<int, 1>{}, 1, hA + 1);
        average_row(y[K0 + 1], y[N0], y[N0 + 1], std::integral_constant<int, 2>{}, R2, hA + 2);
        unpack_row<DT, CL, NW>(gw, g);
        float best[NW * V];
        int32_t pick[NW * V];
        if constexpr (KEYS) {
#pragma unroll
            for (int i = 0; i < NW * V; ++i) {
                const Key key = Key::max(Key::max(km[R0][i], km[1][i]), km[R2][i]);
                best[i] = key.value();
                pick[i] = (int32_t)key.code();
            }
        } else {
            combine_rows<NW * V, true>(m[R0], code[R0], m[1], code[1], m[R2], code[R2], hA < 0, best, pick);
        }
#pragma unroll
        for (int i = 0; i < NW * V; ++i) g[i] = row_ok && win[i / V] ? g[i] : 0.0f;  // windows that do not exist give nothing
        if constexpr (POST != 0) {
            float tp[NW * V];
            post.template apply<NW * V>(k, best, tp);
#pragma unroll
            for (int i = 0; i < NW * V; ++i) g[i] *= tp[i];
        }
        scatter<V, 2, NW, -2, CG, 1, KEYS>(pick, g, gt[R0], gt[1], gt[R2]);  // gt's columns begin at q0 - 1
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int32_t row = min(max(hA + d, 0), k.H - 1);  // rows and columns outside the plane hold zeros
            float w[CG * V];
#pragma unroll
            for (int i = 0; i < CG * V; ++i) w[i] = gt[d == 0 ? R0 : 1][i];
            scale(std::integral_constant<int, CG * V>{}, row, L.q0 - 1, w);
#pragma unroll
            for (int i = 0; i < Q * V; ++i) hs[N0 + d][i] = (w[i] + w[i + V]) + w[i + 2 * V];
        }
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int32_t row = hA - 1 + d;
            if (L.live && row >= r_lo && row < r_hi) {
                float v[Q * V];
#pragma unroll
                for (int i = 0; i < Q * V; ++i)
                    v[i] = (d == 0 ? (hs[K0][i] + hs[K0 + 1][i]) + hs[N0][i] : (hs[K0 + 1][i] + hs[N0][i]) + hs[N0 + 1][i]) * T[d][i];
                if constexpr (DT == DT_F16) {  // two roundings, as in round_store: merged with its conversion, a strip's last column alone was rounded once, so gradients depended on Q
#pragma unroll
                    for (int i = 0; i < Q * V; ++i) asm("" : "+v"(v[i]));
                }
                store_row<DT, CL, Q, OFF>(k, 45, iat, L.q0, k.W, pi, whole, v);
                iat += irow;
            }
        }
        // the last row is the next window row's first (a row above the plane has no cells: its keys stay below every cell's, a value of 0 among them)
        const uint32_t up = hA + 2 >= 0 ? 32u : 0u;
#pragma unroll
        for (int i = 0; i < NW * V; ++i) {
            if constexpr (KEYS) km[R2][i] = km[R2][i].bumped(up);
            else code[R2][i] -= 6;
        }
#pragma unroll
        for (int i = 0; i < Q * V; ++i) {
            T[0][i] = T[2][i];
            T[1][i] = T[3][i];
            T[2][i] = T[4][i];
        }
        ++oh;
    };
    const int32_t oh_end = oh_first + k.rc + 2;  // window rows rc * chunk - 1 .. rc * (chunk + 1): as many for every lane
    for (;;) {
        step(std::integral_constant<int, 0>{});
        if (oh == oh_end) break;
        step(std::integral_constant<int, 1>{});
        if (oh == oh_end) break;
    }
}

#include "bs_backward_keys.h"

template <int DT, bool CL, int S, int P>
void launch1(const BwdK &k, bool wide, int32_t pre, dim3 g, hipStream_t st)
{
    constexpr int Q = K_BWD_STRIP_Q;
    if (wide) bwd_strip_kernel<DT, CL, Q, S, P, -1, -1, uint64_t><<<g, 256, 0, st>>>(k);
    else if (pre == 0 && strip_list_code(k.ew + k.n_ew, k.n_post) == BN_RELU)  // the stacked pooling blocks
        bwd_strip_kernel<DT, CL, Q, S, P, 0, BN_RELU, uint32_t><<<g, 256, 0, st>>>(k);
    else if (pre == 0 && k.n_post == 0) bwd_strip_kernel<DT, CL, Q, S, P, 0, 0, uint32_t><<<g, 256, 0, st>>>(k);
    else if (k.n_post == 0) bwd_strip_kernel<DT, CL, Q, S, P, -1, 0, uint32_t><<<g, 256, 0, st>>>(k);
    else bwd_strip_kernel<DT, CL, Q, S, P, -1, -1, uint32_t><<<g, 256, 0, st>>>(k);
}

template <int DT, bool CL, int Q>
void launch2_compiled(const BwdK &k, bool wide, dim3 g, hipStream_t st)
{
    if (wide) bwd_strip2_kernel<DT, CL, Q, true, BN_RELU, BN_RELU, uint64_t><<<g, 256, 0, st>>>(k);
    else bwd_strip2_kernel<DT, CL, Q, true, BN_RELU, BN_RELU, uint32_t><<<g, 256, 0, st>>>(k);
}

template <int DT, bool CL>
void launch2(const BwdK &k, bool wide, bool compiled, dim3 g, hipStream_t st)
{
    constexpr int Q = bwd_strip2_columns(CL, DT, true), QR = bwd_strip2_columns(CL, DT, false);
    if (compiled && k.strips == Q) launch2_compiled<DT, CL, Q>(k, wide, g, st);
    else if (compiled) launch2_compiled<DT, CL, 4>(k, wide, g, st);
    else if (wide) bwd_strip2_kernel<DT, CL, QR, false, -1, -1, uint64_t><<<g, 256, 0, st>>>(k);
    else bwd_strip2_kernel<DT, CL, QR, false, -1, -1, uint32_t><<<g, 256, 0, st>>>(k);
}

}  // namespace

int32_t bwd_strip_channels(const BwdK &k, bool nhwc, int32_t dtype)
{
    return bwd_strip_keys(k) && nhwc && dtype != BS_F32 && k.C % 2 == 0 ? 2 : 1;
}

bool bwd_strip_keys(const BwdK &k) { return k.wave_rows != 2 && k.n_post == 0 && strip_list_code(k.ew, k.n_ew) == BN_RELU; }

bool bwd_strip_compiled(const BwdK &k)
{
    const int32_t pre = strip_list_code(k.ew, k.n_ew);
    return k.n_post == 0 && (pre == BN_RELU || pre == 0);
}

bool bwd_strip2_compiled(const BwdK &k)
{
    return k.pool.count_include_pad == 1 && strip_list_code(k.ew, k.n_ew) == BN_RELU && strip_list_code(k.ew + k.n_ew, k.n_post) == BN_RELU;
}

bs_status launch_backward_strips(const BwdK &arg, int32_t dtype, int32_t vec, int64_t grid, int32_t threads, void *stream)
{
    BwdK k = arg;
    const PoolK &p = k.pool, &q = k.pool2;
    const bool two = k.wave_rows == 2, nhwc = k.nhwc != 0;
    const bool compiled = two && bwd_strip2_compiled(k);
    const int32_t s = two ? 2 : p.sh, Q = k.strips;
    if (Q != (two ? bwd_strip2_columns(nhwc, dtype, compiled) : K_BWD_STRIP_Q) && !(Q == 2 && bwd_strip_keys(k)) && !(Q == 4 && two)) return BS_ERR_UNSUPPORTED;
    // what the kernels assume: no Add; 3 x 3 windows; strips and chunks that cover the plane; the divisors of the lane numbering
    if (k.n_ew < 0 || k.n_post < 0 || k.n_ew + k.n_post > K_BWD_EW || threads != 256 || grid < 1) return BS_ERR_UNSUPPORTED;
    for (int32_t j = 0; j < k.n_ew + k.n_post; ++j)
        if (k.ew[j].kind == OP_ADD) return BS_ERR_UNSUPPORTED;
    const PoolK &mx = two ? q : p;
    if (k.direct || vec != bwd_strip_channels(k, nhwc, dtype) || mx.kind != OP_MAXPOOL || mx.kh != 3 || mx.kw != 3 || mx.sh != mx.sw || mx.ph != mx.pw ||
        mx.ph < 0 || mx.ph > 1 || (mx.sh != 1 && mx.sh != 2) || (int64_t)(nhwc ? k.div_wv.d * (uint32_t)vec : k.div_c.d) != k.C || (int64_t)k.div_cbs.d != k.cbs ||
        (int64_t)k.div_chunks.d != k.chunks || k.cbs != (k.W + Q - 1) / Q || k.rc < 1 || k.chunks < 1 ||
        (int64_t)k.chunks * k.rc * s < k.H || k.total % ((uint64_t)k.cbs * k.chunks * (k.C / vec)) != 0 ||
        (uint64_t)grid * 256 < k.total || k.Ho < 1 || k.Wo < 1)
        return BS_ERR_UNSUPPORTED;
    if (two && (p.kind != OP_AVGSUM || p.kh != 3 || p.kw != 3 || p.sh != 1 || p.sw != 1 || p.ph != 1 || p.pw != 1 || mx.sh != 2 || mx.ph != 1))
        return BS_ERR_UNSUPPORTED;
    // elements from the first to the last one of each tensor; 32-bit byte offsets where they all end below 4 GiB
    const uint64_t images = k.total / ((uint64_t)k.cbs * k.chunks * (k.C / vec)), es = dtype == BS_F32 ? 4 : 2;
    auto reach = [&](uint64_t pixels, uint64_t extra) { return nhwc ? images * pixels * (k.C + extra) : images * pixels * k.C + (images - 1) * extra; };
    const uint64_t in_px = (uint64_t)k.H * k.W, out_px = (uint64_t)k.Ho * k.Wo;
    k.a_bytes = reach(in_px, k.a_extra) * es;
    k.g_bytes = reach(out_px, k.gout_extra) * es;
    const bool wide = std::max(std::max(k.a_bytes, k.g_bytes), reach(in_px, k.gin_extra) * es) > 0xffffffffull;
    const int32_t pre = strip_list_code(k.ew, k.n_ew);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 g((uint32_t)grid);
#define BS_STRIPS_CL(DT, CL)                                                       \
    do {                                                                           \
        if (two) launch2<DT, CL>(k, wide, compiled, g, st);                       \
        else if (p.sh == 2 && p.ph == 1) launch1<DT, CL, 2, 1>(k, wide, pre, g, st); \
        else if (p.sh == 2) launch1<DT, CL, 2, 0>(k, wide, pre, g, st);            \
        else if (p.ph == 1) launch1<DT, CL, 1, 1>(k, wide, pre, g, st);            \
        else launch1<DT, CL, 1, 0>(k, wide, pre, g, st);                           \
    } while (0)
#define BS_STRIPS(DT)                                                              \
    do {                                                                           \
        if (nhwc) BS_STRIPS_CL(DT, true);                                          \
        else BS_STRIPS_CL(DT, false);                                              \
    } while (0)
    if (dtype != BS_F32 && dtype != BS_BF16 && dtype != BS_F16) return BS_ERR_UNSUPPORTED;
    if (bwd_strip_keys(k)) launch_keys(k, dtype, vec, wide, g, st);
    else if (dtype == BS_F32) BS_STRIPS(DT_F32);
    else if (dtype == BS_BF16) BS_STRIPS(DT_BF16);
    else BS_STRIPS(DT_F16);
#undef BS_STRIPS
#undef BS_STRIPS_CL
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_hip_error((int32_t)e);
        return BS_ERR_HIP;
    }
    return BS_OK;
}

}  // namespace bs
