// bwd_keys_kernel: the backward pass of [BatchNorm -> ReLU or ReLU, max pooling 3 x 3 with stride S = 1 or 2 and padding P = 0 or 1] (the
// ResNet and Inception stems, the pools of SqueezeNet and AlexNet) as strips of columns, for any width and channel count.
//
// The walk is bwd_strip_kernel's: a lane owns Q columns (of V channels) and goes down a chunk of rows; per window row it reads S new input
// rows and one row of upstream gradients, adds the windows' gradients to the picked cells and writes the S rows no later window reaches.
// Behind a ReLU no value is negative, so value and place of a cell are one word that orders like the pair (PickKey): a window's pick is
// a maximum of keys, a ReLU's derivative at the pick is "the maximum is above zero" (once per window instead of once per cell), and the
// BatchNorm's derivative is one factor of the finished sum.  16-bit storage, channels-last: two channels per lane where their number is
// even -- half the addresses and requests.
// What bounds it: memory -- 231 MB of the ResNet stem 64 x 64 x 112 x 112 bfloat16 in 46 us = 5.0 TB/s (269 MB with what is fetched twice; 26 vector
// instructions per cell take 29 of the 46 us; the kernel that compares and selects: 60 us, 36 instructions); float32 94 us = 4.9 TB/s (98).  32 x 192 x 71 x 71 / 2 without padding binary16 38 -> 35 us.  Row-major rows that are no whole
// vectors, 64 x 64 x 111 x 111: float32 145 -> 143, bfloat16 78 -> 76.5.  Strips of 8 columns measured 5 % slower, 2 10 % (large tensors).
// Part of bs_backward_strip.hip (its lanes, places, loads and stores).
#pragma once

// keys of N columns x V channels behind BatchNorm and ReLU
template <int DT, int V, int N>
BS_DEV void strip_keys(const float (&x)[N * V], const float (&a)[V], const float (&b)[V], uint32_t first_code, PickKey<DT> (&key)[N * V])
{
    float y[N * V];
#pragma unroll
    for (int i = 0; i < N * V; ++i) y[i] = __builtin_fmaxf(__builtin_fmaf(x[i], a[i % V], b[i % V]), 0.0f);  // (rounding keeps sign and zero)
    column_keys<DT, V, N>(y, first_code, key);
}

template <int DT, bool CL, int V, int Q, int S, int P, typename OFF>
__global__ __launch_bounds__(256) void bwd_keys_kernel(const BwdK k)
{
    static_assert(Q % S == 0 && (S == 1 || S == 2) && (P == 0 || P == 1), "compiled windows");
    static_assert(V == 1 || (CL && DT != DT_F32 && V == 2), "channels per lane");
    using Key = PickKey<DT>;
    constexpr int OW0 = -((2 - P) / S);            // first window over the strip: q0 / S + OW0 = ceil((q0 + P - 2) / S)
    constexpr int NW = (Q + 1) / S + 1;            // windows over the strip
    constexpr int X0 = OW0 * S - P;                // their first column, from q0
    constexpr int CW = (NW - 1) * S + 3;           // their columns
    constexpr int KEEP = 3 - S, ES = elem_bytes<DT>();
    constexpr int OEND = (P + S - 1) / S;
    static_assert(CW <= 15, "a code holds four bits of column");
    const StripLane L = strip_lane<CL, Q, V>(k);
    const StripPlaces<DT, CL, OFF> at0(k, L);
    const OFF pa = at0.pa, pg = at0.pg, pi = at0.pi, arow = at0.arow, grow = at0.grow, irow = at0.irow;

    const int32_t x0 = L.q0 + X0, ow0 = L.q0 / S + OW0;
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

    HeldParams<V> bn;
    if (k.n_ew == 1) bn.identity();  // ReLU alone
    else bn.load(k.params, OP_BN, k.ew[0].arg, L.c0, k.C);

    const int32_t r_lo = L.chunk * k.rc * S, r_hi = min(r_lo + k.rc * S, k.H);  // rows this chunk writes
    const int32_t oh_first = L.chunk * k.rc + OW0;
    Key m[3][NW * V];
    float s[3][Q * V];
    // rows are requested in order, `at` = the offset of row `next` (clamped to the plane)
    int32_t next = oh_first * S - P, oh_next = oh_first;
    OFF at = at0.abase + (OFF)min(max(next, 0), k.H - 1) * arow;
    OFF gat = at0.gbase + (OFF)min(max(oh_first, 0), k.Ho - 1) * grow;
    OFF iat = at0.ibase + (OFF)r_lo * irow;
    struct Rows {
        uint32_t w[S][row_words<DT, CL, CW>()];
        bool ok[S];
    };
    auto request = [&](auto n_tag, Rows &r) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < decltype(n_tag)::value; ++j) {
            r.ok[j] = next >= 0 && next < k.H;
            load_row<DT, CL, CW, OFF, V>(k, 0, 46, k.a, at, acol, x0, a_fits, a_last, r.w[j]);
            at += next >= 0 && next < k.H - 1 ? arow : (OFF)0;
            ++next;
        }
    };
    uint32_t gw[row_words<DT, CL, NW>()];
    bool g_ok;
    auto request_g = [&]() __attribute__((always_inline)) {
        g_ok = oh_next >= 0 && oh_next < k.Ho;
        load_row<DT, CL, NW, OFF, V>(k, 1, 47, k.g_out, gat, gcol, ow0, g_fits, g_last, gw);
        gat += oh_next >= 0 && oh_next < k.Ho - 1 ? grow : (OFF)0;
        ++oh_next;
    };
    // requested rows -> row maxima of the windows, as window rows DH0, DH0 + 1 ...: code (2 - window row) * 16 + 15 - column
    auto settle = [&](auto n_tag, auto dh_tag, const Rows &r, auto slot_of) __attribute__((always_inline)) {
        constexpr int N = decltype(n_tag)::value, DH0 = decltype(dh_tag)::value;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            float x[CW * V];
            Key key[CW * V];
            unpack_row<DT, CL, CW, V>(r.w[j], x);
            strip_keys<DT, V, CW>(x, bn.a, bn.b, (uint32_t)((2 - (DH0 + j)) * 16 + 15), key);
            if (!(inside && r.ok[j])) {
#pragma unroll
                for (int i = 0; i < CW * V; ++i) {
                    const int32_t c = x0 + i / V;
                    key[i] = Key::choose(r.ok[j] && c >= 0 && c < k.W, key[i], Key::none());
                }
            }
#pragma unroll
            for (int i = 0; i < NW * V; ++i) {
                const int f = (i / V) * S * V + i % V;
                m[slot_of(j)][i] = Key::max(Key::max(key[f], key[f + V]), key[f + 2 * V]);
            }
        }
    };
    Rows rows;
    if constexpr (KEEP > 0) {
        Rows lead[(KEEP + S - 1) / S];
#pragma unroll
        for (int j = 0; j < KEEP; j += S) request(std::integral_constant<int, 1>{}, lead[j / S]);
        // (stride 1: one row per request)
        each_of(std::make_integer_sequence<int, KEEP>{}, [&](auto j_tag) __attribute__((always_inline)) {
            constexpr int J = decltype(j_tag)::value;
            settle(std::integral_constant<int, 1>{}, j_tag, lead[J / S], [](int) { return J; });
        });
#pragma unroll
        for (int d = 0; d < KEEP; ++d)
#pragma unroll
            for (int i = 0; i < Q * V; ++i) s[d][i] = 0.0f;
    }
    // A window row's operands are requested one window row ahead; row-major, where a run of columns is requested under a condition (the
    // tensor's ends), with the row itself (float32 64 x 64 x 111 x 111: 152 us ahead, 143 with the row).
    constexpr bool AHEAD = CL;
    if constexpr (AHEAD) {
        request_g();
        request(std::integral_constant<int, S>{}, rows);
    }

    int32_t oh = oh_first;
    // one window row; its three rows are in ring slots R0 (stride 2: two rows are new, the third's slot and the first's change
    // roles from one window row to the next; stride 1: the rows move up)
    auto step = [&](auto par) __attribute__((always_inline)) {
        constexpr int R0 = decltype(par)::value ? 2 : 0, R2 = 2 - R0;
        const int32_t hA = oh * S - P;
        float g[NW * V];
        if constexpr (!AHEAD) {
            request_g();
            request(std::integral_constant<int, S>{}, rows);
        }
        unpack_row<DT, CL, NW, V>(gw, g);
        const bool row_ok = g_ok;
        settle(std::integral_constant<int, S>{}, std::integral_constant<int, KEEP>{}, rows, [](int j) { return KEEP + j == 2 ? R2 : KEEP + j; });
        if constexpr (AHEAD) {
            request_g();
            request(std::integral_constant<int, S>{}, rows);
        }
        int32_t pick[NW * V];
#pragma unroll
        for (int i = 0; i < NW * V; ++i) {
            const Key best = Key::max(Key::max(m[R0][i], m[1][i]), m[R2][i]);
            pick[i] = (int32_t)best.code();
            // windows that do not exist, and those whose maximum the ReLU has cut off, give nothing
            g[i] = row_ok && win[i / V] && best.positive() ? g[i] : 0.0f;
        }
        // sum[window row][column] += the gradients of the windows that picked the cell, left windows first; rows KEEP .. hold nothing yet
        auto scatter_row = [&](auto dh_tag, float (&sum)[Q * V]) __attribute__((always_inline)) {
            constexpr int dh = decltype(dh_tag)::value;
#pragma unroll
            for (int b = 0; b < NW; ++b)
#pragma unroll
                for (int dw = 0; dw < 3; ++dw) {
                    const int col = X0 + b * S + dw, b0 = col - 2 - X0 <= 0 ? 0 : (col - 2 - X0 + S - 1) / S;
                    if (col >= 0 && col < Q) {
#pragma unroll
                        for (int e = 0; e < V; ++e) {
                            const float t = pick[b * V + e] == (2 - dh) * 16 + 15 - (b * S + dw) ? g[b * V + e] : 0.0f;
                            sum[col * V + e] = dh >= KEEP && b == b0 ? t : sum[col * V + e] + t;
                        }
                    }
                }
        };
        scatter_row(std::integral_constant<int, 0>{}, s[R0]);
        scatter_row(std::integral_constant<int, 1>{}, s[1]);
        scatter_row(std::integral_constant<int, 2>{}, s[R2]);
        // the S rows no later window row holds are complete
#pragma unroll
        for (int d = 0; d < S; ++d) {
            const int32_t row = hA + d;
            const int slot = d == 0 ? R0 : 1;
            if (L.live && row >= r_lo && row < r_hi) {
                float v[Q * V];
#pragma unroll
                for (int i = 0; i < Q * V; ++i) v[i] = s[slot][i] * bn.a[i % V];
                store_row<DT, CL, Q, OFF, V>(k, 48, iat, L.q0, k.W, pi, whole, v);
                iat += irow;
            }
        }
        if constexpr (S == 2) {
#pragma unroll
            for (int i = 0; i < NW * V; ++i) m[R2][i] = m[R2][i].bumped(32u);
        } else {
#pragma unroll
            for (int d = 0; d < KEEP; ++d) {
#pragma unroll
                for (int i = 0; i < NW * V; ++i) m[d][i] = m[d + 1][i].bumped(16u);
#pragma unroll
                for (int i = 0; i < Q * V; ++i) s[d][i] = s[d + 1][i];
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

template <int DT, bool CL, int V, int Q>
void launch_keys_windows(const BwdK &k, bool wide, dim3 g, hipStream_t st)
{
#define BS_KEYS(S, P)                                                              \
    do {                                                                           \
        if (wide) bwd_keys_kernel<DT, CL, V, Q, S, P, uint64_t><<<g, 256, 0, st>>>(k); \
        else bwd_keys_kernel<DT, CL, V, Q, S, P, uint32_t><<<g, 256, 0, st>>>(k);  \
    } while (0)
    if (k.pool.sh == 2 && k.pool.ph == 1) BS_KEYS(2, 1);
    else if (k.pool.sh == 2) BS_KEYS(2, 0);
    else if (k.pool.ph == 1) BS_KEYS(1, 1);
    else BS_KEYS(1, 0);
#undef BS_KEYS
}

template <int DT, bool CL, int V>
void launch_keys_columns(const BwdK &k, bool wide, dim3 g, hipStream_t st)
{
    if (k.strips == 2) launch_keys_windows<DT, CL, V, 2>(k, wide, g, st);
    else launch_keys_windows<DT, CL, V, K_BWD_STRIP_Q>(k, wide, g, st);
}

// (launch_backward_strips has checked the arguments; vec: channels per lane)
void launch_keys(const BwdK &k, int32_t dtype, int32_t vec, bool wide, dim3 g, hipStream_t st)
{
    if (!k.nhwc) {
        if (dtype == BS_F32) launch_keys_columns<DT_F32, false, 1>(k, wide, g, st);
        else if (dtype == BS_BF16) launch_keys_columns<DT_BF16, false, 1>(k, wide, g, st);
        else launch_keys_columns<DT_F16, false, 1>(k, wide, g, st);
    } else if (dtype == BS_F32) {
        launch_keys_columns<DT_F32, true, 1>(k, wide, g, st);
    } else if (vec == 2) {
        if (dtype == BS_BF16) launch_keys_columns<DT_BF16, true, 2>(k, wide, g, st);
        else launch_keys_columns<DT_F16, true, 2>(k, wide, g, st);
    } else {
        if (dtype == BS_BF16) launch_keys_columns<DT_BF16, true, 1>(k, wide, g, st);
        else launch_keys_columns<DT_F16, true, 1>(k, wide, g, st);
    }
}
