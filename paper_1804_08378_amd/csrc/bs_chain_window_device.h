// chain_window_kernel: the blocks <max pooling 3 x 3 / 1 / 1, BatchNorm, ReLU> of pool_chain_kernel where every BatchNorm but the last has
// scales above zero -- one window instead of L of them.
//
// A BatchNorm with a positive scale, a ReLU and the rounding to the storage type never decrease when their input increases (the rounded
// fused multiply-add is monotone), so each commutes with the maximum of the next level, and L stacked 3 x 3 maxima are one maximum over
// (2 L + 1) x (2 L + 1) cells (cells outside the plane are in neither).  The lists of all levels then run once, on the window's maximum.  The
// ReLUs commute with what stands behind them as well: f(max(a, 0)) = max(f(a), f(0)), so a cell goes through the bare multiply-adds of levels 1 .. L - 1 and
// meets one maximum with C in front of the last.  C is the least that level 1's ReLU lets through, 0, behind levels 2 .. L - 1 (0 with two levels): the first BatchNorm
// stands in front of that ReLU and has no part in it.  The same bits as level by level, also for windows without a cell above zero, for infinities and for NaN (left out by a
// maximum; behind a ReLU zero): 1 instruction per cell and level in float32 instead of 3.5, and no level recomputes its rows and columns.
//
// A work-group takes ppg whole planes or a band of rows of one.  (1) A lane takes the window maxima down four columns for QV rows: maxima of the
// run's first cells from below, of its last ones from above and of the cells that all windows share; the rows, those around its own among them,
// are vector loads that the lanes of the neighbouring runs find in the cache.  (2) Through LDS, with one barrier, a lane does the same along Q
// columns of a row, applies the lists and stores.  Values are float32 from the loads on.
// What bounds it: vector instructions and LDS together (8.0 M vector instructions are 54 % of the time at 3.5 cycles each, LDS 62 % of the compute units' cycles), in float32 beside
// memory; with 16-bit storage the lists: 2.5 instructions a cell and level in bfloat16, 1.5 in binary16.  Ten levels 64 x 64 x 56 x 56 float32, level by level -> window, us: three
// tensors in turn (partly in the last cache) 27.5 .. 32.0 -> 20.0 .. 21.0 from one run of the machine to the next, eight in turn (from memory) 31.4 -> 30.4; bfloat16 31.6 -> 22.2, 31.7 -> 22.0.
// Tried: rows staged in LDS first (31.8: two more barriers and round trips), sixteen rows a lane (26 .. 30: half the lanes), packed 16-bit integers of the
// same order for 16-bit storage (nine instructions a pair to convert there and back), eight columns a lane (float32 stores 32 bytes apart).
#pragma once
#include "bs_device.h"

namespace bs {

// Rows and columns a lane takes the maxima of: it reads 2 levels more.
constexpr int K_WINDOW_ROWS = 8, K_WINDOW_COLUMNS = 4;
constexpr int window_pad(int levels) { return (levels + 3) / 4 * 4; }  // columns of LDS between two rows: whole 128-bit reads

// y[i] = maximum of x[i] .. x[i + 2 L], i < Q; x(i, v) gives V values beside each other, y(i, v) takes them.
template <int L, int Q, int V, typename X, typename Y>
BS_DEV void slide_max(X x, Y y)
{
    constexpr int N = 2 * L + 1;
    if constexpr (N >= Q) {
        // the run's first cells from the right, the cells that all windows share, its last ones from the left
        float s[Q - 1][V], core[V], p[V], out[V];
#pragma unroll
        for (int i = 0; i + 1 < Q; ++i) x(i, s[i]);
        x(Q - 1, core);
#pragma unroll
        for (int i = Q; i < N; i += 2) {
            float a[V], b[V];
            x(i, a);
            if (i + 1 < N) x(i + 1, b);
#pragma unroll
            for (int e = 0; e < V; ++e) core[e] = i + 1 < N ? max3(core[e], a[e], b[e]) : max2(core[e], a[e]);
        }
#pragma unroll
        for (int i = Q - 3; i >= 0; --i)
#pragma unroll
            for (int e = 0; e < V; ++e) s[i][e] = max2(s[i][e], s[i + 1][e]);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            if (i > 0) {
                float a[V];
                x(N - 1 + i, a);
#pragma unroll
                for (int e = 0; e < V; ++e) p[e] = i == 1 ? a[e] : max2(p[e], a[e]);
            }
#pragma unroll
            for (int e = 0; e < V; ++e) out[e] = i == 0 ? max2(s[0][e], core[e]) : i + 1 < Q ? max3(s[i][e], core[e], p[e]) : max2(core[e], p[e]);
            y(i, out);
        }
    } else {  // five or seven: threes
        float t[Q + 2 * L][V];
#pragma unroll
        for (int i = 0; i < Q + 2 * L; ++i) x(i, t[i]);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            float out[V];
#pragma unroll
            for (int e = 0; e < V; ++e) {
                // t[i], t[i + 3] become the maxima of three cells from i, i + 3 on
                if (i == 0) {
#pragma unroll
                    for (int j = 0; j < (N == 5 ? 1 : 4); ++j) t[j][e] = max3(t[j][e], t[j + 1][e], t[j + 2][e]);
                } else if (N == 5) {
                    t[i][e] = max3(t[i][e], t[i + 1][e], t[i + 2][e]);
                } else {
                    t[i + 3][e] = max3(t[i + 3][e], t[i + 4][e], t[i + 5][e]);
                }
                out[e] = N == 5 ? max3(t[i][e], t[i + 3][e], t[i + 4][e]) : max3(t[i][e], t[i + 3][e], t[i + 6][e]);
            }
            y(i, out);
        }
    }
    static_assert(N >= Q || N == 5 || N == 7, "runs of eight and less");
}

// The lists of all levels on Q values: u -> max(bare multiply-adds, zero), the last level's as they stand.
template <int DT, int L, int Q>
BS_DEV void window_lists(float (&u)[Q], const float (&sc)[L], const float (&sh)[L], float zero)
{
#pragma unroll
    for (int l = 0; l < L; ++l) {
        if (l + 1 == L) {  // (L > 1)
#pragma unroll
            for (int e = 0; e < Q; ++e) u[e] = max2(u[e], zero);
        }
#pragma unroll
        for (int e = 0; e < Q; ++e) u[e] = __builtin_fmaf(u[e], sc[l], sh[l]);
        if (l + 1 == L) {
#pragma unroll
            for (int e = 0; e < Q; ++e) u[e] = max2(u[e], 0.0f);
        } else if constexpr (DT == DT_BF16) {
            round_store_all<DT, Q>(u);
        } else if constexpr (DT == DT_F16) {
            // two roundings, as in round_store: no conversion merges with its multiply-add; two values a conversion
            static_assert(Q == 4, "four columns");
            asm("" : "+v"(u[0]), "+v"(u[1]), "+v"(u[2]), "+v"(u[3]));
#pragma unroll
            for (int e = 0; e < Q; e += 2) {
                const uint32_t w = pack2<DT>(u[e], u[e + 1]);
                u[e] = half_up<DT>(w & 0xffffu);
                u[e + 1] = half_up<DT>(w >> 16);
            }
        }
    }
}

BS_DEV void lds_read4(const float *p, float *w)
{
    const float4 v = *reinterpret_cast<const float4 *>(p);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
}

// Four columns, or a row's last ones: REM of them (at any multiple of the element size).
template <int DT, int REM, bool NT>
BS_DEV void store_columns_as(char *at, const float (&u)[4], bool all)
{
    constexpr int ES = DT == DT_F32 ? 4 : 2, NW = DT == DT_F32 ? 4 : 2;
    uint32_t w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        if constexpr (DT == DT_F32) w[i] = __float_as_uint(u[i]);
        else w[i] = pack2<DT>(u[2 * i], u[2 * i + 1]);
    }
    if (REM == 0 || all) {
        store_words<NW, REM == 0 ? 4 * ES : ES, NT>(at, w);
    } else {
        if constexpr (REM & 2) {
            uint32_t head[NW / 2];
#pragma unroll
            for (int i = 0; i < NW / 2; ++i) head[i] = w[i];
            store_words<NW / 2, ES, NT>(at, head);
        }
        if constexpr (REM & 1) {
            const uint32_t last = w[REM & 2 ? NW / 2 : 0];
            char *const to = at + (REM & 2) * ES;
            if constexpr (DT == DT_F32) store_words<1, 4, NT>(to, {last});
            else if constexpr (NT) __builtin_nontemporal_store((uint16_t)last, reinterpret_cast<uint16_t *>(to));
            else *reinterpret_cast<uint16_t *>(to) = (uint16_t)last;
        }
    }
}

// Past the caches unless a later launch of the stack reads them.  Plain / non-temporal, geometric means over 160 drawn sizes, three inputs in turn / eight: outputs up to 4 MB
// 1.00 / 1.01, 4 .. 48 MB 1.05 / 1.06, 48 .. 120 MB 1.13 / 0.98 (three inputs stay in the last cache then, because the outputs do not drive them out).  Where another kernel reads the
// output at once they gain up to 8 MB of float32 (1.03) and cost 1 .. 7 % beyond 24 MB and with 16-bit storage; ten levels 64 x 64 x 56 x 56 float32, us, three inputs 21.9 / 21.0,
// eight 28.1 / 30.6, with a reader 43.5 / 48.1 (level by level 28.5, 31.4, 47.1).  Between the launches of one stack, which always reads them: 16 levels in four launches 93.5 / 107.6, 40 in five
// 113.7 / 137.0.
template <int DT, int REM>
BS_DEV void store_columns(char *at, const float (&u)[4], bool all, bool streamed)
{
    if (streamed) {  // (the same for every lane)
        asm volatile("");  // else the compiler makes one plain store of the two
        store_columns_as<DT, REM, true>(at, u, all);
        asm volatile("");
    } else {
        store_columns_as<DT, REM, false>(at, u, all);
    }
}

// REM: a row's columns beyond whole vectors of four.  With 0 all vectors are aligned; else a row's last vector is read as its last four columns
// and moved to its place.
template <int DT, int L, int REM>
__global__ __launch_bounds__(K_WINDOW_THREADS, 4) void chain_window_kernel(const ChainWindowK k)
{
    static_assert(L >= window_fewest(DT), "fewer levels go level by level");
    constexpr int ES = DT == DT_F32 ? 4 : 2, PAD = window_pad(L), QV = K_WINDOW_ROWS, Q = K_WINDOW_COLUMNS;
    constexpr bool WHOLE = REM == 0;
    extern __shared__ float4 lds_vectors[];
    float *const lds = reinterpret_cast<float *>(lds_vectors);
    quiet_maxima();

    const uint32_t block = xcd_contiguous(blockIdx.x, gridDim.x);
    const uint32_t group = fdiv(block, k.div_chunks);
    const int32_t o0 = (int32_t)(block - group * k.div_chunks.d) * k.rc, here = min(k.rc, k.H - o0);  // output rows
    const uint32_t plane0 = group * (uint32_t)k.ppg;
    const int32_t planes = min(k.ppg, (int32_t)(k.planes - plane0));  // of this work-group
    const int32_t tid = (int32_t)threadIdx.x, threads = (int32_t)blockDim.x;

    // (1) task -> (plane, run of rows, vector).  Offsets from the band's first row fit 32 bits.
    const int32_t tasks = planes * (int32_t)k.div_plane_tasks.d, low = max(o0 - L, 0), high = min(o0 + k.rows + L, k.H) - 1 - low;
    const uint32_t img0 = fdiv(plane0, k.div_c), row_bytes = (uint32_t)k.W * ES, plane_bytes = (uint32_t)k.H * row_bytes;
    const char *const in0 = static_cast<const char *>(image_base<DT>(k.in, img0, k.in_extra)) + (size_t)plane0 * ((size_t)k.H * k.W * ES) + (size_t)(uint32_t)low * row_bytes;
    for (int32_t t = tid; t < tasks; t += threads) {
        int32_t p = 0, in_plane = t;
        uint32_t at = 0;
        if (k.ppg > 1) {
            p = (int32_t)fdiv((uint32_t)t, k.div_plane_tasks);
            in_plane = t - p * (int32_t)k.div_plane_tasks.d;
            at = (uint32_t)p * plane_bytes + (fdiv(plane0 + (uint32_t)p, k.div_c) - img0) * k.in_extra * ES;
        }
        const int32_t slot = (int32_t)fdiv((uint32_t)in_plane, k.div_lanes), v = in_plane - slot * (int32_t)k.div_lanes.d;
        if (v >= k.vecs) continue;
        const int32_t col = WHOLE ? v * 4 : min(v * 4, k.W - 4), top = o0 + slot * QV - L - low;
        at += (uint32_t)col * ES;
        float *const to = lds + (p * k.rows + slot * QV) * k.pitch + PAD + v * 4;
        const bool tail = !WHOLE && col != v * 4;
        slide_max<L, QV, 4>(
            [&](int i, float(&x)[4]) __attribute__((always_inline)) {
                // a row outside the plane: the plane's first or last one, which every window that reaches beyond it holds
                const char *const from = in0 + (at + (uint32_t)min(max(top + i, 0), high) * row_bytes);
                struct __attribute__((packed, aligned(2))) W2 { uint32_t w[2]; };
                struct __attribute__((packed, aligned(4))) W4 { uint32_t w[4]; };
                if constexpr (DT == DT_F32) {
                    uint4 q;
                    if constexpr (WHOLE) {
                        q = *reinterpret_cast<const uint4 *>(from);
                    } else {
                        const W4 w = *reinterpret_cast<const W4 *>(from);
                        q = make_uint4(w.w[0], w.w[1], w.w[2], w.w[3]);
                    }
                    x[0] = __uint_as_float(q.x); x[1] = __uint_as_float(q.y); x[2] = __uint_as_float(q.z); x[3] = __uint_as_float(q.w);
                } else {
                    uint2 q;
                    if constexpr (WHOLE) {
                        q = *reinterpret_cast<const uint2 *>(from);
                    } else {
                        const W2 w = *reinterpret_cast<const W2 *>(from);
                        q = make_uint2(w.w[0], w.w[1]);
                    }
                    if constexpr (DT == DT_BF16) {
                        x[0] = __uint_as_float(q.x << 16); x[1] = __uint_as_float(q.x & 0xffff0000u); x[2] = __uint_as_float(q.y << 16); x[3] = __uint_as_float(q.y & 0xffff0000u);
                    } else {
                        x[0] = half_up<DT>(q.x & 0xffffu); x[1] = half_up<DT>(q.x >> 16); x[2] = half_up<DT>(q.y & 0xffffu); x[3] = half_up<DT>(q.y >> 16);
                    }
                }
            },
            [&](int i, const float(&y)[4]) __attribute__((always_inline)) {
                float m[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) m[e] = WHOLE || !tail ? y[e] : e < REM ? y[(e + 4 - REM) % 4] : -INFINITY;
                *reinterpret_cast<float4 *>(to + i * k.pitch) = make_float4(m[0], m[1], m[2], m[3]);
            });
    }
    // the PAD columns beside a row: those behind it are those in front of the next one
    const int32_t beside = PAD / 4, all_beside = planes * k.rows * beside;
    const float4 outside = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    for (int32_t t = tid; t < all_beside; t += threads) {
        const int32_t g = (int32_t)((uint32_t)t / (uint32_t)beside);
        *reinterpret_cast<float4 *>(lds + (g + 1) * k.pitch + (t - g * beside) * 4) = outside;
    }
    if (tid < beside) *reinterpret_cast<float4 *>(lds + tid * 4) = outside;

    // (2) thread -> (plane, row, run of Q columns).  The levels' parameters are requested in front of the barrier.
    const int32_t p = k.ppg > 1 ? min((int32_t)fdiv((uint32_t)tid, k.div_second), planes - 1) : 0, in_plane = tid - p * (int32_t)k.div_second.d;
    const int32_t r_in = (int32_t)fdiv((uint32_t)in_plane, k.div_lanes), run = in_plane - r_in * (int32_t)k.div_lanes.d, col = run * Q;
    const uint32_t plane = plane0 + (uint32_t)p, img = k.ppg > 1 ? fdiv(plane, k.div_c) : img0, c = plane - img * (uint32_t)k.C;
    float sc[L], sh[L], zero = 0.0f;
#pragma unroll
    for (int l = 0; l < L; ++l) {
        sc[l] = k.params[k.bn[l] + c];
        sh[l] = k.params[k.bn[l] + k.C + c];
    }
    __syncthreads();
    if (r_in >= k.row_slots || run >= k.vecs) return;
    // what the levels behind the first ReLU make of its 0
#pragma unroll
    for (int l = 1; l + 1 < L; ++l) zero = __builtin_fmaxf(round_store<DT>(__builtin_fmaf(zero, sc[l], sh[l])), 0.0f);
    char *const outp = static_cast<char *>(image_base<DT>(k.out, img, k.out_extra)) + ((size_t)plane * k.H + (size_t)(uint32_t)o0) * row_bytes + (uint32_t)col * ES;
    for (int32_t row = r_in; row < here; row += k.row_slots) {
        const float *const from = lds + (p * k.rows + row) * k.pitch + col;
        float x[Q + 2 * L], u[Q];
#pragma unroll
        for (int i = 0; i < Q + 2 * PAD; i += 4) {
            float w[4];
            lds_read4(from + i, w);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e >= PAD - L && i + e < PAD + Q + L) x[i + e - (PAD - L)] = w[e];
        }
        slide_max<L, Q, 1>([&](int i, float(&v)[1]) __attribute__((always_inline)) { v[0] = x[i]; },
                           [&](int i, const float(&v)[1]) __attribute__((always_inline)) { u[i] = v[0]; });
        window_lists<DT, L, Q>(u, sc, sh, zero);
        store_columns<DT, REM>(outp + (uint32_t)row * row_bytes, u, col + 4 <= k.W, k.streamed != 0);
    }
}

}  // namespace bs
