// chain_window_nhwc_kernel: chain_window_kernel's blocks (one window of (2 L + 1) x (2 L + 1) cells, the lists of all levels behind it) channels-last.
//
// A lane takes the window maxima down eight rows of one column and four consecutive channels; its vector loads are contiguous over the lanes' channels.
// Four rows at a time go through LDS, [row][column][channel], where a lane does the same along four columns, applies the lists and stores.  The
// rest of the eight rows' state stays in registers meanwhile, so LDS holds four rows only.  A row is asked of the caches (8 + 2 L) / 8 times.
// Against level by level over drawn sizes, geometric means: vectors of four channels float32 1.34 (396 sizes, 0.82 .. 2.8), 16-bit storage 1.38 (270, 0.90 .. 2.3), one channel a lane
// float32 1.84 (201, 0.88 .. 3.3), 16-bit 1.62 (320, 0.77 .. 7.6: slower only on large tensors with four to six levels).
// What bounds it: vector instructions (the lists; in float32 as many for the windows) and the LDS round trips between its two passes.  Ten levels bfloat16
// 3 x 240 x 102 x 102 24.9 us (1.2 TB/s), float32 3 x 432 x 137 x 137 87.9 (2.2 TB/s).
#include <algorithm>

#include "bs_chain_window_device.h"
#include "bs_internal.h"

namespace bs {
namespace {

constexpr int K_ROWS = 8, K_STEP = 4, K_Q = 4, K_THREADS = 512;

template <int DT, int V>
BS_DEV void load_pixel(const char *p, float (&x)[V])
{
    Raw<DT, V> r;
    r.q = *reinterpret_cast<const typename Raw<DT, V>::type *>(p);
    unpack<DT, V>(r, x);
}

template <int DT, int V, int L>
__global__ __launch_bounds__(K_THREADS, 4) void chain_window_nhwc_kernel(const ChainWindowNhwcK k)
{
    constexpr uint32_t ES = DT == DT_F32 ? 4 : 2;
    extern __shared__ float4 lds_vectors[];
    float *const lds = reinterpret_cast<float *>(lds_vectors);
    quiet_maxima();

    // work-group -> (image, band, column tile, channel group), the last one fastest: groups that share cache lines, bands that share rows on one XCD
    uint32_t b = xcd_contiguous(blockIdx.x, gridDim.x), a = fdiv(b, k.div_groups);
    const int32_t c0 = (int32_t)(b - a * k.div_groups.d) * k.lanes * V;
    b = fdiv(a, k.div_tiles);
    const int32_t w0 = (int32_t)(a - b * k.div_tiles.d) * k.tile_w;
    const uint32_t img = fdiv(b, k.div_bands);
    const int32_t o0 = (int32_t)(b - img * k.div_bands.d) * K_ROWS;
    const int32_t tid = (int32_t)threadIdx.x, threads = (int32_t)blockDim.x, px = k.lanes * V;  // px: words of a pixel in LDS

    // the thread's column and channels; beyond the plane: its nearest column, which every window that reaches there holds
    const int32_t j = (int32_t)fdiv((uint32_t)tid, k.div_lanes), lane = tid - j * k.lanes;
    const bool single = k.tiles == 1, live = j < k.work;
    const int32_t c = min(c0 + lane * V, k.C - V), x = min(max(single ? j : w0 - L + j, 0), k.W - 1);
    const uint32_t pin = ((uint32_t)k.C + k.in_xp) * ES, pout = ((uint32_t)k.C + k.out_xp) * ES;
    const char *const inp = static_cast<const char *>(k.in) + ((size_t)img * (size_t)(k.H * k.W) + (size_t)x) * pin + (uint32_t)c * ES;
    const size_t in_row = (size_t)(uint32_t)k.W * pin;
    float *const mine = lds + (single ? L + j : j) * px + lane * V;

    // columns of LDS beside a single tile: the lowest value, once
    const int32_t columns = single ? (k.W + 3) / 4 * 4 + 2 * L : k.work;
    if (single) {
        const int32_t left = L * px, right = (columns - L - k.W) * px, all = K_STEP * (left + right);
        for (int32_t t = tid; t < all; t += threads) {
            const int32_t r = t / (left + right), i = t - r * (left + right);
            lds[r * k.row_words + (i < left ? i : k.W * px + i)] = -INFINITY;
        }
    }
    // the levels' scales and shifts of the group's channels, what the levels behind the first ReLU make of its 0
    float *const table = lds + K_STEP * k.row_words;
    if (tid < px) {
        const int32_t ch = min(c0 + tid, k.C - 1);
        float zero = 0.0f;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const float s = k.params[k.bn[l] + ch], h = k.params[k.bn[l] + k.C + ch];
            table[(2 * l) * px + tid] = s;
            table[(2 * l + 1) * px + tid] = h;
            if (l > 0 && l + 1 < L) zero = __builtin_fmaxf(round_store<DT>(__builtin_fmaf(zero, s, h)), 0.0f);
        }
        table[2 * L * px + tid] = zero;
    }

    // four rows from LDS: row r of the band on
    const int32_t runs = (min(k.tile_w, k.W - w0) + K_Q - 1) / K_Q, tasks = runs * K_STEP * k.lanes;
    char *const outp = static_cast<char *>(k.out) + ((size_t)img * (size_t)(k.H * k.W) + (size_t)(uint32_t)w0) * pout + (uint32_t)c0 * ES;
    auto finish = [&](int32_t r) __attribute__((always_inline)) {
        for (int32_t t = tid; t < tasks; t += threads) {
            const int32_t q = (int32_t)fdiv((uint32_t)t, k.div_lanes), ln = t - q * k.lanes, row = q % K_STEP, run = q / K_STEP;
            const int32_t h = o0 + r + row;
            if (h >= k.H || c0 + ln * V >= k.C) continue;
            const float *const from = lds + row * k.row_words + run * K_Q * px + ln * V;
            float u[K_Q * V];
            slide_max<L, K_Q, V>(
                [&](int i, float(&w)[V]) __attribute__((always_inline)) {
                    if constexpr (V == 4) lds_read4(from + i * px, w);
                    else w[0] = from[i * px];
                },
                [&](int i, const float(&w)[V]) __attribute__((always_inline)) {
#pragma unroll
                    for (int e = 0; e < V; ++e) u[i * V + e] = w[e];
                });
            const float *const tab = table + ln * V;
            auto bn = [&](int i, float(&w)[V]) __attribute__((always_inline)) {
                if constexpr (V == 4) lds_read4(tab + i * px, w);
                else w[0] = tab[i * px];
            };
#pragma unroll
            for (int l = 0; l < L; ++l) {
                float s[V], sh[V];
                bn(2 * l, s);
                bn(2 * l + 1, sh);
                if (l + 1 == L) {
                    float zero[V];
                    bn(2 * L, zero);
#pragma unroll
                    for (int i = 0; i < K_Q * V; ++i) u[i] = max2(u[i], zero[i % V]);
                }
#pragma unroll
                for (int i = 0; i < K_Q * V; ++i) u[i] = __builtin_fmaf(u[i], s[i % V], sh[i % V]);
                if (l + 1 == L) {
#pragma unroll
                    for (int i = 0; i < K_Q * V; ++i) u[i] = max2(u[i], 0.0f);
                } else if constexpr (DT == DT_BF16) {
                    round_store_all<DT, K_Q * V>(u);
                } else if constexpr (DT == DT_F16) {
#pragma unroll
                    for (int i = 0; i < K_Q * V; i += 4) {  // as in window_lists
                        asm("" : "+v"(u[i]), "+v"(u[i + 1]), "+v"(u[i + 2]), "+v"(u[i + 3]));
#pragma unroll
                        for (int e = i; e < i + 4; e += 2) {
                            const uint32_t w = pack2<DT>(u[e], u[e + 1]);
                            u[e] = half_up<DT>(w & 0xffffu);
                            u[e + 1] = half_up<DT>(w >> 16);
                        }
                    }
                }
            }
            char *const at = outp + (size_t)(uint32_t)h * ((size_t)(uint32_t)k.W * pout) + (uint32_t)(run * K_Q) * pout + (uint32_t)(ln * V) * ES;
#pragma unroll
            for (int i = 0; i < K_Q; ++i) {
                if (w0 + run * K_Q + i >= k.W) break;
                float o[V];
#pragma unroll
                for (int e = 0; e < V; ++e) o[e] = u[i * V + e];
                store_elems<DT, V, false>(at + (uint32_t)i * pout, 0, o);  // (non-temporal: 66 x 40 x 81 x 81 float32 51 -> 70 us)
            }
        }
    };
    slide_max<L, K_ROWS, V>(
        [&](int i, float(&w)[V]) __attribute__((always_inline)) { load_pixel<DT, V>(inp + (size_t)(uint32_t)min(max(o0 - L + i, 0), k.H - 1) * in_row, w); },
        [&](int i, const float(&w)[V]) __attribute__((always_inline)) {
            float *const to = mine + i % K_STEP * k.row_words;
            if (live) {
                if constexpr (V == 4) *reinterpret_cast<float4 *>(to) = make_float4(w[0], w[1], w[2], w[3]);
                else to[0] = w[0];
            }
            if (i % K_STEP == K_STEP - 1) {
                __syncthreads();
                finish(i + 1 - K_STEP);
                if (i + 1 < K_ROWS) __syncthreads();
            }
        });
}

template <int DT, int V, int L = K_BLOCKS_NHWC_MIN>
void launch_levels(const ChainWindowNhwcK &k, dim3 grid, dim3 block, uint32_t bytes, hipStream_t st)
{
    if constexpr (L <= K_BLOCKS_MAX) {
        if (k.n_levels == L) chain_window_nhwc_kernel<DT, V, L><<<grid, block, bytes, st>>>(k);
        else launch_levels<DT, V, L + 1>(k, grid, block, bytes, st);
    }
}

}  // namespace

uint64_t window_nhwc_lds(const ChainWindowNhwcK &k) { return 4ull * ((uint64_t)K_STEP * k.row_words + (uint64_t)(2 * k.n_levels + 1) * k.lanes * k.vec); }

// Channels, columns and threads of a work-group: up to 32 channels (8 lanes of four, so that a pixel's bytes fill most of a cache line), whole rows if 512
// threads hold them, else fewer channels or the fewest column tiles, whichever reads less.
bool window_nhwc_geometry(ChainWindowNhwcK &k, int64_t images, int32_t dtype, int64_t *grid, int32_t *threads)
{
    const int32_t L = k.n_levels;
    if (L < K_BLOCKS_NHWC_MIN || L > K_BLOCKS_MAX || k.W < 1 || k.H < 1 || k.C < 1) return false;
    // Large float32 tensors, rows without column tiles level by level, few levels: that kernel fills the chip and recomputes rows only.  Level by level -> window, us: six levels
    // 44 x 176 x 57 x 57 51.8 -> 63.6, 26 x 464 x 42 x 42 0.90 times as fast, five 21 x 360 x 50 x 50 0.84, four 444 x 16 x 56 x 56 0.84; 0.96 on average over 34 drawn sizes (0.80 .. 1.35).  Below, 10 to
    // 14 M cells 1.31 (10 sizes), 14 to 18 M 1.03 (16); seven levels and more 1.17 (34); rows of more than 64 columns 1.14 (21).
    if (dtype == BS_F32 && L <= 6 && k.W <= 64 && images * k.C * (int64_t)k.H * k.W >= 18000000) return false;
    k.vec = k.C % 4 == 0 ? 4 : 1;
    const int32_t all = k.C / k.vec, most = k.vec == 4 ? 8 : 32;
    double best = 0.0;
    bool found = false;
    for (int32_t want = most; want >= most / 4; want /= 2) {
        const int32_t groups = (all + want - 1) / want, lanes = (all + groups - 1) / groups;
        int32_t tiles = 1, tile_w = k.W, work = k.W;
        while (work * lanes > K_THREADS) {
            ++tiles;
            tile_w = ((k.W + tiles - 1) / tiles + 3) / 4 * 4;
            work = tile_w + 2 * L;
            if (tile_w == 4 && work * lanes > K_THREADS) break;
        }
        if (work * lanes > K_THREADS) continue;
        tiles = (k.W + tile_w - 1) / tile_w;
        if (tiles == 1) {
            tile_w = k.W;
            work = k.W;
        }
        const double cost = (double)tiles * work / k.W * (want == most ? 1.0 : want == most / 2 ? 1.25 : 1.8);
        if (found && cost >= best) continue;
        found = true;
        best = cost;
        k.lanes = lanes;
        k.tiles = tiles;
        k.tile_w = tile_w;
        k.work = work;
    }
    if (!found) return false;
    // One channel a lane and narrow tiles or few channels: float32 goes level by level (ten levels 6 x 310 x 110 x 110 105 -> 147 us, five levels
    // 27 x 326 x 53 x 53 72 -> 99; rows of 32 columns, 14 x 345 x 160 x 32 150 -> 101; binary16 3 x 318 x 141 x 141 128 -> 89).  Over drawn sizes, up to 1.3 the window is 1.84 times as fast
    // (201 sizes); beyond, 0.93 from 12 M cells on (89 sizes), 1.24 from 8 to 12 M, and never slower below 6 M (88 sizes, 1.0 .. 2.7), where the rule refuses more than it need.
    if (dtype == BS_F32 && k.vec == 1 && best > 1.3) return false;
    const int32_t columns = k.tiles == 1 ? (k.W + 3) / 4 * 4 + 2 * L : k.work, px = k.lanes * k.vec;
    k.row_words = (columns * px + 3) / 4 * 4;
    if (k.row_words % 64 == 0) k.row_words += 32;  // rows on other banks
    const int32_t groups = (all + k.lanes - 1) / k.lanes, bands = (k.H + K_ROWS - 1) / K_ROWS;
    k.div_groups = make_fastdiv((uint32_t)groups);
    k.div_tiles = make_fastdiv((uint32_t)k.tiles);
    k.div_bands = make_fastdiv((uint32_t)bands);
    k.div_lanes = make_fastdiv((uint32_t)k.lanes);
    *threads = (std::max(k.work * k.lanes, px) + 63) / 64 * 64;
    *grid = images * bands * k.tiles * groups;
    return *grid <= 0x7fffffffll && window_nhwc_lds(k) <= 64 * 1024;
}

bs_status launch_window_nhwc(const ChainWindowNhwcK &k, int64_t images, int32_t dtype, int64_t grid_n, int32_t threads, void *stream)
{
    const int32_t es = dtype == BS_F32 ? 4 : 2, L = k.n_levels, px = k.lanes * k.vec;
    // what the kernel assumes: a thread per column it reads and vector, a row of LDS that holds every run of four columns with what lies beside it, tiles and bands
    // that cover the plane, vectors that channel slices keep aligned, offsets inside a row below 4 GiB
    if (L < K_BLOCKS_NHWC_MIN || L > K_BLOCKS_MAX || k.W < 1 || k.H < 1 || (k.vec != 4 && k.vec != 1) || k.C % k.vec != 0 || k.lanes < 1 || k.tiles < 1 ||
        (k.tiles == 1 ? k.tile_w != k.W || k.work != k.W : k.tile_w % 4 != 0 || k.work != k.tile_w + 2 * L) || (int64_t)k.tiles * k.tile_w < k.W ||
        (int64_t)(k.tiles - 1) * k.tile_w >= k.W || (int64_t)k.work * k.lanes > threads || px > threads || threads > K_THREADS || threads % 64 != 0 ||
        k.row_words < (k.tiles == 1 ? (k.W + 3) / 4 * 4 + 2 * L : k.work) * px || k.row_words % 4 != 0 || window_nhwc_lds(k) > 64 * 1024 ||
        k.div_lanes.d != (uint32_t)k.lanes || k.div_tiles.d != (uint32_t)k.tiles || k.div_bands.d != (uint32_t)((k.H + K_ROWS - 1) / K_ROWS) ||
        k.div_groups.d != (uint32_t)((k.C / k.vec + k.lanes - 1) / k.lanes) ||
        grid_n != images * (int64_t)k.div_bands.d * k.tiles * (int64_t)k.div_groups.d || grid_n > 0x7fffffffll ||
        (uint64_t)k.W * ((uint64_t)k.C + std::max(k.in_xp, k.out_xp)) * es > 0xffffffffull || (k.vec == 4 && (k.in_xp % 4 != 0 || k.out_xp % 4 != 0)))
        return BS_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((uint32_t)grid_n), block((uint32_t)threads);
    const uint32_t bytes = (uint32_t)window_nhwc_lds(k);
    if (dtype == BS_F32) k.vec == 1 ? launch_levels<DT_F32, 1>(k, grid, block, bytes, st) : launch_levels<DT_F32, 4>(k, grid, block, bytes, st);
    else if (dtype == BS_BF16) k.vec == 1 ? launch_levels<DT_BF16, 1>(k, grid, block, bytes, st) : launch_levels<DT_BF16, 4>(k, grid, block, bytes, st);
    else if (dtype == BS_F16) k.vec == 1 ? launch_levels<DT_F16, 1>(k, grid, block, bytes, st) : launch_levels<DT_F16, 4>(k, grid, block, bytes, st);
    else return BS_ERR_UNSUPPORTED;
    return BS_OK;
}

}  // namespace bs
