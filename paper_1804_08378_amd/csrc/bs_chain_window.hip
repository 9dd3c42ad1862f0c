// Host side of chain_window_kernel: geometry, instances compiled into the library (float32 and bfloat16; binary16 is a run-time build, as
// for the other kernels with signature tables) and the launcher.
#include <algorithm>
#include <cstdio>
#include <string>

#include "bs_chain_window_device.h"
#include "bs_internal.h"

namespace bs {

// LDS: rows of columns with `pad` words between them, in front of the first and behind the last.
static int64_t window_words(const ChainWindowK &k) { return ((int64_t)k.ppg * k.rows * k.pitch + window_pad(k.n_levels)); }
static int64_t window_lds_bytes(const ChainWindowK &k) { return 4 * window_words(k); }
uint64_t window_lds(const ChainWindowK &k) { return (uint64_t)window_lds_bytes(k); }

// Rows, planes and threads of a work-group: bands of a plane of up to 256 lanes of pass (1) and 32 KiB, smaller ones where there would be less than
// four work-groups per compute unit; small planes share a work-group.  64 / 128 / 256 lanes, us: 64 x 64 x 56 x 56 float32 ten levels 26.2 / 24.5 / 24.5,
// 15 x 80 x 134 x 134 bfloat16 eight levels 39.7 / 31.7 / 30.8.  Four rows of pass (2) a thread; two leave half of the resident waves idle in
// pass (1) (bfloat16 as above 42), eight make pass (2) long (36).
bool window_geometry(ChainWindowK &k, int32_t dtype, const Limits &lim, int64_t *grid, int32_t *threads)
{
    const int32_t L = k.n_levels, pad = window_pad(L), vecs = (k.W + 3) / 4;
    const int32_t QV = K_WINDOW_ROWS, row_runs = (k.H + QV - 1) / QV;
    // Lanes of a row: its vectors, or, where that idles one of eight at most, the next multiple of sixteen (of eight with six levels and more), so that the lanes
    // an LDS access takes at a time lie in one row, without bank conflicts (64 x 64 x 56 x 56 float32 ten levels 23.0 -> 21.6 us, 15 x 88 x 207 x 87 binary16 nine
    // levels 51.6 -> 46.6; in eights with two levels 9 x 368 x 86 x 86 float32 40.2 -> 44.0).
    int32_t lanes = vecs;
    for (int32_t step = 16; step >= (L >= 6 ? 8 : 16) && lanes == vecs; step /= 2) {
        const int32_t up = (vecs + step - 1) / step * step;
        if (8 * (up - vecs) <= up) lanes = up;
    }
    if (L < window_fewest(dtype) || L > K_BLOCKS_MAX || k.W < 4 || k.H < 1 || k.planes < 1) return false;
    k.pitch = vecs * 4 + pad;
    const int64_t most = (int64_t)std::min<uint64_t>(lim.max_lds_bytes, 64 * 1024);
    // rows of the plane per work-group: up to 256 lanes of pass (1)
    int32_t per = std::max(1, std::min(row_runs, 256 / lanes));
    while (per > 1 && (4ll * per * QV * k.pitch > std::min<int64_t>(most, 32 * 1024) ||
                       (int64_t)k.planes * ((row_runs + per - 1) / per) < 4ll * lim.num_cus))
        --per;
    k.chunks = (row_runs + per - 1) / per;
    per = (row_runs + k.chunks - 1) / k.chunks;
    k.chunks = (row_runs + per - 1) / per;
    k.rc = k.chunks > 1 ? per * QV : k.H;
    k.rows = per * QV;
    const int32_t tasks = lanes * per;
    k.ppg = 1;
    if (k.chunks == 1)
        while (k.ppg * 2 * tasks <= 160 && (int64_t)k.planes >= (int64_t)k.ppg * 8 * lim.num_cus) k.ppg *= 2;
    while (k.ppg > 1 && window_lds_bytes(k) > std::min<int64_t>(most, 32 * 1024)) k.ppg /= 2;
    if (window_lds_bytes(k) > most) return false;
    // threads: one of pass (1) each, and no more than four rows of pass (2)
    const int32_t second = (k.rows + 3) / 4 * lanes;
    *threads = std::min(K_WINDOW_THREADS, (std::max(tasks, second) * k.ppg + 63) / 64 * 64);
    if (*threads < lanes) return false;
    k.row_slots = *threads / (lanes * k.ppg);
    k.vecs = vecs;
    *grid = ((int64_t)k.planes + k.ppg - 1) / k.ppg * k.chunks;
    if (*grid > 0x7fffffffll) return false;
    k.div_chunks = make_fastdiv((uint32_t)k.chunks);
    k.div_c = make_fastdiv((uint32_t)k.C);
    k.div_plane_tasks = make_fastdiv((uint32_t)tasks);
    k.div_lanes = make_fastdiv((uint32_t)lanes);
    k.div_second = make_fastdiv((uint32_t)(k.row_slots * lanes));
    return true;
}

// A work-group's planes are reached through offsets of 32 bits: one plane each where the images of a channel slice lie further apart.
static bool window_reaches(const ChainWindowK &k, int32_t dtype)
{
    return k.ppg == 1 || (uint64_t)k.ppg * ((uint64_t)k.H * k.W + k.in_extra) * (dtype == BS_F32 ? 4 : 2) <= 0xffffffffull;
}
void window_for_slices(ChainWindowK &k, int32_t dtype, int32_t threads, int64_t *grid)
{
    if (window_reaches(k, dtype)) return;
    k.ppg = 1;
    k.row_slots = threads / (int32_t)k.div_lanes.d;
    k.div_second = make_fastdiv((uint32_t)k.row_slots * k.div_lanes.d);
    *grid = (int64_t)k.planes * k.chunks;
}

// What the kernel assumes about its argument block and launch (window_geometry makes it so): rows of LDS that hold every run of columns with what
// lies beside it and every run of rows, chunks of whole runs that cover the plane.
bool window_launchable(const ChainWindowK &k, int32_t dtype, int64_t planes, int64_t grid, int32_t threads)
{
    const int32_t es = dtype == BS_F32 ? 4 : 2, L = k.n_levels, QV = K_WINDOW_ROWS;
    if (L < window_fewest(dtype) || L > K_BLOCKS_MAX || k.W < 4 || k.H < 1 || k.C < 1 || k.rc < 1 || k.chunks < 1 || k.ppg < 1 || k.row_slots < 1 || threads < 64 ||
        threads > K_WINDOW_THREADS || threads % 64 != 0)
        return false;
    const int32_t vecs = (k.W + 3) / 4, lanes = (int32_t)k.div_lanes.d;
    return k.vecs == vecs && lanes >= vecs && (int64_t)k.planes == planes && (int64_t)k.row_slots * lanes * k.ppg <= threads &&
           ((uint64_t)k.rows + 2 * L) * k.W * es <= 0xffffffffull &&
           window_reaches(k, dtype) &&
           k.pitch == vecs * 4 + window_pad(L) && k.rows == (k.rc + QV - 1) / QV * QV &&
           (k.chunks == 1 ? k.rc == k.H : k.rc == k.rows && k.ppg == 1) && (int64_t)k.chunks * k.rc >= k.H && (int64_t)(k.chunks - 1) * k.rc < k.H &&
           window_lds_bytes(k) <= 64 * 1024 && k.div_chunks.d == (uint32_t)k.chunks && k.div_c.d == (uint32_t)k.C &&
           k.div_plane_tasks.d == (uint32_t)(k.rows / QV * lanes) && k.div_second.d == (uint32_t)(k.row_slots * lanes) &&
           grid == (planes + k.ppg - 1) / k.ppg * k.chunks && grid <= 0x7fffffffll;
}

std::string window_expr(const ChainWindowK &k, int32_t dtype)
{
    char b[96];
    std::snprintf(b, sizeof b, "bs::chain_window_kernel<%d, %d, %d>", dtype, k.n_levels, k.W % 4);
    return b;
}

template <int DT, int REM, int L = window_fewest(DT)>
static void launch_levels(const ChainWindowK &k, dim3 grid, dim3 block, uint32_t lds, hipStream_t st)
{
    if constexpr (L <= K_BLOCKS_MAX) {
        if (k.n_levels == L) chain_window_kernel<DT, L, REM><<<grid, block, lds, st>>>(k);
        else launch_levels<DT, REM, L + 1>(k, grid, block, lds, st);
    }
}
template <int DT>
static void launch_columns(const ChainWindowK &k, dim3 grid, dim3 block, uint32_t lds, hipStream_t st)
{
    switch (k.W % 4) {
    case 0: launch_levels<DT, 0>(k, grid, block, lds, st); break;
    case 1: launch_levels<DT, 1>(k, grid, block, lds, st); break;
    case 2: launch_levels<DT, 2>(k, grid, block, lds, st); break;
    default: launch_levels<DT, 3>(k, grid, block, lds, st);
    }
}

bs_status launch_window(const ChainWindowK &k, int32_t dtype, int64_t grid_n, int32_t threads, void *stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((uint32_t)grid_n), block((uint32_t)threads);
    const uint32_t lds = (uint32_t)window_lds(k);
    if (!blocks_compiled(dtype)) return BS_ERR_UNSUPPORTED;
    if (dtype == BS_F32) launch_columns<DT_F32>(k, grid, block, lds, st);
    else launch_columns<DT_BF16>(k, grid, block, lds, st);
    return BS_OK;
}

}  // namespace bs
