// Host side of pool_chain_kernel: instances compiled into the library (float32 and bfloat16, two to ten blocks; binary16 is a run-time
// build, as for the other kernels with signature tables) and the launcher.
#include <cstdio>
#include <string>

#include "bs_chain_device.h"
#include "bs_internal.h"

namespace bs {

bool blocks_compiled(int32_t dtype) { return dtype_has_tables(dtype); }

std::string blocks_expr(const ChainK &k, int32_t dtype)
{
    char b[96];
    std::snprintf(b, sizeof b, "bs::pool_chain_kernel<%d, %s, %d>", dtype, k.W % 2 ? "true" : "false", k.n_levels);
    return b;
}

// Most output rows of a chunk: the rows it reads, L above and below its own among them, span less than 4 GiB (of float32).
int32_t blocks_most_rows(const ChainK &k) { return (int32_t)(0xffffffffll / (4ll * k.W)) - 2 * k.n_levels; }

// What the kernel assumes about its argument block and launch: column tiles that fit a wave with an idle lane between two segments and
// halos that hold the levels' reach, chunks that cover the plane and whose rows 32-bit offsets reach, a grid that covers every (group of segments, chunk).
bool blocks_launchable(const ChainK &k, int64_t planes, int64_t grid, int32_t threads)
{
    if (k.n_levels < 2 || k.n_levels > K_BLOCKS_MAX || k.W < 2 || k.H < 1 || k.tiles < 1 || k.rc < 1 || k.chunks < 1 || k.spw < 1) return false;
    const int32_t columns = k.tile_w + k.halo_w * (k.tiles < 3 ? k.tiles - 1 : 2);
    return k.tile_w % 2 == 0 && k.halo_w % 2 == 0 && k.halo_w >= k.n_levels && (int64_t)k.tiles * k.tile_w >= k.W && 2 * (k.pitch - 1) >= columns &&
           k.spw * k.pitch <= 65 && k.div_pitch.d == (uint32_t)k.pitch && k.div_chunks.d == (uint32_t)k.chunks &&
           k.div_tiles.d == (uint32_t)k.tiles && k.div_c.d == (uint32_t)k.C && (int64_t)k.chunks * k.rc >= k.H && k.rc <= blocks_most_rows(k) && k.units == (uint64_t)(planes * k.tiles) &&
           threads >= 64 && threads <= 256 && threads % 64 == 0 &&
           grid * (threads / 64) >= (((int64_t)k.units + k.spw - 1) / k.spw) * k.chunks;
}

template <int DT, bool RAGGED, int L = 2>
static void launch_levels(const ChainK &k, dim3 grid, dim3 block, hipStream_t st)
{
    if constexpr (L <= K_BLOCKS_MAX) {
        if (k.n_levels == L) pool_chain_kernel<DT, RAGGED, L><<<grid, block, 0, st>>>(k);
        else launch_levels<DT, RAGGED, L + 1>(k, grid, block, st);
    }
}

bs_status launch_blocks(const ChainK &k, int32_t dtype, int64_t grid_n, int32_t threads, void *stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((uint32_t)grid_n), block((uint32_t)threads);
    if (!blocks_compiled(dtype)) return BS_ERR_UNSUPPORTED;
    if (dtype == BS_F32 && k.W % 2 == 0) launch_levels<DT_F32, false>(k, grid, block, st);
    else if (dtype == BS_F32) launch_levels<DT_F32, true>(k, grid, block, st);
    else if (k.W % 2 == 0) launch_levels<DT_BF16, false>(k, grid, block, st);
    else launch_levels<DT_BF16, true>(k, grid, block, st);
    return BS_OK;
}

}  // namespace bs
