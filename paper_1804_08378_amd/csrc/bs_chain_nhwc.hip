// pool_chain_nhwc_kernel: the blocks <max pooling 3 x 3 / 1 / 1, BatchNorm, ReLU> of pool_chain_kernel on channels-last tensors,
// where they are not one window (chain_window_nhwc_kernel).
//
// The levels are pool_chain_kernel's: a lane owns two columns of one channel, neighbouring columns are neighbouring lanes, rows ripple through
// all levels in registers.  In memory the channels of a pixel lie together, so a work-group of eight waves takes the same columns of `cg`
// channels: its threads fetch three rows at a time as vectors of channels, hand them to the lanes through LDS (one row of columns per
// channel), and take the results back the same way.  Both buffers are double, so a pass of three rows has one barrier; the rows of the pass
// after the next are on their way while a pass is worked on.
// What bounds it: issue as in row-major, with 14 to 20 % more vector instructions for handing the channels over, LDS bank conflicts in four of ten of its
// LDS cycles, and waiting for loads and barriers (35 % of the waves' time); two steps per launch as strips read and write every plane between
// the launches.  us, strips (two blocks a launch) -> this kernel, four / seven / ten blocks, tensors from memory: 64 x 64 x 56 x 56 float32 48 / 87 / 108 -> 30 /
// 31 / 38, bfloat16 35 / 63 / 83 -> 23 / 32 / 42; 16 x 248 x 159 x 30 float32 81 / 135 / 165 -> 42 / 45 / 54; 13 x 200 x 43 x 43 bfloat16 21 / 38 / 52 -> 16 / 25 / 35;
// 35 x 72 x 13 x 13 float32 9.7 / 19 / 26 -> 8.3 / 14 / 19.
#include <algorithm>

#include "bs_chain_device.h"
#include "bs_internal.h"

namespace bs {
namespace {

constexpr int K_THREADS = 512, K_ROWS = 3;  // threads of a work-group; rows of a pass (a ring slot's place is known at compile time)

// most vectors one thread moves per pass: spw * pitch <= 65 lanes, two columns each, eight waves
template <int VEC>
constexpr int chain_vectors() { return (K_ROWS * 8 * 130 / VEC + K_THREADS - 1) / K_THREADS; }

template <int DT, int VEC, int L>
__global__ __launch_bounds__(K_THREADS, VEC == 1 ? 2 : 4) void pool_chain_nhwc_kernel(const ChainNhwcK k)
{
    constexpr int NV = chain_vectors<VEC>();
    constexpr uint32_t ES = DT != DT_F32 ? 2 : 4;
    extern __shared__ float lds[];
    const uint32_t half = (uint32_t)(K_ROWS * k.cg * k.lp);  // floats of one buffer: [row][channel][column]
    float *const bin = lds, *const bout = lds + 2 * half;

    // work-group -> (image, chunk, column tile, channel group), the last one fastest: groups that share cache lines on one XCD
    uint32_t u = xcd_contiguous(blockIdx.x, gridDim.x);
    uint32_t v = fdiv(u, k.div_groups);
    const int32_t cfirst = (int32_t)(u - v * k.div_groups.d) * k.cg;
    u = fdiv(v, k.div_tiles);
    const int32_t w0 = (int32_t)(v - u * k.div_tiles.d) * k.tile_w;
    const uint32_t img = fdiv(u, k.div_chunks);
    const int32_t chunk = (int32_t)(u - img * k.div_chunks.d);
    const int32_t x0 = max(w0 - k.halo_w, 0);

    // the lane's columns and channel
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, seg = fdiv(lane, k.div_pitch);
    const int32_t j = (int32_t)(lane - seg * (uint32_t)k.pitch), at = x0 + 2 * j;
    int32_t ch = (int32_t)(wave * (uint32_t)k.spw + seg);
    const bool live = j + 1 < k.pitch && seg < (uint32_t)k.spw && cfirst + ch < k.C && at < k.W;
    ch = live ? ch : 0;
    const int32_t c = live ? cfirst + ch : 0;
    const uint32_t mine = (uint32_t)(ch * k.lp + (live ? 2 * j : 0)), row_floats = (uint32_t)(k.cg * k.lp);
    const bool second = live && at + 1 < k.W;  // the lane's second column lies in the plane

    float sc[L][2], sh[L][2];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const float a = k.params[k.bn[l] + c], b = k.params[k.bn[l] + k.C + c];
        sc[l][0] = live ? a : 0.0f;
        sh[l][0] = live ? b : 0.0f;
        sc[l][1] = second ? a : 0.0f;
        sh[l][1] = second ? b : 0.0f;
    }

    // the thread's vectors of a pass: (row, pixel, channel vector) -> byte offset in an image's row, place in LDS
    const uint32_t pin = (uint32_t)(k.C + (int32_t)k.in_xp) * ES, pout = (uint32_t)(k.C + (int32_t)k.out_xp) * ES;
    const char *const inp = static_cast<const char *>(k.in) + (size_t)img * (size_t)(k.H * k.W) * pin;
    char *const outp = static_cast<char *>(k.out) + (size_t)img * (size_t)(k.H * k.W) * pout;
    const uint32_t nv = (uint32_t)k.cols * k.div_cv.d;
    int32_t vrow[NV];
    uint32_t vin[NV], vout[NV], vlds[NV];
    bool vthere[NV], vstore[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const uint32_t t = threadIdx.x + (uint32_t)(i * K_THREADS), r = fdiv(t, k.div_nv), rem = t - r * nv;
        const uint32_t pix = fdiv(rem, k.div_cv), cv = rem - pix * k.div_cv.d;
        const int32_t col = x0 + (int32_t)pix, cc = cfirst + (int32_t)(cv * VEC);
        vthere[i] = t < K_ROWS * nv && cc < k.C;
        vrow[i] = vthere[i] ? (int32_t)r : 0;
        vin[i] = vthere[i] ? (uint32_t)min(col, k.W - 1) * pin + (uint32_t)cc * ES : 0u;
        vstore[i] = vthere[i] && col >= w0 && col < min(w0 + k.tile_w, k.W);
        vout[i] = vstore[i] ? (uint32_t)col * pout + (uint32_t)cc * ES : 0u;
        vlds[i] = vthere[i] ? (uint32_t)vrow[i] * row_floats + cv * VEC * (uint32_t)k.lp + pix : 0u;
    }

    const int32_t o0 = chunk * k.rc, o1 = min(o0 + k.rc, k.H);  // output rows of the chunk
    const int32_t first = max(o0 - L, 0), last = o1 - 1 + L;    // input rows (those behind the plane: padding)
    const int32_t fast_from = max(first, L), fast_to = min(k.H - 1, last);

    Raw<DT, VEC> raw[NV];
    auto request = [&](int32_t h0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const size_t row = (size_t)(uint32_t)min(max(h0 + vrow[i], 0), k.H - 1) * ((uint32_t)k.W * pin);
            raw[i] = load_raw<DT, VEC>(inp + row + vin[i], 0);
        }
    };
    auto put_in = [&](uint32_t buffer) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (vthere[i]) {
                float x[VEC];
                unpack<DT, VEC>(raw[i], x);
#pragma unroll
                for (int e = 0; e < VEC; ++e) bin[buffer * half + vlds[i] + (uint32_t)(e * k.lp)] = x[e];
            }
    };
    auto take_out = [&](uint32_t buffer, int32_t h0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int32_t r = h0 + vrow[i] - L;
            if (vstore[i] && r >= o0 && r < o1) {
                float y[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) y[e] = bout[buffer * half + vlds[i] + (uint32_t)(e * k.lp)];
                store_elems<DT, VEC, false>(outp + (size_t)(uint32_t)r * ((uint32_t)k.W * pout) + vout[i], 0, y);
            }
        }
    };

    float ring[L][3][2];  // row maxima of the three newest rows of level l (level 0: the input)
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i) ring[l][p][i] = l == 0 ? -INFINITY : 0.0f;
    // one input row; P: its place in the rings and among the rows of the pass.  EDGE: some levels' rows may not exist.
    auto row_step = [&](auto p_tag, auto edge_tag, uint32_t buffer, int32_t h) __attribute__((always_inline)) {
        constexpr int P = decltype(p_tag)::value;
        constexpr bool EDGE = decltype(edge_tag)::value != 0;
        const float2 in2 = *reinterpret_cast<const float2 *>(bin + buffer * half + (uint32_t)P * row_floats + mine);
        const bool row_there = !EDGE || h < k.H;
        const float x[2] = {__builtin_canonicalizef(live && row_there ? in2.x : -INFINITY), __builtin_canonicalizef(second && row_there ? in2.y : -INFINITY)};
        chain_input(x, ring[0][P]);
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const bool row = !EDGE || (h >= l + 1 && h < l + 1 + k.H);  // does level l + 1 have a row h - l - 1?  Else padding.
            float a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = row ? sc[l][i] : 0.0f;
                b[i] = row ? sh[l][i] : 0.0f;
            }
            if (l + 1 < L) {
                if (l == 0) chain_level<DT_F32>(ring[l], a, b, ring[l + 1 < L ? l + 1 : 0][P]);
                else chain_level<DT>(ring[l], a, b, ring[l + 1 < L ? l + 1 : 0][P]);
                continue;
            }
            float w[2];
            chain_windows(ring[l], w);
            if (l > 0) round_store_all<DT, 2>(w);
#pragma unroll
            for (int i = 0; i < 2; ++i) w[i] = __builtin_fmaxf(__builtin_fmaf(w[i], a[i], b[i]), 0.0f);
            if (live) *reinterpret_cast<float2 *>(bout + buffer * half + (uint32_t)P * row_floats + mine) = make_float2(w[0], w[1]);
        }
    };
    uint32_t buffer = 0;
    auto pass = [&](auto edge_tag, int32_t h0) __attribute__((always_inline)) {
        row_step(IntTag<0>{}, edge_tag, buffer, h0);
        row_step(IntTag<1>{}, edge_tag, buffer, h0 + 1);
        row_step(IntTag<2>{}, edge_tag, buffer, h0 + 2);
        put_in(buffer ^ 1u);  // the next pass's rows (its buffer was read in the pass before this one)
        request(h0 + 2 * K_ROWS);
        __syncthreads();
        take_out(buffer, h0);  // (written again two passes on, behind the next barrier)
        buffer ^= 1u;
    };
    request(first);
    put_in(0);
    request(first + K_ROWS);
    __syncthreads();
    int32_t h = first;  // the same for every thread of the work-group
    for (; h < fast_from; h += K_ROWS) pass(IntTag<1>{}, h);
    for (; h + K_ROWS - 1 <= fast_to; h += K_ROWS) pass(IntTag<0>{}, h);
    for (; h <= last; h += K_ROWS) pass(IntTag<1>{}, h);
}

template <int DT, int VEC, int L = K_BLOCKS_NHWC_MIN>
void launch_levels(const ChainNhwcK &k, dim3 grid, uint32_t bytes, hipStream_t st)
{
    if constexpr (L <= K_BLOCKS_MAX) {
        if (k.n_levels == L) pool_chain_nhwc_kernel<DT, VEC, L><<<grid, K_THREADS, bytes, st>>>(k);
        else launch_levels<DT, VEC, L + 1>(k, grid, bytes, st);
    }
}

}  // namespace

// Segments, channel groups, LDS rows, chunks and the grid for n images; false: the kernel does not take the plane.
bool chain_nhwc_geometry(ChainNhwcK &k, int64_t n, int32_t dtype, int32_t num_cus, int64_t *grid)
{
    const int32_t L = k.n_levels, full = dtype == BS_F32 ? 4 : 8;
    if (L < 2 || L > K_BLOCKS_MAX || k.W < 2 || k.H < 1 || k.C < 1) return false;
    k.vec = k.C % full == 0 ? full : 1;
    k.halo_w = (L + 1) / 2 * 2;
    int32_t columns = 0;
    for (k.tiles = 1;; ++k.tiles) {
        k.tile_w = ((k.W + k.tiles - 1) / k.tiles + 1) / 2 * 2;
        columns = k.tile_w + k.halo_w * std::min(k.tiles - 1, 2);
        if (columns <= 128) break;
    }
    k.tiles = (k.W + k.tile_w - 1) / k.tile_w;
    k.pitch = columns / 2 + 1;
    k.cols = columns;
    // channels per work-group: eight waves of as many segments as fit, no more than there are; rows of columns in LDS start 4 (8) banks apart so
    // that a vector's channels and 16 (8) pixels fall on different banks; both buffers twice within 64 KiB
    for (k.spw = std::min(65 / k.pitch, (k.C + 7) / 8); k.spw >= 1; --k.spw) {
        k.cg = 8 * k.spw;
        k.lp = (columns + 11) / 16 * 16 + 4;
        if ((int64_t)k.cg * k.lp * K_ROWS * 16 > 64 * 1024) k.lp = (columns + 3) / 8 * 8 + 4;
        if ((int64_t)k.cg * k.lp * K_ROWS * 16 <= 64 * 1024) break;
    }
    if (k.spw < 1) return false;
    // rows per chunk as in row-major (plan_blocks): rows walked x instructions x cycles per instruction at that many waves of a SIMD
    const int64_t groups = (k.C + k.cg - 1) / k.cg, base = n * k.tiles * groups;
    double best = 0.0;
    k.rc = k.H;
    for (int32_t chunks = 1; chunks <= k.H; ++chunks) {
        const int32_t r = (k.H + chunks - 1) / chunks;
        if (chunks > 1 && r < std::max((L + 1) / 2, std::min(6, (k.H + 1) / 2))) break;
        const int64_t count = (k.H + r - 1) / r, resident = 2 * ((base * count + num_cus - 1) / num_cus);  // waves of a SIMD
        const double walked = r + (chunks > 1 ? 2 : 1) * L, cycles = walked * (9 * L + 40) * (double)std::max<int64_t>(10, 6 + 3 * resident);
        if (chunks == 1 || cycles < 0.97 * best) {
            best = cycles;
            k.rc = r;
        }
    }
    k.chunks = (k.H + k.rc - 1) / k.rc;
    k.div_groups = make_fastdiv((uint32_t)groups);
    k.div_tiles = make_fastdiv((uint32_t)k.tiles);
    k.div_chunks = make_fastdiv((uint32_t)k.chunks);
    k.div_pitch = make_fastdiv((uint32_t)k.pitch);
    k.div_cv = make_fastdiv((uint32_t)(k.cg / k.vec));
    k.div_nv = make_fastdiv((uint32_t)(k.cols * (k.cg / k.vec)));
    *grid = base * k.chunks;
    return *grid <= 0x7fffffffll;
}

uint64_t chain_nhwc_lds_bytes(const ChainNhwcK &k) { return (uint64_t)k.cg * k.lp * K_ROWS * 16; }

bs_status launch_chain_nhwc(const ChainNhwcK &k, int64_t images, int32_t dtype, int64_t grid_n, void *stream)
{
    const int32_t full = dtype == BS_F32 ? 4 : 8, es = dtype == BS_F32 ? 4 : 2;
    const int64_t groups = k.cg > 0 ? (k.C + k.cg - 1) / k.cg : 0;
    // what the kernel assumes: tiles, halos, lanes, buffers and vectors as chain_nhwc_geometry lays them out, offsets inside a row below 4 GiB,
    // channel slices that keep a vector's alignment
    const int32_t columns = k.tile_w + k.halo_w * (k.tiles < 3 ? k.tiles - 1 : 2);
    if (k.n_levels < K_BLOCKS_NHWC_MIN || k.n_levels > K_BLOCKS_MAX || (k.vec != 1 && (k.vec != full || k.C % full != 0)) || k.W < 2 || k.H < 1 || k.rc < 1 ||
        k.halo_w < k.n_levels || k.halo_w % 2 != 0 || k.tile_w % 2 != 0 || (int64_t)k.tiles * k.tile_w < k.W || 2 * (k.pitch - 1) < columns || k.cols != columns ||
        k.spw < 1 || k.spw * k.pitch > 65 || k.cg != 8 * k.spw || k.lp < k.cols || k.lp % 2 != 0 || chain_nhwc_lds_bytes(k) > 64 * 1024 ||
        (int64_t)k.chunks * k.rc < k.H || k.div_groups.d != (uint32_t)groups || k.div_tiles.d != (uint32_t)k.tiles || k.div_chunks.d != (uint32_t)k.chunks ||
        k.div_pitch.d != (uint32_t)k.pitch || k.div_cv.d != (uint32_t)(k.cg / k.vec) || k.div_nv.d != (uint32_t)(k.cols * (k.cg / k.vec)) ||
        (int64_t)K_ROWS * k.cols * (k.cg / k.vec) > (int64_t)K_THREADS * (k.vec == 1 ? chain_vectors<1>() : k.vec == 4 ? chain_vectors<4>() : chain_vectors<8>()) ||
        grid_n != images * k.tiles * groups * k.chunks || grid_n > 0x7fffffffll ||
        (uint64_t)k.W * ((uint64_t)k.C + std::max(k.in_xp, k.out_xp)) * es > 0xffffffffull ||
        (k.vec != 1 && (k.in_xp % (uint32_t)full != 0 || k.out_xp % (uint32_t)full != 0)))
        return BS_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((uint32_t)grid_n);
    const uint32_t bytes = (uint32_t)chain_nhwc_lds_bytes(k);
    if (dtype == BS_F32) k.vec == 1 ? launch_levels<DT_F32, 1>(k, grid, bytes, st) : launch_levels<DT_F32, 4>(k, grid, bytes, st);
    else if (dtype == BS_BF16) k.vec == 1 ? launch_levels<DT_BF16, 1>(k, grid, bytes, st) : launch_levels<DT_BF16, 8>(k, grid, bytes, st);
    else if (dtype == BS_F16) k.vec == 1 ? launch_levels<DT_F16, 1>(k, grid, bytes, st) : launch_levels<DT_F16, 8>(k, grid, bytes, st);
    else return BS_ERR_UNSUPPORTED;
    return BS_OK;
}

}  // namespace bs
