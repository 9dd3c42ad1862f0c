// pool_band_kernel: one pooling step with stride 2 (max 3 x 3 with and without padding and picks, float32 also max 2 x 2 and average 2 x 2) and
// BatchNorm -> ReLU on row-major planes whose rows are no whole vectors.
//
// The rows under a band of output rows are one run of memory whatever their length: a work-group fetches it as aligned 128-bit vectors, several of each
// thread on their way at a time, to LDS as it lies in memory (lists in front of the pooling applied on the way), and a lane takes its window from there.
// The strips it stands in for read their columns as vectors at whatever address they begin, a row pair of a lane in flight.  float32: a lane takes one output;
// 16-bit storage: four, whose columns are words of two (one output a lane, nine 16-bit reads each: 26.4 us where four took 20.8).
// What bounds it: memory (32 x 64 x 147 x 147 binary16 3 x 3 maximum 28.0 -> 21.6 us, 5.1 TB/s; 3 x 314 x 145 x 145 float32 27.8 -> 17.6, 5.6 TB/s).
#include <algorithm>

#include "bs_internal.h"
#include "bs_strip_device.h"

namespace bs {
namespace {

constexpr int K_BAND_THREADS = 256, K_BAND_BYTES = 16 * 1024;

// MAX: maximum (else the average of four), K x K, padding P; IDX: with picks, the list in front; else a maximum's list stands behind it, an average's in front.
// 16-bit storage: 3 x 3 maxima only (strips are as fast with 2 x 2 windows, pool_band_geometry).
template <int DT, bool MAX, int K, int P, bool IDX>
__global__ __launch_bounds__(K_BAND_THREADS) void pool_band_kernel(const PoolBandK k)
{
    static_assert(DT == DT_F32 || (MAX && K == 3), "16-bit storage: 3 x 3 maxima");
    constexpr int ES = DT == DT_F32 ? 4 : 2, VEC = 16 / ES, U = 4;
    constexpr bool PRE = IDX || !MAX;
    extern __shared__ uint4 lds_vectors[];
    uint4 *const band = lds_vectors + 1;  // (a window of the first row may begin in front of it, one of the last row end behind)
    quiet_maxima();
    const uint32_t block = xcd_contiguous(blockIdx.x, gridDim.x), plane = fdiv(block, k.div_bands), img = fdiv(plane, k.div_c);
    const int32_t oh0 = (int32_t)(block - plane * k.div_bands.d) * k.rows, oh1 = min(oh0 + k.rows, k.Ho);
    const uint32_t c = plane - img * (uint32_t)k.C;
    const float scale = k.bn < 0 ? 1.0f : k.params[k.bn + c], shift = k.bn < 0 ? 0.0f : k.params[k.bn + k.C + c];

    // the run: rows r0 .. r1 of the plane, from the vector that holds its first element on
    const int32_t r0 = max(oh0 * 2 - P, 0), r1 = min((oh1 - 1) * 2 - P + K, k.H);
    const size_t plane_at = ((size_t)plane * k.H * k.W + (size_t)img * k.in_extra) * ES;
    const size_t from = plane_at + (size_t)((uint32_t)r0 * (uint32_t)k.W) * ES, first = from & ~(size_t)15;
    const int32_t lead = (int32_t)(from - first) / ES, vectors = (lead + (r1 - r0) * k.W + VEC - 1) / VEC;
    const char *const inp = static_cast<const char *>(k.in) + first;
    const bool whole = first + (size_t)vectors * 16 <= k.in_bytes;  // else the last vector reaches beyond the tensor
    const int32_t inside = whole ? vectors : vectors - 1;
    auto prepared = [&](uint4 q) __attribute__((always_inline)) {
        if constexpr (PRE) {
            Raw<DT, VEC> r;
            r.q = q;
            float x[VEC];
            unpack<DT, VEC>(r, x);
#pragma unroll
            for (int e = 0; e < VEC; ++e) x[e] = __builtin_fmaf(x[e], scale, shift);
            uint32_t w[4];
            if constexpr (DT == DT_F16) {  // (two roundings, as in round_store)
#pragma unroll
                for (int e = 0; e < VEC; e += 4) asm("" : "+v"(x[e]), "+v"(x[e + 1]), "+v"(x[e + 2]), "+v"(x[e + 3]));
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) x[e] = __builtin_fmaxf(x[e], 0.0f);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (DT == DT_F32) w[e] = __float_as_uint(x[e]);
                else w[e] = pack2<DT>(x[2 * e % VEC], x[(2 * e + 1) % VEC]);
            }
            q = make_uint4(w[0], w[1], w[2], w[3]);
        }
        return q;
    };
    for (int32_t v = (int32_t)threadIdx.x; v < inside; v += U * (int32_t)blockDim.x) {
        Raw<DT, VEC> raw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) raw[u] = load_raw<DT, VEC>(inp + (size_t)(uint32_t)min(v + u * (int32_t)blockDim.x, inside - 1) * 16, 0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (v + u * (int32_t)blockDim.x < inside) band[v + u * (int32_t)blockDim.x] = prepared(raw[u].q);
    }
    if (!whole && threadIdx.x == 0) {  // at the tensor's end, one element at a time
        const char *const last = inp + (size_t)(uint32_t)inside * 16;
        const int32_t there = (int32_t)((int64_t)(k.in_bytes - first) - (int64_t)inside * 16) / ES;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            if (e < there) {
                if constexpr (DT == DT_F32) w[e % 4] = *reinterpret_cast<const uint32_t *>(last + 4 * e);
                else w[e / 2] |= (uint32_t)*reinterpret_cast<const uint16_t *>(last + 2 * e) << (e % 2 * 16);
            }
        band[inside] = prepared(make_uint4(w[0], w[1], w[2], w[3]));
    }
    __syncthreads();

    const char *const lds = reinterpret_cast<const char *>(band) + lead * ES;
    const size_t out_at = ((size_t)plane * k.Ho + (size_t)oh0) * k.Wo;
    char *const outp = static_cast<char *>(k.out) + (out_at + (size_t)img * k.out_extra) * ES;
    if constexpr (DT == DT_F32) {
        const int32_t outputs = (oh1 - oh0) * k.Wo;
        for (int32_t o = (int32_t)threadIdx.x; o < outputs; o += (int32_t)blockDim.x) {
            const int32_t oh = (int32_t)fdiv((uint32_t)o, k.div_wo), ow = o - oh * k.Wo;
            // a cell outside the plane: its nearest one, which the window holds as well
            int32_t row[K], col[K];
#pragma unroll
            for (int d = 0; d < K; ++d) {
                row[d] = min(max((oh0 + oh) * 2 - P + d, 0), k.H - 1);
                col[d] = min(max(ow * 2 - P + d, 0), k.W - 1);
            }
            float w[K * K];
#pragma unroll
            for (int i = 0; i < K; ++i)
#pragma unroll
                for (int j = 0; j < K; ++j) w[i * K + j] = *reinterpret_cast<const float *>(lds + ((row[i] - r0) * k.W + col[j]) * 4);
            float y;
            if constexpr (!MAX) {
                y = 0.0f + w[0];
#pragma unroll
                for (int i = 1; i < K * K; ++i) y += w[i];
                y *= 1.0f / (K * K);
            } else if constexpr (!IDX) {
                y = K == 2 ? max2(max3(w[0], w[1], w[2]), w[3]) : max3(max3(w[0], w[1], w[2]), max3(w[3], w[4 % (K * K)], w[5 % (K * K)]), max3(w[6 % (K * K)], w[7 % (K * K)], w[8 % (K * K)]));
                y = __builtin_fmaxf(__builtin_fmaf(y, scale, shift), 0.0f);
            } else {
                int32_t at = 0;
                y = w[0];
#pragma unroll
                for (int i = 1; i < K * K; ++i) take_if_more(w[i], i, y, at);
                const int32_t dh = at >= 2 * K ? 2 : at >= K ? 1 : 0, dw = at - dh * K;
                k.idx[out_at + (uint32_t)o] = min(max((oh0 + oh) * 2 - P + dh, 0), k.H - 1) * k.W + min(max(ow * 2 - P + dw, 0), k.W - 1);
            }
            reinterpret_cast<float *>(outp)[o] = y;
        }
    } else {
        // four outputs a lane: the columns under them are words of two, half a word further where they begin at an odd element
        constexpr int Q = 4, NC = 2 * (Q - 1) + K, NW = (NC + 1) / 2;
        const int32_t runs = (int32_t)k.div_runs.d, tasks = (oh1 - oh0) * runs;
        for (int32_t t = (int32_t)threadIdx.x; t < tasks; t += (int32_t)blockDim.x) {
            const int32_t oh = (int32_t)fdiv((uint32_t)t, k.div_runs), ow = (t - oh * runs) * Q, col = ow * 2 - P;
            int32_t row[K];
            uint32_t w[K][NW];  // columns col, col + 1, ... of the rows
#pragma unroll
            for (int i = 0; i < K; ++i) {
                row[i] = min(max((oh0 + oh) * 2 - P + i, 0), k.H - 1);  // outside the plane: its nearest row, which the window holds as well
                const int32_t at = lead + (row[i] - r0) * k.W + col;
                const uint32_t *const words = reinterpret_cast<const uint32_t *>(band) + (at >> 1);
                uint32_t x[NW + 1];
#pragma unroll
                for (int n = 0; n < NW + 1; ++n) x[n] = words[n];
#pragma unroll
                for (int n = 0; n < NW; ++n) w[i][n] = __builtin_amdgcn_alignbit(x[n + 1], x[n], (at & 1) * 16);
            }
            float y[Q];
            if constexpr (!IDX) {
                float m[NC];
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    m[j] = max3(run_element<DT>(w[0], j), run_element<DT>(w[1], j), run_element<DT>(w[K - 1], j));
                    m[j] = (uint32_t)(col + j) < (uint32_t)k.W ? m[j] : -INFINITY;
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    y[q] = max3(m[2 * q], m[2 * q + 1], m[2 * q + K - 1]);
                    y[q] = __builtin_fmaxf(__builtin_fmaf(y[q], scale, shift), 0.0f);
                }
            } else {
                // per column the first maximum of its rows, then of the window's columns: keys of value and, growing towards the first cell, 4 * row + column
                uint32_t key[NC];
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    uint32_t c[K];
#pragma unroll
                    for (int i = 0; i < K; ++i) c[i] = (j % 2 ? w[i][j / 2] & 0xffff0000u : w[i][j / 2] << 16) | (uint32_t)(4 * (K - i));
                    key[j] = max(max(c[0], c[1]), c[K - 1]);
                    key[j] = (uint32_t)(col + j) < (uint32_t)k.W ? key[j] : 0u;
                }
                int32_t pick[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const uint32_t best = max(max(key[2 * q] + 2u, key[2 * q + 1] + 1u), key[2 * q + K - 1]);
                    y[q] = half_up<DT>(best >> 16);
                    const int32_t code = (int32_t)(best & 0xffffu), r = code >> 2;  // r: K for the first row
                    pick[q] = (r == K ? row[0] : r == K - 1 ? row[1] : row[K - 1]) * k.W + col + 2 * q + 2 - (code & 3);
                }
                int32_t *const to = k.idx + out_at + (uint32_t)(oh * k.Wo + ow);
                struct __attribute__((packed, aligned(4))) I4 { int32_t p[4]; };
                if (ow + Q <= k.Wo) *reinterpret_cast<I4 *>(to) = {{pick[0], pick[1], pick[2], pick[3]}};
                else {
#pragma unroll
                    for (int q = 0; q + 1 < Q; ++q)
                        if (ow + q < k.Wo) to[q] = pick[q];
                }
            }
            char *const to = outp + (uint32_t)(oh * k.Wo + ow) * 2u;
#pragma unroll
            for (int q = 0; q < Q; ++q) y[q] = round_store<DT>(y[q]);
            const uint32_t lo = pack2<DT>(y[0], y[1]), hi = pack2<DT>(y[2], y[3]);
            if (ow + Q <= k.Wo) {
                // (Non-temporal stores gain nothing.  Plain / non-temporal, binary16, us, three inputs in turn: 32 x 64 x 147 x 147 21.9 / 20.9, 21 x 64 x 199 x 199 25.9 / 26.5,
                // 64 x 96 x 75 x 75 17.1 / 17.5; eight inputs 22.7 / 23.8, 26.0 / 27.3, 19.5 / 20.5; with a reader behind each call 30.0 / 31.5, 35.6 / 40.2, 23.4 / 24.9.)
                struct __attribute__((packed, aligned(2))) W2 { uint32_t a, b; };
                *reinterpret_cast<W2 *>(to) = {lo, hi};
            } else {
                const int32_t rest = k.Wo - ow;
                struct __attribute__((packed, aligned(2))) W1 { uint32_t a; };
                if (rest & 2) *reinterpret_cast<W1 *>(to) = {lo};
                if (rest & 1) *reinterpret_cast<uint16_t *>(to + (rest & 2) * 2) = (uint16_t)(rest & 2 ? hi : lo);
            }
        }
    }
}

template <int DT>
void launch_as(const PoolBandK &k, dim3 grid, dim3 block, uint32_t lds, hipStream_t st)
{
    if constexpr (DT == DT_F32) {
        if (k.k == 2) return k.kind != OP_MAXPOOL ? pool_band_kernel<DT, false, 2, 0, false><<<grid, block, lds, st>>>(k) : pool_band_kernel<DT, true, 2, 0, false><<<grid, block, lds, st>>>(k);
    }
    if (k.idx) k.pad ? pool_band_kernel<DT, true, 3, 1, true><<<grid, block, lds, st>>>(k) : pool_band_kernel<DT, true, 3, 0, true><<<grid, block, lds, st>>>(k);
    else k.pad ? pool_band_kernel<DT, true, 3, 1, false><<<grid, block, lds, st>>>(k) : pool_band_kernel<DT, true, 3, 0, false><<<grid, block, lds, st>>>(k);
}

// LDS of a band: its rows, what their first vector holds in front of them, 16 bytes in front and 32 behind.
int64_t band_bytes(const PoolBandK &k, int32_t rows, int32_t es)
{
    const int64_t in_rows = std::min<int64_t>((int64_t)(rows - 1) * 2 + k.k, k.H);
    return (in_rows * k.W * es + 15 + 15) / 16 * 16 + 16 + 32;
}

}  // namespace

uint64_t pool_band_lds(const PoolBandK &b, int32_t dtype) { return (uint64_t)band_bytes(b, b.rows, dtype == BS_F32 ? 4 : 2); }

// The strips' step as bands, if the kernel exists for it.
bool pool_band_geometry(PoolBandK &b, const StripK &k, bool idx, int64_t planes, int32_t dtype, int32_t num_cus, int64_t *grid, int32_t *threads)
{
    const PoolK &p = k.pool2;
    const int32_t es = dtype == BS_F32 ? 4 : 2;
    if (k.nhwc || k.pool1.kind != 0 || p.kh != p.kw || p.ph != p.pw || p.sh != 2 || p.sw != 2 || k.n_mid != 0) return false;
    const bool max = p.kind == OP_MAXPOOL;
    if (max ? !((p.kh == 2 && p.ph == 0 && !idx) || (p.kh == 3 && p.ph <= 1)) : !(p.kh == 2 && p.ph == 0 && 2 * k.Ho <= k.H && 2 * k.Wo <= k.W)) return false;
    // Strips -> bands, us.  float32: 2 x 2 maximum 13 x 480 x 62 x 62 35.1 -> 21.3, average 21 x 26 x 185 x 185 20.9 -> 15.7, 3 x 3 maximum 3 x 314 x 145 x 145 27.8 -> 17.6,
    // 96 x 360 x 12 x 18 13.0 -> 11.0.  16-bit storage: 3 x 3 maximum 32 x 64 x 147 x 147 binary16 28.2 -> 21.3, 60 x 120 x 59 x 59 16.4 -> 13.6, with picks
    // 15 x 264 x 79 x 79 bfloat16 (and backward) 68 -> 59; no gain with 2 x 2 windows (8 x 240 x 109 x 109 11.8 -> 12.1, average 3 x 80 x 219 x 219 7.1 -> 8.1),
    // on small planes (38 x 240 x 11 x 11 with picks and backward 12.2 -> 13.8) and without picks on inputs the last cache holds (2 x 254 x 171 x 171, 30 MB, 9.0 -> 10.0;
    // 7 x 176 x 134 x 134, 44 MB, 15.1 -> 13.1).  Over 220 drawn sizes that this takes, geometric means: float32 2 x 2 1.29 (0.98 .. 1.8), 3 x 3 1.32 without picks and 1.42 with
    // (0.97 .. 2.4); 16-bit storage 3 x 3 1.16 without picks (0.89 .. 2.4; with eight inputs in turn 1.32, 0.97 and more) and 1.16 with (0.91 .. 3.3).
    const int64_t cells = (int64_t)k.H * k.W;
    if (dtype == BS_F32 ? cells < 200 : p.kh == 2 || cells < 600 || (!idx && planes * cells < 20 << 20)) return false;
    const bool front = idx || !max;  // where the list has to stand
    const EwOp *list = front ? k.pre : k.post;
    const int32_t n = front ? k.n_pre : k.n_post, other = front ? k.n_post : k.n_pre;
    if (other != 0 || strip_list_code(list, n) != BN_RELU) return false;
    b = PoolBandK{};
    b.bn = n == 2 ? list[0].arg : -1;
    b.C = k.C; b.H = k.H; b.W = k.W; b.Ho = k.Ho; b.Wo = k.Wo;
    b.kind = p.kind; b.k = p.kh; b.pad = p.ph;
    // as many output rows as 16 KiB hold the rows of (8 / 16 / 32 KiB, us: 32 x 64 x 147 x 147 binary16 23.9 / 21.2 / 24.7, 8 x 125 x 150 x 150 float32 23.4 / 20.3 / 24.1), fewer where there would be less than eight work-groups per compute unit, evened out
    int32_t rows = k.Ho;
    while (rows > 1 && (band_bytes(b, rows, es) > K_BAND_BYTES || planes * ((k.Ho + rows - 1) / rows) < 8ll * num_cus)) --rows;
    if (band_bytes(b, rows, es) > 64 * 1024) return false;
    b.bands = (k.Ho + rows - 1) / rows;
    b.rows = (k.Ho + b.bands - 1) / b.bands;
    b.bands = (k.Ho + b.rows - 1) / b.rows;
    b.div_bands = make_fastdiv((uint32_t)b.bands);
    b.div_c = make_fastdiv((uint32_t)b.C);
    b.div_wo = make_fastdiv((uint32_t)b.Wo);
    b.div_runs = make_fastdiv((uint32_t)((b.Wo + 3) / 4));
    *threads = (int32_t)std::min<int64_t>(K_BAND_THREADS, std::max<int64_t>(64, (std::max<int64_t>(band_bytes(b, b.rows, es) / 32, dtype == BS_F32 ? b.rows * b.Wo / 2 : b.rows * ((b.Wo + 3) / 4)) + 63) / 64 * 64));
    *grid = planes * b.bands;
    return *grid <= 0x7fffffffll;
}

bs_status launch_pool_band(const PoolBandK &b, int64_t planes, int32_t dtype, int64_t grid_n, int32_t threads, void *stream)
{
    const int32_t es = dtype == BS_F32 ? 4 : 2;
    PoolBandK k = b;
    const int64_t bytes = band_bytes(k, k.rows, es), images = planes / std::max(k.C, 1);
    // what the kernel assumes: an instance for the step, bands that cover the output, LDS for a band's run, a window per output with a cell in the plane
    if (!(k.kind == OP_MAXPOOL ? (k.k == 2 && k.pad == 0 && !k.idx) || (k.k == 3 && (k.pad == 0 || k.pad == 1)) : k.k == 2 && k.pad == 0) || (dtype != BS_F32 && k.k == 2) || k.C < 1 || planes % k.C != 0 || k.H < 1 || k.W < 1 || k.Ho < 1 || k.Wo < 1 || k.rows < 1 || (int64_t)k.bands * k.rows < k.Ho || (int64_t)(k.bands - 1) * k.rows >= k.Ho ||
        (k.Ho - 1) * 2 - k.pad >= k.H || (k.Wo - 1) * 2 - k.pad >= k.W || bytes > 64 * 1024 || grid_n != planes * k.bands || grid_n > 0x7fffffffll || threads < 64 ||
        threads > K_BAND_THREADS || threads % 64 != 0 || k.div_bands.d != (uint32_t)k.bands || k.div_c.d != (uint32_t)k.C || k.div_wo.d != (uint32_t)k.Wo || k.div_runs.d != (uint32_t)((k.Wo + 3) / 4) ||
        (k.kind != OP_MAXPOOL && (2 * k.Ho > k.H || 2 * k.Wo > k.W)) || (uint64_t)k.H * k.W > 0x7fffffffull)
        return BS_ERR_UNSUPPORTED;
    k.in_bytes = ((uint64_t)planes * k.H * k.W + (uint64_t)(images - 1) * k.in_extra) * es;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((uint32_t)grid_n), block((uint32_t)threads);
    if (dtype == BS_F32) launch_as<DT_F32>(k, grid, block, (uint32_t)bytes, st);
    else if (dtype == BS_BF16) launch_as<DT_BF16>(k, grid, block, (uint32_t)bytes, st);
    else if (dtype == BS_F16) launch_as<DT_F16>(k, grid, block, (uint32_t)bytes, st);
    else return BS_ERR_UNSUPPORTED;
    return BS_OK;
}

}  // namespace bs
