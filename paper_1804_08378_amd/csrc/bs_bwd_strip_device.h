// Places, loads and stores of the backward kernels whose lanes walk strips of columns (bs_backward_strip.hip, bs_backward_keys.hip).
#pragma once
#include "bs_bwd_device.h"
#include "bs_strip_device.h"

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
    const char *p = static_cast<const char *>(base) + audited_bytes<DT, OFF>(k, which, site, off, V);
    if constexpr (V == 2) return *reinterpret_cast<const uint32_t *>(p);
    uint32_t w[1];
    load_run<DT, 1>(p, w);
    return w[0];
}

// Non-temporal: the input gradient is written once.  Measured, channels-last backward (bwd_keys_kernel), us, plain / non-temporal: ResNet stem bfloat16
// 50.2 / 46.2, float32 100.9 / 94; 32 x 192 x 71 x 71 bfloat16 38.3 / 35.2.
template <int DT, typename OFF, int V = 1>
BS_DEV void store_at(const BwdK &k, int site, void *base, OFF off, const float *v)
{
    char *p = static_cast<char *>(base) + audited_bytes<DT, OFF>(k, 2, site, off, V);
    if constexpr (DT == DT_F32) __builtin_nontemporal_store(v[0], reinterpret_cast<float *>(p));
    else if constexpr (V == 2) __builtin_nontemporal_store(pack2<DT>(v[0], v[1]), reinterpret_cast<uint32_t *>(p));
    else __builtin_nontemporal_store(half_bits<DT>(v[0]), reinterpret_cast<uint16_t *>(p));
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

}  // namespace
}  // namespace bs
