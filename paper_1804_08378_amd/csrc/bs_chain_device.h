// pool_chain_kernel: L blocks <max pooling 3 x 3 / 1 / 1, BatchNorm, ReLU> in registers -- the stacked blocks of Section 5.1, where
// they are not one window (chain_window_kernel: every BatchNorm but the last with scales above zero; the rules are at plan_window).
//
// A lane owns two columns of a plane and walks down a chunk of its rows; every new input row ripples through all L levels in the same
// step, because level l's row h - l needs level l - 1's rows up to h - l + 1, which that step has just produced.  Per level the lane
// keeps three rows of *row maxima* (the maximum over each window's three columns), so a window's value is one three-operand maximum.
//
// What bounds it is instruction issue at the two waves per SIMD that planes of this size give (ten levels: one vector instruction per 6.1 cycles in
// float32, 5.3 in bfloat16), in float32 beside the latency of the loads (waves wait 36 % of their time; bfloat16 16 %), so the step is written for
// few instructions: 3.5 per cell and level.
//   Columns: the maximum of a lane's two columns and ReLU's zero is one three-operand instruction shared by two windows (a max
//   pooling follows, so "not below zero" may be applied to the window instead of the cell); the neighbouring lane's edge column is
//   an operand of the window's last maximum (data-parallel-primitive operand), not a move.
//   Edges: behind a ReLU a cell outside the plane may count as zero instead of -inf.  Between two rows of lanes lies one lane whose
//   BatchNorm has scale and shift zero, so that its values are the padding on both sides; columns beyond a ragged row's end have
//   zero scale and shift as well.  No masks in the loop; only the first level, which reads raw values, is padded with -inf.
//   Rows: all lanes of a wave are at the same row (segments of a wave are different planes, the same chunk), so the passes whose rows
//   exist on every level are a loop of their own without any test of them.
// Measured, us, 64 x 64 x 56 x 56 float32 (102.8 MB), calls back to back over tensors from memory / on one tensor that the last cache holds: ten levels
// 32.5 / 27.8 in one launch (the kernel for other lists, 14 instructions per cell and level: 62.3 / 58.0 in two); four levels 26.6 / 18.9 (3.9 TB/s from memory).
// Rounding to the storage type commutes with maximum and ReLU: a level's values are rounded after the next level's maximum.
#pragma once
#include "bs_xrows_device.h"

namespace bs {

// These steps are written as instructions: the compiler cannot know that values which came through a lane shift or an asm block are no
// signalling NaNs and would first copy each of them through a maximum with itself (a level's values are results of fused multiply-adds,
// and the input is made canonical once).  An operand read from another lane needs two wait states after the instruction that wrote it:
// every block below has two instructions between the two.
#define BS_CHAIN_KEEP(a, b) ""
#define BS_CHAIN_BF16(a, b) /* nearest-even, both values, and back */ \
    "v_cvt_pk_bf16_f32 %[" a "], %[" a "], %[" b "]\n\t"             \
    "v_and_b32 %[" b "], 0xffff0000, %[" a "]\n\t"                   \
    "v_lshlrev_b32 %[" a "], 16, %[" a "]\n\t"
#define BS_CHAIN_F16(a, b)                     \
    "v_cvt_f16_f32 %[" a "], %[" a "]\n\t"    \
    "v_cvt_f16_f32 %[" b "], %[" b "]\n\t"    \
    "v_cvt_f32_f16 %[" a "], %[" a "]\n\t"    \
    "v_cvt_f32_f16 %[" b "], %[" b "]\n\t"
#define BS_CHAIN_SHR " wave_shr:1 row_mask:0xf bank_mask:0xf"
#define BS_CHAIN_SHL " wave_shl:1 row_mask:0xf bank_mask:0xf"

// Window maxima of a lane's columns from their three rows of row maxima.
BS_DEV void chain_windows(const float (&r)[3][2], float (&v)[2])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) asm("v_max3_f32 %0, %1, %2, %3" : "=v"(v[i]) : "v"(r[0][i]), "v"(r[1][i]), "v"(r[2][i]));
}
// ... rounded to the storage type (ROUND), through BatchNorm (c, h: scale and shift, of each column where PC > 1), and the row maxima behind
// the ReLU of the columns: n[0] with the last column of the lane before, n[1] with the first one of the lane behind (the wave's ends: 0).
#define BS_CHAIN_LEVEL(ROUND)                                                                                                       \
    asm("v_max3_f32 %[a], %[r0], %[r1], %[r2]\n\t"                                                                                   \
        "v_max3_f32 %[b], %[s0], %[s1], %[s2]\n\t" ROUND("a", "b")                                                                   \
        "v_fma_f32 %[b], %[b], %[c1], %[h1]\n\t"                                                                                     \
        "v_fma_f32 %[a], %[a], %[c0], %[h0]\n\t"                                                                                     \
        "v_max3_f32 %[q], %[a], %[b], 0\n\t"                                                                                         \
        "v_max_f32_dpp %[n0], %[b], %[q]" BS_CHAIN_SHR " bound_ctrl:1\n\t"                                                           \
        "v_max_f32_dpp %[n1], %[a], %[q]" BS_CHAIN_SHL " bound_ctrl:1"                                                               \
        : [a] "=&v"(a), [b] "=&v"(b), [q] "=&v"(q), [n0] "=&v"(n[0]), [n1] "=&v"(n[1])                                               \
        : [r0] "v"(r[0][0]), [r1] "v"(r[1][0]), [r2] "v"(r[2][0]), [s0] "v"(r[0][1]), [s1] "v"(r[1][1]), [s2] "v"(r[2][1]),          \
          [c0] "v"(c[0]), [h0] "v"(h[0]), [c1] "v"(c[PC - 1]), [h1] "v"(h[PC - 1]))
template <int ROUND, int PC>
BS_DEV void chain_level(const float (&r)[3][2], const float (&c)[PC], const float (&h)[PC], float (&n)[2])
{
    float a, b, q;
    if constexpr (ROUND == DT_F32) BS_CHAIN_LEVEL(BS_CHAIN_KEEP);
    else if constexpr (ROUND == DT_BF16) BS_CHAIN_LEVEL(BS_CHAIN_BF16);
    else BS_CHAIN_LEVEL(BS_CHAIN_F16);
}
// Row maxima of the input's two columns: no neighbour beyond the wave's ends.
BS_DEV void chain_input(const float (&x)[2], float (&n)[2])
{
    n[0] = n[1] = __builtin_fmaxf(x[0], x[1]);
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %[n0], %[x1], %[n0]" BS_CHAIN_SHR "\n\t"
        "v_max_f32_dpp %[n1], %[x0], %[n1]" BS_CHAIN_SHL
        : [n0] "+&v"(n[0]), [n1] "+&v"(n[1])
        : [x0] "v"(x[0]), [x1] "v"(x[1]));
}

// Two consecutive elements of a row, as they lie in memory.
template <int DT>
struct ChainRow {
    uint32_t w[DT != DT_F32 ? 1 : 2];
};
template <int DT>
BS_DEV void chain_unpack(const ChainRow<DT> &r, float (&x)[2])
{
    if constexpr (DT == DT_F32) {
        x[0] = __uint_as_float(r.w[0]);
        x[1] = __uint_as_float(r.w[1]);
    } else {
        x[0] = half_up<DT>(r.w[0] & 0xffffu);
        x[1] = half_up<DT>(r.w[0] >> 16);
    }
}
// Vector registers of an instance: rings, parameters, requested rows and the rest; the waves per SIMD that leaves room for.
constexpr int chain_waves(int dt, bool ragged, int levels)
{
    const int regs = 6 * levels + (ragged ? 4 : 2) * levels + 6 * (dt == DT_F32 ? 2 : 1) + 24;
    return regs <= 64 ? 8 : regs <= 96 ? 5 : regs <= 128 ? 4 : 3;
}

// RAGGED: rows of an odd number of columns (the last lane reads the row's last two and shifts them).
template <int DT, bool RAGGED, int L>
__global__ __launch_bounds__(256, chain_waves(DT, RAGGED, L)) void pool_chain_kernel(const ChainK k)
{
    // Rows per pass (a multiple of three: a ring slot's place is known at compile time).  Twelve: bfloat16 whole planes of 56 rows 18.3 -> 15.7 us
    // with two levels, but 4 to 20 % slower on small planes and short chunks.
    constexpr int U = 6;
    constexpr int PC = RAGGED ? 2 : 1;      // parameters per lane and level
    constexpr uint32_t ES = DT != DT_F32 ? 2 : 4;

    // wave -> (group of segments, chunk), lane -> (segment, column pair), segment -> (plane, column tile)
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)));
    const uint32_t group = fdiv(wave, k.div_chunks);
    const int32_t chunk = (int32_t)(wave - group * (uint32_t)k.chunks);
    const uint32_t lane = threadIdx.x & 63u, seg = fdiv(lane, k.div_pitch);
    const int32_t j = (int32_t)(lane - seg * (uint32_t)k.pitch);
    uint32_t unit = group * (uint32_t)k.spw + seg;
    bool live = j + 1 < k.pitch && seg < (uint32_t)k.spw && unit < k.units;
    unit = live ? unit : 0u;
    const uint32_t plane = fdiv(unit, k.div_tiles), img = fdiv(plane, k.div_c);
    const int32_t c = (int32_t)(plane - img * (uint32_t)k.C), w0 = (int32_t)(unit - plane * (uint32_t)k.tiles) * k.tile_w;
    const int32_t at = max(w0 - k.halo_w, 0) + 2 * j;                        // the lane's first column
    live = live && at < k.W;
    const int32_t col0 = live ? at : 0, beyond = RAGGED && live && at + 2 > k.W ? 1 : 0;  // beyond: columns of the lane behind the row's end
    const bool stores = live && at >= w0 && at < w0 + k.tile_w;

    float sc[L][PC], sh[L][PC];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const float a = k.params[k.bn[l] + c], b = k.params[k.bn[l] + k.C + c];
#pragma unroll
        for (int i = 0; i < PC; ++i) {
            const bool own = live && i + beyond < 2;
            sc[l][i] = own ? a : 0.0f;
            sh[l][i] = own ? b : 0.0f;
        }
    }

    const uint32_t pitch = (uint32_t)k.W * ES;

    const int32_t o0 = chunk * k.rc, o1 = min(o0 + k.rc, k.H);  // output rows of the chunk
    const int32_t first = max(o0 - L, 0), last = o1 - 1 + L;  // input rows (those behind the plane: padding)
    const int32_t fast_from = max(first, L), fast_to = min(k.H - 1, last);  // input rows whose step has a real row on every level
    // The first rows read and written; the others follow at 32-bit offsets (the rows of a chunk span less than 4 GiB, a float32 plane may have more).
    const size_t plane_at = (size_t)plane * (size_t)(k.H * k.W);
    const char *inp = static_cast<const char *>(image_base<DT>(k.in, img, k.in_extra)) + (plane_at + (size_t)first * (size_t)k.W + (uint32_t)(col0 - beyond)) * ES;
    char *outp = static_cast<char *>(image_base<DT>(k.out, img, k.out_extra)) + (plane_at + (size_t)o0 * (size_t)k.W + (uint32_t)col0) * ES;

    float ring[L][3][2];  // row maxima of the three newest rows of level l (level 0: the input)
#pragma unroll
    for (int l = 0; l < L; ++l)
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i) ring[l][p][i] = l == 0 ? -INFINITY : 0.0f;

    auto fetch = [&](int32_t h, ChainRow<DT> &r) __attribute__((always_inline)) {
        const char *p = inp + (uint32_t)(min(h, k.H - 1) - first) * pitch;
        __builtin_memcpy(r.w, RAGGED ? p : static_cast<const char *>(__builtin_assume_aligned(p, 2 * ES)), 2 * ES);
    };
    // one input row; P: its place in the rings.  EDGE: some levels' rows may not exist.
    auto row_step = [&](auto p_tag, auto edge_tag, float (&x)[2], int32_t h) __attribute__((always_inline)) {
        constexpr int P = decltype(p_tag)::value;
        constexpr bool EDGE = decltype(edge_tag)::value != 0;
        if constexpr (RAGGED) {
            x[0] = beyond ? x[1] : x[0];
            x[1] = beyond ? -INFINITY : x[1];
        }
        const bool real = live && (!EDGE || h < k.H);
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i] = __builtin_canonicalizef(real ? x[i] : -INFINITY);
        chain_input(x, ring[0][P]);
#pragma unroll
        for (int l = 0; l < L; ++l) {
            const bool row = !EDGE || (h >= l + 1 && h < l + 1 + k.H);  // does level l + 1 have a row h - l - 1?  Else padding.
            float a[PC], b[PC];
#pragma unroll
            for (int i = 0; i < PC; ++i) {
                a[i] = row ? sc[l][i] : 0.0f;
                b[i] = row ? sh[l][i] : 0.0f;
            }
            if (l + 1 < L) {
                if (l == 0) chain_level<DT_F32>(ring[l], a, b, ring[l + 1 < L ? l + 1 : 0][P]);
                else chain_level<DT>(ring[l], a, b, ring[l + 1 < L ? l + 1 : 0][P]);
                continue;
            }
            float v[2];
            chain_windows(ring[l], v);
            if (l > 0) round_store_all<DT, 2>(v);
#pragma unroll
            for (int i = 0; i < 2; ++i) v[i] = __builtin_fmaxf(__builtin_fmaf(v[i], a[i % PC], b[i % PC]), 0.0f);
            const int32_t r = h - L;
            if (stores && r >= o0 && (!EDGE || r < o1)) {
                char *p = outp + (uint32_t)(r - o0) * pitch;
                if (!RAGGED) {
                    store_elems<DT, 2, false>(p, 0, v);
                } else {  // at any multiple of the element size
                    uint32_t w[DT != DT_F32 ? 1 : 2];
                    if constexpr (DT == DT_F32) {
                        w[0] = __float_as_uint(v[0]);
                        w[1] = __float_as_uint(v[1]);
                    } else {
                        w[0] = pack2<DT>(v[0], v[1]);
                    }
                    if (beyond) __builtin_memcpy(p, w, ES);
                    else __builtin_memcpy(p, w, 2 * ES);
                }
            }
        }
    };

    // A row is requested U rows ahead (rows outside the plane: the nearest row inside).
    ChainRow<DT> ahead[U];
#pragma unroll
    for (int n = 0; n < U; ++n) fetch(first + n, ahead[n]);
    auto pass = [&](auto edge_tag, int32_t h0) __attribute__((always_inline)) {
        auto one = [&](auto n_tag) __attribute__((always_inline)) {
            constexpr int N = decltype(n_tag)::value;
            float x[2];
            chain_unpack<DT>(ahead[N], x);
            fetch(h0 + U + N, ahead[N]);
            row_step(IntTag<N % 3>{}, edge_tag, x, h0 + N);
        };
        one(IntTag<0>{});
        one(IntTag<1>{});
        one(IntTag<2>{});
        one(IntTag<3>{});
        one(IntTag<4>{});
        one(IntTag<5>{});
    };
    int32_t h = first;  // the same for every lane
    for (; h < fast_from; h += U) pass(IntTag<1>{}, h);
    for (; h + U - 1 <= fast_to; h += U) pass(IntTag<0>{}, h);
    for (; h <= last; h += U) pass(IntTag<1>{}, h);
}

}  // namespace bs
