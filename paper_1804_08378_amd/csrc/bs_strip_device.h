// Device helpers shared by the kernels whose lanes walk strips of columns (bs_strip.hip, bs_backward_strip.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "bs_device.h"

namespace bs {

template <int DT>
constexpr int elem_bytes() { return DT == DT_F32 ? 4 : 2; }

// N consecutive elements at any multiple of the element size, as they lie in memory (128-, 64-, 32- and 16-bit loads).
template <int DT, int N>
constexpr int run_words() { return (N * elem_bytes<DT>() + 3) / 4; }
template <int DT, int N>
BS_DEV void load_run(const char *p, uint32_t (&w)[run_words<DT, N>()])
{
    constexpr int BYTES = N * elem_bytes<DT>();
    constexpr int n16 = BYTES / 16, n8 = (BYTES % 16) / 8, n4 = (BYTES % 8) / 4, n2 = (BYTES % 4) / 2;
#pragma unroll
    for (int i = 0; i < n16; ++i) __builtin_memcpy(w + 4 * i, p + 16 * i, 16);
    if constexpr (n8) __builtin_memcpy(w + 4 * n16, p + 16 * n16, 8);
    if constexpr (n4) __builtin_memcpy(w + 4 * n16 + 2 * n8, p + 16 * n16 + 8 * n8, 4);
    if constexpr (n2) {
        uint16_t h;
        __builtin_memcpy(&h, p + BYTES - 2, 2);
        w[run_words<DT, N>() - 1] = h;
    }
}
template <int DT>
BS_DEV float run_element(const uint32_t *w, int i)
{
    if constexpr (DT == DT_F32) return __uint_as_float(w[i]);
    else if constexpr (DT == DT_BF16) return __uint_as_float(i % 2 ? w[i / 2] & 0xffff0000u : w[i / 2] << 16);
    else return half_up<DT>(i % 2 ? w[i / 2] >> 16 : w[i / 2] & 0xffffu);
}

// N (2 or 4) consecutive elements at any multiple of the element size.
template <int DT, int N>
BS_DEV void store_run(char *p, const float (&v)[N])
{
    if constexpr (DT == DT_F32) {
        __builtin_memcpy(p, v, 4 * N);
    } else {
        uint32_t w[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) w[i] = pack2<DT>(v[2 * i], v[2 * i + 1]);
        __builtin_memcpy(p, w, 2 * N);
    }
}

// f(integral_constant<0>), f(integral_constant<1>) ...
template <int... B, typename F>
BS_DEV void each_of(std::integer_sequence<int, B...>, F f)
{
    (f(std::integral_constant<int, B>{}), ...);
}

constexpr bool ends_in_relu(int code) { return code > 0 && ew_code_kind(code, ew_code_len(code) - 1) == OP_RELU; }

// BatchNorm, ReLU: compiled into the strip kernels.  A ReLU alone runs in those instances as well, behind a BatchNorm with scale 1
// and shift +0: x * 1 + 0 is x, but for -0, which the ReLU makes +0 in either case.
constexpr int BN_RELU = OP_BN + OP_RELU * K_EW_BASE;
inline int32_t strip_list_code(const EwOp *ew, int32_t n)
{
    if (n == 1 && ew[0].kind == OP_RELU) return BN_RELU;
    int32_t c = 0, digit = 1;
    if (n > 6) return -1;
    for (int32_t j = 0; j < n; ++j, digit *= K_EW_BASE) c += ew[j].kind * digit;
    return c;
}

// Where an element-wise operation's parameters come from: held in registers, or read at this use.  bn(): BatchNorm's scale and shift
// of V channels from `c` on; first(), second(): leaky ReLU's slope, clamp's bounds.
template <int V>
struct HeldParams {
    float a[V], b[V];
    BS_DEV void bn(float (&scale)[V], float (&shift)[V]) const
    {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            scale[e] = a[e];
            shift[e] = b[e];
        }
    }
    BS_DEV float first() const { return a[0]; }
    BS_DEV float second() const { return b[0]; }
    // of operation `kind` with argument `arg`, once per lane
    BS_DEV void load(const float *params, int32_t kind, int32_t arg, int32_t c, int32_t C)
    {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] = b[e] = 0.0f;
            if (kind == OP_BN) {
                a[e] = params[arg + c + e];
                b[e] = params[arg + C + c + e];
            } else if (kind != OP_RELU) {
                a[e] = params[arg];
                if (kind == OP_CLAMP) b[e] = params[arg + 1];
            }
        }
    }
    BS_DEV void identity()  // the BatchNorm in front of a ReLU alone
    {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] = 1.0f;
            b[e] = 0.0f;
        }
    }
};
template <int V>
struct ReadParams {
    const float *params;
    int32_t arg, c, C;
    BS_DEV void bn(float (&scale)[V], float (&shift)[V]) const
    {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            scale[e] = params[arg + c + e];
            shift[e] = params[arg + C + c + e];
        }
    }
    BS_DEV float first() const { return params[arg]; }
    BS_DEV float second() const { return params[arg + 1]; }
};

// The q-th of four values (taken by value: an index into an array would put the array into scratch memory).
BS_DEV float one_of(int32_t q, float v0, float v1, float v2, float v3)
{
    const float low = q == 0 ? v0 : v1, high = q == 2 ? v2 : v3;
    return q < 2 ? low : high;
}

// v > best: best = v, at = c.  NaN is never more; of zeros of both signs the first one stays.  Left to the compiler's
// scheduler: between a vector compare and the select that reads its lane mask gfx950 needs two wait states, which it fills with the
// neighbouring windows' work; inside an asm block nothing would.
BS_DEV void take_if_more(float v, int32_t c, float &best, int32_t &at)
{
    const bool more = v > best;
    best = more ? v : best;
    at = more ? c : at;
}
// The same where `best` only serves comparisons and derivatives, which the sign of a zero does not change: the value by the maximum
// instruction, so that a lane mask is read once.  Measured on MI355X, us, this or take_if_more: two-level backward kernel (whose masks
// then fit the scalar registers) halo_stress channels-last float32 114 / 120, bfloat16 121 / 126, binary16 113 / 121; one-level
// kernel, ResNet stem channels-last bfloat16 57.6 / 54.1, binary16 55.6 / 52.7.
BS_DEV void max_if_more(float v, int32_t c, float &best, int32_t &at)
{
    at = v > best ? c : at;
    best = __builtin_fmaxf(best, v);
}
// Row maxima of N adjacent windows (S columns apart) of window row DH: value and code 3 * DH + window column of the first
// one.  A column outside the plane holds -infinity.  Window LEAD begins one column left of the plane when `lead` is set
// (padding): its scan starts at column 1, so that a window of nothing but -infinity picks its first cell inside.  NaN is
// never a maximum.
// NONAN: no value is NaN (a ReLU stands in front).  BY_MAX: max_if_more instead of take_if_more.
template <int V, int S, int N, int CW, int DH, int LEAD, bool NONAN, bool BY_MAX = false>
BS_DEV void row_maxima(const float (&y)[CW * V], bool lead, float (&m)[N * V], int32_t (&code)[N * V])
{
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float first = NONAN ? y[b * S * V + e] : __builtin_fmaxf(y[b * S * V + e], -INFINITY);
            float best = first;
            int32_t at = LEAD == b && lead ? 3 * DH + 1 : 3 * DH;
#pragma unroll
            for (int d = 1; d < 3; ++d) {
                if constexpr (BY_MAX) max_if_more(y[(b * S + d) * V + e], 3 * DH + d, best, at);
                else take_if_more(y[(b * S + d) * V + e], 3 * DH + d, best, at);
            }
            m[b * V + e] = best;
            code[b * V + e] = at;
        }
}

// A value that is not negative (behind a ReLU: never NaN, no -0) and the order of its cell among those it is compared with, in one word that
// orders like the pair: the greatest key is the greatest value and, among equal ones, the greatest code.  Codes grow towards the first cell
// in row-major order, so a maximum of keys is the first maximum -- one instruction where a compare and two selects (with their wait
// states) take three.  16-bit storage: value bits above 16 bits of code.  float32: the value's bits above the code's in a double (at most
// 0x7f800000 above: never a NaN; the maximum keeps denormals).  Key 0: no cell.
template <int DT>
struct PickKey {
    uint32_t k;
    static constexpr int BITS = 16;
    BS_DEV static PickKey none() { return {0u}; }
    // v: rounded to the storage type
    BS_DEV static PickKey of(float v, uint32_t code)
    {
        if constexpr (DT == DT_BF16) return {__float_as_uint(v) | code};
        else return {(uint32_t)half_bits<DT>(v) << 16 | code};
    }
    BS_DEV uint32_t code() const { return k & 0xffffu; }
    BS_DEV bool positive() const { return k > 0xffffu; }
    BS_DEV float value() const { return half_up<DT>(k >> 16); }
    BS_DEV PickKey bumped(uint32_t by) const { return {k + by}; }
    BS_DEV static PickKey max(PickKey a, PickKey b) { return {a.k > b.k ? a.k : b.k}; }
    BS_DEV static PickKey choose(bool c, PickKey a, PickKey b) { return {c ? a.k : b.k}; }
};
template <>
struct PickKey<DT_F32> {
    uint32_t lo, hi;
    static constexpr int BITS = 32;
    BS_DEV static PickKey none() { return {0u, 0u}; }
    BS_DEV static PickKey of(float v, uint32_t code) { return {code, __float_as_uint(v)}; }
    BS_DEV uint32_t code() const { return lo; }
    BS_DEV bool positive() const { return hi != 0u; }
    BS_DEV float value() const { return __uint_as_float(hi); }
    BS_DEV PickKey bumped(uint32_t by) const { return {lo + by, hi}; }
    // (the instruction: fmax would first make both operands canonical)
    BS_DEV static PickKey max(PickKey a, PickKey b)
    {
        const uint64_t x = (uint64_t)a.hi << 32 | a.lo, y = (uint64_t)b.hi << 32 | b.lo;
        uint64_t d;
        asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(x), "v"(y));
        return {(uint32_t)d, (uint32_t)(d >> 32)};
    }
    BS_DEV static PickKey choose(bool c, PickKey a, PickKey b) { return {c ? a.lo : b.lo, c ? a.hi : b.hi}; }
};

// Keys of N columns x V channels (all channels of a column share its code, one less per column) from values that are not negative, rounded
// to the storage type here.
template <int DT, int V, int N>
BS_DEV void column_keys(float (&y)[N * V], uint32_t first_code, PickKey<DT> (&key)[N * V])
{
    if constexpr (DT == DT_BF16) {
        constexpr int E = N * V / 2 * 2;
#pragma unroll
        for (int i = 0; i < E; i += 2) {
            uint32_t w = pack2<DT>(y[i], y[i + 1]);
            asm("" : "+v"(w));  // one conversion for both halves
            key[i].k = w << 16 | (first_code - (uint32_t)(i / V));
            key[i + 1].k = (w & 0xffff0000u) | (first_code - (uint32_t)((i + 1) / V));
        }
        if constexpr (E < N * V) key[E] = PickKey<DT>::of(round_store<DT>(y[E]), first_code - (uint32_t)(E / V));
    } else {
#pragma unroll
        for (int i = 0; i < N * V; ++i) {
            if constexpr (DT == DT_F16) asm("" : "+v"(y[i]));  // two roundings: float32, then binary16 (round_store)
            key[i] = PickKey<DT>::of(y[i], first_code - (uint32_t)(i / V));
        }
    }
}

}  // namespace bs
