// Internal helpers shared by the translation units of libmkq (host side checks,
// launch plumbing, small device utilities).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <mutex>

#include "launch_rules.h"
#include "mkq.h"

namespace mkq {

constexpr int QMIN = -8;
constexpr int QMAX = 7;

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool scale_ok(float s) { return s > 0.0f && s < __builtin_inff(); }
// Every entry point converts its stream argument here before it launches anything.  The runtime keeps the
// last error of the thread until somebody reads it: one left behind by an earlier call of the process (not
// ours, and handled or ignored there) must not be taken for a failure of our launch, so it is read away here.
inline hipStream_t as_stream(void *s)
{
    (void)hipGetLastError();
    return reinterpret_cast<hipStream_t>(s);
}
inline int launch_status() { return hipGetLastError() == hipSuccess ? MKQ_OK : MKQ_ERR_HIP; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Per-device, once-only setup values (dynamic LDS limits, resident workgroups per CU, CU counts).
// One object per kernel instantiation; get() runs `init` the first time it is called with a given
// device current and returns its (positive) result from then on; a result <= 0 is an error and is
// not cached.  Safe to call from several threads.
constexpr int MAX_DEVICES = 64;
struct PerDeviceOnce {
    std::mutex mu;
    int val[MAX_DEVICES] = {};
    template <class F>
    int get(F &&init)
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return -1;
        std::lock_guard<std::mutex> lock(mu);
        if (val[dev] <= 0) {
            const int v = init();
            if (v <= 0) return v < 0 ? v : -1;
            val[dev] = v;
        }
        return val[dev];
    }
};

// Compute units of the current device; false if the runtime cannot say.
inline bool device_cus(int *cus)
{
    static PerDeviceOnce once;
    const int v = once.get([]() -> int {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return -1;
        return n;
    });
    if (v <= 0) return false;
    *cus = v;
    return true;
}

// ---- device utilities ------------------------------------------------------

// Eq. 1, integer part, for one value: binary32 divide, clamp to the signed
// 4-bit range, round half to even.  NaN -> 0.
__device__ __forceinline__ int quantize_code(float x, float s)
{
    float v = x / s;                    // correctly rounded (no fast-math)
    v = (v != v) ? 0.0f : v;
    v = fminf(fmaxf(v, (float)QMIN), (float)QMAX);
    return (int)__builtin_rintf(v);     // v_rndne_f32
}

// The same code for many values under one step, without a division per value.  With rs = RN(1/s),
// q = RN(x * rs) differs from the exact quotient x/s by at most |x/s| * 2^-23 (two roundings), and the
// correctly rounded quotient differs from it by at most |x/s| * 2^-24; inside the clamp range that is
// less than `margin` in all.  So unless q lies within `margin` of a rounding boundary k + 1/2, the
// correctly rounded quotient rounds to the same integer (values beyond the clamp range clamp alike);
// the rare value that does lie that close takes the division.  For steps outside [2^-100, 2^100]
// (where 1/s could lose precision) the threshold is negative and every value takes the division.
struct QuantStep {
    float s, rs, thr;
};
template <int BITS>
__device__ __forceinline__ QuantStep quant_step(float s)
{
    // (covers both forms below: 1.5 * 2^-23 * 9 resp. * 129 for the plain product, 33.5 * 2^-24 resp.
    // 513.5 * 2^-24 for the biased one; rounded up)
    constexpr float margin = (BITS == 4) ? 4.0e-6f : 5.0e-5f;
    QuantStep q;
    q.s = s;
    q.rs = 1.0f / s;
    q.thr = (s >= 0x1p-100f && s <= 0x1p100f) ? 0.5f - margin : -1.0f;
    return q;
}
template <int BITS>
__device__ __forceinline__ int quantize_code_rs(float x, const QuantStep &q)
{
    constexpr float lo = (BITS == 4) ? (float)QMIN : -128.0f, hi = (BITS == 4) ? (float)QMAX : 127.0f;
    float v = x * q.rs;
    v = (v != v) ? 0.0f : v;
    v = fminf(fmaxf(v, lo), hi);
    const float r = __builtin_rintf(v);
    if (__builtin_expect(fabsf(v - r) > q.thr, 0)) {
        float w = x / q.s;
        w = (w != w) ? 0.0f : w;
        w = fminf(fmaxf(w, lo), hi);
        return (int)__builtin_rintf(w);
    }
    return (int)r;
}

// Eq. 1 at 8 bits: clamp to [-128, 127]; 8 codes as 8 bytes, element 0 lowest.
__device__ __forceinline__ int quantize_code8(float x, float s)
{
    float v = x / s;
    v = (v != v) ? 0.0f : v;
    v = fminf(fmaxf(v, -128.0f), 127.0f);
    return (int)__builtin_rintf(v);
}

__device__ __forceinline__ uint2 bytes8(const int (&c)[8])
{
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        lo |= ((uint32_t)c[i] & 0xFFu) << (8 * i);
        hi |= ((uint32_t)c[4 + i] & 0xFFu) << (8 * i);
    }
    return make_uint2(lo, hi);
}

// Eq. 1 for eight values under one step, packed as they are stored: BITS = 4 -> eight nibbles in .x (value 0
// lowest), BITS = 8 -> eight bytes in .x, .y.  Division-free as above, in a form that takes six vector
// operations per value: v = fma(x, rs, 2^(BITS-1)) is the quotient moved to [0, 2^BITS - 1] (one rounding;
// for quotients inside the clamp range it differs from the correctly rounded x / s plus the bias by less
// than `margin`), it is rounded, clamped and written into its byte by one conversion instruction, and the
// bias comes off all codes at once as a flip of their sign bits.  If any of the eight lies within `margin`
// of a rounding boundary, or is NaN or infinite (v - rint(v) is then NaN), all eight take the division.
template <int BITS>
__device__ __forceinline__ uint2 quantize8(const float (&x)[8], const QuantStep &q)
{
    constexpr float bias = (BITS == 4) ? 8.0f : 128.0f, top = (BITS == 4) ? 15.0f : 255.0f;
    uint32_t a = 0, b = 0;
    bool divide = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = __builtin_fmaf(x[e], q.rs, bias);
        const float r = __builtin_rintf(v);
        divide |= !(fabsf(v - r) <= q.thr);
        const float c = __builtin_amdgcn_fmed3f(r, 0.0f, top);
        // 4 bits: even values in the bytes of a, odd ones in b; 8 bits: values 0..3 in a, 4..7 in b
        const bool to_b = (BITS == 4) ? (e & 1) : (e >= 4);
        const unsigned at = (BITS == 4) ? (e >> 1) : (e & 3);
        if (to_b) b = __builtin_amdgcn_cvt_pk_u8_f32(c, at, b);
        else a = __builtin_amdgcn_cvt_pk_u8_f32(c, at, a);
    }
    uint2 out = (BITS == 4) ? make_uint2((a | (b << 4)) ^ 0x88888888u, 0u)
                            : make_uint2(a ^ 0x80808080u, b ^ 0x80808080u);
    if (__builtin_expect(divide, 0)) {
        int cd[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) cd[e] = (BITS == 4) ? quantize_code(x[e], q.s) : quantize_code8(x[e], q.s);
        if (BITS == 4) {
            uint32_t packed = 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) packed |= ((uint32_t)cd[e] & 0xFu) << (4 * e);
            out = make_uint2(packed, 0u);
        } else {
            out = bytes8(cd);
        }
    }
    return out;
}

// f of a lane's value and that of lane ^ OFF, for an f that does not depend on their order.  All 2 OFF lanes have to be
// active (16 for OFF = 4, where the values also have to agree between lane and lane ^ 8, as they do after a step of 8).
// Lane permutations of the vector unit: what __shfl_xor gives takes a trip through LDS, about 100 cycles, and the two
// reductions of a row's LayerNorm are ten of them one after the other.
template <int OFF, class F>
__device__ __forceinline__ float lane_pair(float v, F &&f)
{
    static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8 || OFF == 16 || OFF == 32, "a power of two within a wave");
    const unsigned u = __float_as_uint(v);
    if constexpr (OFF >= 16) {
        const auto r = OFF == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false) : __builtin_amdgcn_permlane16_swap(u, u, false, false);
        return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
    } else {
        constexpr int PERM = OFF == 1 ? 0xB1 : OFF == 2 ? 0x4E : 0x120 + OFF;  // of four lanes: 1 0 3 2, 2 3 0 1; of 16: turned by OFF
        return f(v, __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)u, PERM, 0xF, 0xF, true)));
    }
}

// Over LANES neighbouring lanes (32 or 64), from the far ones to the near ones
template <int LANES, class F>
__device__ __forceinline__ float lane_reduce(float v, F &&f)
{
    if constexpr (LANES == 64) v = lane_pair<32>(v, f);
    v = lane_pair<16>(v, f);
    v = lane_pair<8>(v, f);
    v = lane_pair<4>(v, f);
    v = lane_pair<2>(v, f);
    return lane_pair<1>(v, f);
}

struct AddF32 {
    __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct MaxF32 {
    __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
__device__ __forceinline__ float wave_max(float v) { return lane_reduce<64>(v, MaxF32()); }
__device__ __forceinline__ float wave_sum(float v) { return lane_reduce<64>(v, AddF32()); }

// A LayerNorm's sum of squares: sq and those of eight more values of the lane, FIRST: of its first eight.  Written out, because several
// kernels have the same rows at different token counts and the compiler, left to contract a * a + b * b, keeps either product exact.
template <bool FIRST>
__device__ __forceinline__ float add_squares(float sq, const float (&d)[8])
{
    sq = FIRST ? __fmaf_rn(d[0], d[0], d[1] * d[1]) : __fmaf_rn(d[1], d[1], __fmaf_rn(d[0], d[0], sq));
#pragma unroll
    for (int e = 2; e < 8; ++e) sq = __fmaf_rn(d[e], d[e], sq);
    return sq;
}

__device__ __forceinline__ float half_bits_to_float(uint16_t h)
{
    return __half2float(__ushort_as_half(h));
}

__device__ __forceinline__ uint16_t float_to_half_bits(float f)
{
    return __half_as_ushort(__float2half_rn(f));
}

// binary32 -> bfloat16, round to nearest even (NaN kept quiet)
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u) {
        if (u & 0x007FFFFFu) u |= 0x00400000u;
        return (uint16_t)(u >> 16);
    }
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// 8 consecutive elements of a binary32 / binary16 row as binary32 (16-byte aligned address).
template <typename T>
__device__ __forceinline__ void load8(const T *p, float (&v)[8]);

template <>
__device__ __forceinline__ void load8<float>(const float *p, float (&v)[8])
{
    const float4 a = *reinterpret_cast<const float4 *>(p);
    const float4 b = *reinterpret_cast<const float4 *>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

template <>
__device__ __forceinline__ void load8<__half>(const __half *p, float (&v)[8])
{
    const uint4 a = *reinterpret_cast<const uint4 *>(p);
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = half_bits_to_float((uint16_t)(w[i] & 0xFFFFu));
        v[2 * i + 1] = half_bits_to_float((uint16_t)(w[i] >> 16));
    }
}

// Two binary32 values -> two 16-bit floats in one word (low half = a), round to
// nearest even, one v_cvt_pk_* instruction each on gfx950.
typedef float mkq_f2 __attribute__((ext_vector_type(2)));
typedef __bf16 mkq_bf2 __attribute__((ext_vector_type(2)));
typedef _Float16 mkq_h2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2_bf16(float a, float b)
{
    const mkq_f2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, mkq_bf2));
}
__device__ __forceinline__ uint32_t pack2_f16(float a, float b)
{
    const mkq_f2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, mkq_h2));
}

// GELU, erf form, binary32 (activation functions stay in float32, section 5), without branches.
// gelu(x) = x Phi(x) = max(x, 0) - |x| u with u = Phi(-|x|), and log2(u) is so smooth that one polynomial of degree 8
// gives it: -1 at 0 exactly, the other coefficients a minimax fit (linear program over Chebyshev nodes, our own) of the
// error of |x| u on [0, 6.5], 1.3e-8 there; the leading one is negative, so beyond the fit u goes on falling to 0.
// What bounds the epilogues that use it is vector issue: eleven operations with one quarter-rate exponential, 56 cycles
// per value and wave.  The form before (Abramowitz & Stegun 7.1.26: reciprocal, five coefficients, exp(-x^2 / 2)) took
// thirteen with two quarter-rate ones, 76 cycles.  Evaluated in binary32 against binary64: largest error on [-10, 10] 2.5e-7
// (before 3.3e-7; most of it the rounding of results near 4), root mean square under unit Gaussian inputs 1.4e-8 (3.4e-8).
__device__ __forceinline__ float gelu_erf(float x)
{
    const float ax = fabsf(x);
    float l = __builtin_fmaf(-1.5206792360580395e-06f, ax, 2.3473889547716273e-05f);
    l = __builtin_fmaf(l, ax, -1.0947861108404527e-04f);
    l = __builtin_fmaf(l, ax, -3.2621452154775064e-04f);
    l = __builtin_fmaf(l, ax, 7.318362107740638e-03f);
    l = __builtin_fmaf(l, ax, -5.268055803436432e-02f);
    l = __builtin_fmaf(l, ax, -4.591433832864385e-01f);
    l = __builtin_fmaf(l, ax, -1.1511134697079117f);
    l = __builtin_fmaf(l, ax, -1.0f);
    const float u = __builtin_amdgcn_exp2f(l);
    // max(x, 0) as a median of three: one instruction (fmaxf first quiets its operand with a second one); a
    // NaN still reaches the result through the product
    return __builtin_fmaf(-ax, u, __builtin_amdgcn_fmed3f(x, 0.0f, __builtin_inff()));
}

// The same for results that keep small values (binary32, bfloat16).  The fit above is absolute, as fine as the steps of codes
// and of binary16 near 0 ask, but coarse relative to results below 2.5e-7 (x < -5.2): 0.7 % at x = -5.5, 9 % at -6.5, 70 % at
// -8.  Degree 12 (the same method, absolute error on [0, 5] and relative error on [5, 13.1] together) has 0.04 %, 0.13 %,
// 0.11 % there and 0.9 % at -12.8, below which u ends with the normal numbers (7.1.26: 0.25 %, 0.5 %, 1 %, 3.7 %), and an
// absolute error of 3e-9 on [-5, 0] before rounding.  16 cycles more than the form above.
__device__ __forceinline__ float gelu_erf_tail(float x)
{
    const float ax = fabsf(x);
    float l = __builtin_fmaf(-6.406064857618525e-11f, ax, 3.993946363502951e-09f);
    l = __builtin_fmaf(l, ax, -1.0693068087399058e-07f);
    l = __builtin_fmaf(l, ax, 1.6153275431240008e-06f);
    l = __builtin_fmaf(l, ax, -1.517171398074849e-05f);
    l = __builtin_fmaf(l, ax, 9.05153156689754e-05f);
    l = __builtin_fmaf(l, ax, -3.076529474177308e-04f);
    l = __builtin_fmaf(l, ax, 3.0761933375104446e-05f);
    l = __builtin_fmaf(l, ax, 6.93251821915039e-03f);
    l = __builtin_fmaf(l, ax, -5.244305172617609e-02f);
    l = __builtin_fmaf(l, ax, -4.5921737336664303e-01f);
    l = __builtin_fmaf(l, ax, -1.1511048507359467f);
    l = __builtin_fmaf(l, ax, -1.0f);
    const float u = __builtin_amdgcn_exp2f(l);
    return __builtin_fmaf(-ax, u, __builtin_amdgcn_fmed3f(x, 0.0f, __builtin_inff()));
}

}  // namespace mkq
