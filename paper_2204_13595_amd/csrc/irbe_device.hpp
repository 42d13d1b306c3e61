// Device-side building blocks: counter-based random numbers, bounded integers,
// wavefront/block reductions and precision traits.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace irbe {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): 10 rounds of two 32x32->64
// multiplications with the Weyl key schedule.
// ---------------------------------------------------------------------------
struct Words4 {
    uint32_t x, y, z, w;
};

__device__ __forceinline__ Words4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                           uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);  // hi1 ^ c1 ^ k0
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);  // hi0 ^ c3 ^ k1
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return {c0, c1, c2, c3};
}

// Word stream: block b = Philox({c0, b, step lo, (step hi << 1) | tag}, seed).
struct WordStream {
    uint32_t k0, k1, c0, c2, c3, block;
    Words4 buf;
    int pos;

    __device__ __forceinline__ WordStream(uint64_t seed, uint64_t step, uint32_t id, uint32_t tag)
        : k0((uint32_t)seed), k1((uint32_t)(seed >> 32)), c0(id), c2((uint32_t)step),
          c3(((uint32_t)(step >> 32) << 1) | (tag & 1u)), block(0), buf{0, 0, 0, 0}, pos(4)
    {
    }

    __device__ __forceinline__ uint32_t next()
    {
        if (pos == 4) {
            buf = philox10(c0, block, c2, c3, k0, k1);
            ++block;
            pos = 0;
        }
        const uint32_t v = pos == 0 ? buf.x : pos == 1 ? buf.y : pos == 2 ? buf.z : buf.w;
        ++pos;
        return v;
    }

    // Uniform in [0, n), n >= 1 (Lemire 2019, multiply-shift with rejection).
    __device__ __forceinline__ uint32_t below(uint32_t n)
    {
        uint64_t m = (uint64_t)next() * (uint64_t)n;
        uint32_t l = (uint32_t)m;
        if (l < n) {
            const uint32_t thr = (0u - n) % n;
            while (l < thr) {
                m = (uint64_t)next() * (uint64_t)n;
                l = (uint32_t)m;
            }
        }
        return (uint32_t)(m >> 32);
    }
};

// Workgroups are dispatched round-robin over the XCDs (8 on MI355X), each with
// its own L2. Mapping hardware block b to logical block xcd_block(b) gives every
// XCD one contiguous range of logical blocks, i.e. one compact region of the
// cell-sorted atoms, so the neighbour data an XCD reads stays in its own L2. A
// bijection of [0, nb) for any nb.
constexpr int kNumXcd = 8;

__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb)
{
    const int64_t x = b % kNumXcd, i = b / kNumXcd;
    const int64_t q = nb / kNumXcd, r = nb % kNumXcd;
    return x * q + (x < r ? x : r) + i;
}

constexpr uint32_t kTagShell = 0u;
constexpr uint32_t kTagKspace = 1u;

// Value of v in lane t (t uniform across the wavefront): v_readlane into a scalar.
__device__ __forceinline__ int bcast(int v, int t) { return __builtin_amdgcn_readlane(v, t); }
__device__ __forceinline__ uint32_t bcast(uint32_t v, int t) { return (uint32_t)__builtin_amdgcn_readlane((int)v, t); }
__device__ __forceinline__ float bcast(float v, int t)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), t));
}
__device__ __forceinline__ double bcast(double v, int t)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), t);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), t);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Position of the (k + 1)-th set bit of m (which has more than k), by the counts
// of halves of 16, 8, 4, 2 and 1 bits.
__device__ __forceinline__ int nth_set_bit(uint32_t m, uint32_t k)
{
    int b = 0;
#pragma unroll
    for (int s = 16; s >= 1; s >>= 1) {
        const uint32_t c = __popc(__builtin_amdgcn_ubfe(m, b, s));
        const bool up = k >= c;
        k -= up ? c : 0u;
        b += up ? s : 0;
    }
    return b;
}

// ---------------------------------------------------------------------------
// Reductions (fixed order: deterministic for a fixed launch shape).
// ---------------------------------------------------------------------------
// One 32-bit word of another lane: the lane 32 or 16 lanes away (the two swapped
// copies of a register hold both halves, so their sum is the butterfly's), or by
// data-parallel primitive CTRL within a row of 16.
template <int OFF>
__device__ __forceinline__ void lane_swap(uint32_t x, uint32_t& a, uint32_t& b)
{
    if constexpr (OFF == 32) {
        const auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = s[0];
        b = s[1];
    } else if constexpr (OFF == 16) {
        const auto s = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = s[0];
        b = s[1];
    } else {
        // (once the values repeat every 2 OFF lanes, rotating a row by OFF is the exchange with lane ^ OFF)
        constexpr int ctrl = OFF == 8 ? 0x128 : (OFF == 4 ? 0x124 : (OFF == 2 ? 0x4e : 0xb1));
        a = x;
        b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xf, 0xf, true);
    }
}

template <int OFF>
__device__ __forceinline__ float butterfly_add(float v)
{
    uint32_t a, b;
    lane_swap<OFF>(__float_as_uint(v), a, b);
    return __uint_as_float(a) + __uint_as_float(b);
}

template <int OFF>
__device__ __forceinline__ double butterfly_add(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    uint32_t la, lb, ha, hb;
    lane_swap<OFF>((uint32_t)u, la, lb);
    lane_swap<OFF>((uint32_t)(u >> 32), ha, hb);
    return __longlong_as_double((long long)(((unsigned long long)ha << 32) | la)) +
           __longlong_as_double((long long)(((unsigned long long)hb << 32) | lb));
}

// Sum over the wavefront in every lane: the butterfly over lane distances 32, 16,
// 8, 4, 2, 1 (the order of additions of a __shfl_xor loop, and bit for bit its
// result) in vector instructions only; a __shfl_xor is one LDS operation and its
// wait per step and 32-bit word.
template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
    v = butterfly_add<32>(v);
    v = butterfly_add<16>(v);
    v = butterfly_add<8>(v);
    v = butterfly_add<4>(v);
    v = butterfly_add<2>(v);
    return butterfly_add<1>(v);
}

// Two values at once: the first halves of each 2 OFF lanes get a's sums over the
// lane distance OFF (32 or 16), the second halves b's.
template <int OFF>
__device__ __forceinline__ float merge_add(float a, float b)
{
    const auto s = OFF == 32 ? __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false)
                             : __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

template <int OFF>
__device__ __forceinline__ double merge_add(double a, double b)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(a);
    const unsigned long long v = (unsigned long long)__double_as_longlong(b);
    const auto l = OFF == 32 ? __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)v, false, false)
                             : __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)v, false, false);
    const auto h =
        OFF == 32 ? __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(v >> 32), false, false)
                  : __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(v >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0])) +
           __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

// Four sums over the wavefront, each bit for bit wave_sum's: that of v0 in the first
// row of 16 lanes, of v1 in the second, of v2 in the third, of v3 in the fourth. One
// tree instead of four: 15 vector instructions in FP32 where four take 56.
template <typename T>
__device__ __forceinline__ T wave_sum4(T v0, T v1, T v2, T v3)
{
    T v = merge_add<16>(merge_add<32>(v0, v2), merge_add<32>(v1, v3));
    v = butterfly_add<8>(v);
    v = butterfly_add<4>(v);
    v = butterfly_add<2>(v);
    return butterfly_add<1>(v);
}

// Sums NV values per thread over a block of BLOCK threads; thread v < NV of the
// block receives total v in the return value (others: 0). lds: NV * (BLOCK/64).
template <int NV, int BLOCK>
__device__ __forceinline__ double block_sum_vec(double* vals, double* lds, int v_out_idx, double& out)
{
    constexpr int NW = BLOCK / 64;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const double s = wave_sum(vals[v]);
        if (lane == 0) lds[v * NW + wave] = s;
    }
    __syncthreads();
    out = 0.0;
    if (v_out_idx < NV) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) t += lds[v_out_idx * NW + w];
        out = t;
    }
    __syncthreads();
    return out;
}

// ---------------------------------------------------------------------------
// Precision traits.
// ---------------------------------------------------------------------------
template <typename real>
struct Math;

template <>
struct Math<float> {
    static __device__ __forceinline__ float max_() { return 3.402823466e38f; }
    // exp(x^2) erfc(x) for x = bx r >= 0, given kx = 0.45 bx: t P(t) with t = 1 / (1 + 0.45 x) and P of degree 9,
    // fitted for the least largest relative error (4.1e-8; evaluated in FP32 2.4e-7 at
    // most and 6.3e-8 RMS over 0..6, against the FP64 function).
    static __device__ __forceinline__ float erfcx_(float kx, float r)
    {
        const float t = __builtin_amdgcn_rcpf(fmaf(kx, r, 1.0f));
        float p = -0.0404629376f;
        p = fmaf(p, t, 0.186647444f);
        p = fmaf(p, t, -0.29324348f);
        p = fmaf(p, t, 0.135188052f);
        p = fmaf(p, t, -0.0181984669f);
        p = fmaf(p, t, 0.118523407f);
        p = fmaf(p, t, 0.175533885f);
        p = fmaf(p, t, 0.228242367f);
        p = fmaf(p, t, 0.253884472f);
        p = fmaf(p, t, 0.253885299f);
        return t * p;
    }
    // erfc(x) for x >= 0 given ex = exp(-x^2): the Chebyshev-fitted form of
    // Numerical Recipes (Press et al., Sec. 6.2, "erfcc"), fractional error
    // below 1.2e-7: erfc(x) = t exp(-x^2 + P(t)), t = 1/(1 + x/2).
    static __device__ __forceinline__ float erfc_ex(float x, float ex)
    {
        const float t = __builtin_amdgcn_rcpf(fmaf(0.5f, x, 1.0f));
        float p = 0.17087277f;
        p = fmaf(p, t, -0.82215223f);
        p = fmaf(p, t, 1.48851587f);
        p = fmaf(p, t, -1.13520398f);
        p = fmaf(p, t, 0.27886807f);
        p = fmaf(p, t, -0.18628806f);
        p = fmaf(p, t, 0.09678418f);
        p = fmaf(p, t, 0.37409196f);
        p = fmaf(p, t, 1.00002368f);
        p = fmaf(p, t, -1.26551223f);
        return t * ex * __expf(p);
    }
    static __device__ __forceinline__ float exp_(float x) { return __expf(x); }
    // exp(-x^2) given x and -x^2 log2(e)
    static __device__ __forceinline__ float gauss_(float, float cx2) { return __builtin_amdgcn_exp2f(cx2); }
    static __device__ __forceinline__ float erf_(float x) { return erff(x); }
    // the hardware reciprocal square root: the arguments are squared pair
    // separations, far from the denormal range that rsqrtf rescales for
    static __device__ __forceinline__ float rsqrt_(float x) { return __builtin_amdgcn_rsqf(x); }
    static __device__ __forceinline__ float sqrt_(float x) { return sqrtf(x); }
    // sin and cos of 2 pi x for a phase x in revolutions, |x| <= 1/2.
    static __device__ __forceinline__ void sincos_rev(float x, float* s, float* c)
    {
        *s = __builtin_amdgcn_sinf(x);
        *c = __builtin_amdgcn_cosf(x);
    }
};

template <>
struct Math<double> {
    static __device__ __forceinline__ double max_() { return 1.7976931348623157e308; }
    static __device__ __forceinline__ double erfc_ex(double x, double) { return erfc(x); }
    static __device__ __forceinline__ double exp_(double x) { return exp(x); }
    static __device__ __forceinline__ double gauss_(double x, double) { return exp(-x * x); }
    static __device__ __forceinline__ double erf_(double x) { return erf(x); }
    static __device__ __forceinline__ double rsqrt_(double x) { return rsqrt(x); }
    static __device__ __forceinline__ double sqrt_(double x) { return sqrt(x); }
    static __device__ __forceinline__ void sincos_rev(double x, double* s, double* c) { sincospi(2.0 * x, s, c); }
};

// Exact k.r phase: (m . s) mod 2^32, returned in revolutions in [-1/2, 1/2).
// (24-bit products of the low parts and a byte dot product of the high ones give the
// same bits but measured 10-25 % slower in every kernel here.)
template <typename real>
__device__ __forceinline__ real phase_rev(int mx, int my, int mz, uint32_t sx, uint32_t sy, uint32_t sz)
{
    const uint32_t ph = (uint32_t)mx * sx + (uint32_t)my * sy + (uint32_t)mz * sz;
    return (real)(int32_t)ph * (real)2.3283064365386963e-10;  // 2^-32
}

}  // namespace irbe
