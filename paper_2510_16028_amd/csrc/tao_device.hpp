// Device-side helpers shared by the gfx950 kernels of the tolerance engine.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace tao {

constexpr int kWave = 64;

// Smallest binary32 value >= v, for v >= 0 (NaN and +inf pass through).  The
// conversion itself rounds to nearest; one step up repairs a round-down.
__device__ __forceinline__ float up32(double v) {
    float f = (float)v;
    if ((double)f < v) f = __uint_as_float(__float_as_uint(f) + 1u);
    return f;
}

// Cheaper upper rounding for the streaming kernels, which also takes the place of the guard
// factor: for v >= 0 the result is a binary32 value >= v (1 + m) and at most one binary32 step
// above the smallest such value, where m is the rounding margin the caller asks for.
//  - Normal results: with mul = 1 + 2^-24 + 2m the product v mul lies above the midpoint of the
//    binary32 neighbours of v (1 + m) (their distance is at most 2^-23 of the lower one), so the
//    conversion's round-to-nearest lands on the upper neighbour or beyond: no compare, no step.
//  - Results below 2^-126 (subnormal, or zero): the spacing is absolute there and one step is a
//    large relative amount, so v (1 + m) is rounded up exactly (sub = 1 + m): the result is the
//    smallest representable value >= v sub, and 0 stays 0.
// The defaults serve the element-wise kernels (a handful of binary64 roundings and, for GELU, an
// exponential accurate to 2^-40); the row kernels pass constants that grow with the row length.
// NaN and +inf pass through.
constexpr double kUpMul = 1.0 + 0x1p-24 + 0x1p-32;
constexpr double kUpSub = 1.0 + 0x1p-36;
__device__ __forceinline__ float up32g(double v, double mul = kUpMul, double sub = kUpSub) {
    float f = (float)(v * mul);
    if (f < 0x1p-126f) {
        const double w = v * sub;
        f = (float)w;
        if ((double)f < w) f = __uint_as_float(__float_as_uint(f) + 1u);
    }
    return f;
}

// Reductions over the 64 lanes, the result in every lane: four exchanges inside rows of 16 lanes (quads, halves, rows: data-parallel
// moves), then rows and halves of the wavefront swapped -- register moves throughout, where a shuffle through LDS takes some hundred
// cycles a step (LayerNorm of 512 x 768 with its check: see rowops.hip).  Each step combines what two groups of lanes hold in
// an order that is the same for both, so all lanes get the same bits.
template <int STEP>
__device__ __forceinline__ void lane_pair(unsigned v, unsigned& a, unsigned& b) {
    typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
    a = v;
    if constexpr (STEP == 0)      b = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, true);      // quad_perm 1,0,3,2
    else if constexpr (STEP == 1) b = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, true);      // quad_perm 2,3,0,1
    else if constexpr (STEP == 2) b = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true);     // row_half_mirror
    else if constexpr (STEP == 3) b = (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xf, 0xf, true);     // row_mirror
    else {
        const uintx2 r = STEP == 4 ? __builtin_amdgcn_permlane16_swap(v, v, false, false) : __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = r[0]; b = r[1];
    }
}
template <int STEP, class T>
__device__ __forceinline__ void lane_pair(T v, T& a, T& b) {
    if constexpr (sizeof(T) == 4) {
        unsigned x, y;
        lane_pair<STEP>(__builtin_bit_cast(unsigned, v), x, y);
        a = __builtin_bit_cast(T, x); b = __builtin_bit_cast(T, y);
    } else {
        const unsigned long long w = __builtin_bit_cast(unsigned long long, v);
        unsigned xl, yl, xh, yh;
        lane_pair<STEP>((unsigned)w, xl, yl);
        lane_pair<STEP>((unsigned)(w >> 32), xh, yh);
        a = __builtin_bit_cast(T, (unsigned long long)xh << 32 | xl);
        b = __builtin_bit_cast(T, (unsigned long long)yh << 32 | yl);
    }
}
template <int FIRST = 0, int STEPS = 6, class T, class Op>
__device__ __forceinline__ T wave_all(T v, Op op) {
    if constexpr (FIRST < STEPS) {
        T a, b;
        lane_pair<FIRST>(v, a, b);
        return wave_all<FIRST + 1, STEPS>(op(a, b), op);
    } else {
        return v;
    }
}
template <class T>
__device__ __forceinline__ T wave_sum(T v) { return wave_all(v, [](T a, T b) { return a + b; }); }
template <class T>
__device__ __forceinline__ T wave_max(T v) { return wave_all(v, [](T a, T b) { return a > b ? a : b; }); }
__device__ __forceinline__ float wave_max(float v) { return wave_all(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ int wave_or(int v) { return wave_all(v, [](int a, int b) { return a | b; }); }
// Sum over the lanes up to this one, of 32 or 64 bits.
template <class T>
__device__ __forceinline__ T wave_scan(T v) {
    static_assert(std::is_same<T, unsigned>::value || std::is_same<T, unsigned long long>::value, "one or two words");
    auto step = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
        const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, ctrl.value, rows.value, 0xf, false);
        if constexpr (sizeof(T) == 8) {
            const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), ctrl.value, rows.value, 0xf, false);
            v += (T)hi << 32 | lo;
        } else {
            v += lo;
        }
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});       // row_shr 1, 2, 4, 8
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});       // last lane of a row to the next, rows 1 and 3
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});       // last lane of the lower half to the upper
    return v;
}

// Streaming 16-byte load: the data is used once, so it is marked non-temporal.
__device__ __forceinline__ float4 ntload4(const float4* p) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f v = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

// Streaming 16-byte store of data that is not read again by this kernel.
__device__ __forceinline__ void ntstore4(float4* p, float4 v) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<v4f*>(p));
}

// 16-byte global load when the caller has established alignment, else four
// guarded scalar loads; elements at or beyond `limit` read as `fill`.
// STREAM: the data is read once by the kernel (non-temporal load).
template <bool STREAM = false>
__device__ __forceinline__ float4 load4(const float* __restrict__ p, long idx, long limit,
                                        bool vec_ok, float fill) {
    float4 r;
    if (vec_ok && idx + 3 < limit) {
        r = STREAM ? ntload4(reinterpret_cast<const float4*>(p + idx))
                   : *reinterpret_cast<const float4*>(p + idx);
    } else {
        r.x = (idx + 0 < limit) ? p[idx + 0] : fill;
        r.y = (idx + 1 < limit) ? p[idx + 1] : fill;
        r.z = (idx + 2 < limit) ? p[idx + 2] : fill;
        r.w = (idx + 3 < limit) ? p[idx + 3] : fill;
    }
    return r;
}
__device__ __forceinline__ void store4(float* __restrict__ p, long idx, long limit, bool vec_ok,
                                       float4 v) {
    if (vec_ok && idx + 3 < limit) {
        ntstore4(reinterpret_cast<float4*>(p + idx), v);      // bounds are written once, never re-read here
    } else {
        if (idx + 0 < limit) p[idx + 0] = v.x;
        if (idx + 1 < limit) p[idx + 1] = v.y;
        if (idx + 2 < limit) p[idx + 2] = v.z;
        if (idx + 3 < limit) p[idx + 3] = v.w;
    }
}

}  // namespace tao
