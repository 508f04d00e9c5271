// Cross-lane sums by DPP row operations, shared by the reductions of the
// backward and learning-step kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace dpd {

// One DPP step of a lane reduction: x from the lane that CTRL selects (rows
// outside RMASK read zero).
template <int CTRL, int RMASK>
__device__ __forceinline__ float dpp_from(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, RMASK, 0xf, false));
}

// The same for FP64 values: each half of the double moved by its own DPP
// step (rows outside RMASK read zero, i.e. +0.0).
template <int CTRL, int RMASK>
__device__ __forceinline__ double dpp_from(double x)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, RMASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, RMASK, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Sum over the 64 lanes, complete in lane 63 (the other lanes hold partial
// sums), by DPP row operations -- no LDS round trips: quad sums (quad_perm
// 1,0,3,2 and 2,3,0,1), 8- and 16-lane sums (row_half_mirror, row_mirror),
// then rows 1 and 3 add rows 0 and 2 (row_bcast:15) and rows 2 and 3 add the
// sum of rows 0..1 (row_bcast:31).  Fixed order: the same inputs give the
// same bits.
template <class T>
__device__ __forceinline__ T wave_sum_to_lane63(T v)
{
    v += dpp_from<0xB1, 0xf>(v);
    v += dpp_from<0x4E, 0xf>(v);
    v += dpp_from<0x141, 0xf>(v);
    v += dpp_from<0x140, 0xf>(v);
    v += dpp_from<0x142, 0xa>(v);
    v += dpp_from<0x143, 0xc>(v);
    return v;
}

// a + b with the upper half of a's lanes (of each 2 O lanes) and the lower half
// of b's exchanged first: lanes whose bit O is clear get a summed over that bit,
// the others b.
template <int O>
__device__ __forceinline__ void half_swap(unsigned &x, unsigned &y)
{
    static_assert(O == 32 || O == 16, "the widths of the exchange instructions");
    if constexpr (O == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    }
}
template <int O>
__device__ __forceinline__ float swap_add(float a, float b)
{
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    half_swap<O>(x, y);
    return __uint_as_float(x) + __uint_as_float(y);
}
template <int O>
__device__ __forceinline__ double swap_add(double a, double b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    unsigned al = (unsigned)ua, ah = (unsigned)(ua >> 32), bl = (unsigned)ub, bh = (unsigned)(ub >> 32);
    half_swap<O>(al, bl);
    half_swap<O>(ah, bh);
    return __longlong_as_double((long long)(((unsigned long long)ah << 32) | al)) +
           __longlong_as_double((long long)(((unsigned long long)bh << 32) | bl));
}

// The same over 16 lanes and less: each lane keeps the value that its bit O
// selects and adds the copy of lane l ^ O (l ^ 4 by two exchanges, l ^ 7 ^ 3).
template <int O, class T>
__device__ __forceinline__ T keep_add(T a, T b, int lane)
{
    const bool up = (lane & O) != 0;
    T v = up ? a : b;
    if constexpr (O == 8) v = dpp_from<0x128, 0xf>(v);                           // row_ror:8
    if constexpr (O == 4) v = dpp_from<0x1B, 0xf>(dpp_from<0x141, 0xf>(v));      // row_half_mirror, quad_perm 3,2,1,0
    if constexpr (O == 2) v = dpp_from<0x4E, 0xf>(v);                            // quad_perm 2,3,0,1
    if constexpr (O == 1) v = dpp_from<0xB1, 0xf>(v);                            // quad_perm 1,0,3,2
    return (up ? b : a) + v;
}

// N <= 64 per-lane FP32 values summed over the wave in T (float or double),
// transposed: lane l returns the sum of v[l] over all 64 lanes (zero for l >= N).
// Six butterfly stages, each halving the values still held: a lane keeps the one
// that its lane bit selects and adds its partner's copy.  No LDS.  Fixed order:
// the same inputs give the same bits.
template <class T, int N>
__device__ __forceinline__ T wave_transpose_sum(const float *v, int lane)
{
    static_assert(N >= 1 && N <= 64, "one register per lane and group");
    const auto at = [&](int e) { return e < N ? (T)v[e] : (T)0; };
    T a[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const T x = i < N ? swap_add<32>(at(i), at(i + 32)) : (T)0;
        const T y = i + 16 < N ? swap_add<32>(at(i + 16), at(i + 48)) : (T)0;
        a[i] = i < N ? swap_add<16>(x, y) : (T)0;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = keep_add<8>(a[i], a[i + 8], lane);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = keep_add<4>(a[i], a[i + 4], lane);
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = keep_add<2>(a[i], a[i + 2], lane);
    return keep_add<1>(a[0], a[1], lane);
}

// Calls f(std::integral_constant<int, G>) for G = 0 .. NG-1.
template <int G, int NG>
struct ForEachGroup {
    template <class F>
    __device__ __forceinline__ static void run(F &f)
    {
        f(std::integral_constant<int, G>{});
        ForEachGroup<G + 1, NG>::run(f);
    }
};
template <int NG>
struct ForEachGroup<NG, NG> {
    template <class F>
    __device__ __forceinline__ static void run(F &)
    {
    }
};

// The wave sums of E per-lane accumulators, formed in T, added to FP64 totals
// held transposed (entry 64 g + l in lane l of tot[g]).
template <class T, int E>
__device__ __forceinline__ void wave_sums_into(const float (&acc)[E], double (&tot)[(E + 63) / 64], int lane)
{
    auto one = [&](auto gc) {
        constexpr int g = decltype(gc)::value;
        constexpr int n = E - 64 * g < 64 ? E - 64 * g : 64;
        tot[g] += (double)wave_transpose_sum<T, n>(&acc[64 * g], lane);
    };
    ForEachGroup<0, (E + 63) / 64>::run(one);
}

}  // namespace dpd
