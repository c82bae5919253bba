// Device helpers shared by the fused step kernels (general tiles and the
// structured step): compile-time lattice components, global-address-space
// pointers, a batch member's buffers.
#pragma once

#include <type_traits>
#include <utility>

#include "device.h"

namespace sdg {
namespace {

// ---- compile-time lattice components.  Velocity loops are unrolled with the
// index as a constant, so products with the components 0 and +-1 are written as
// what they are (IEEE rules forbid the compiler to drop x * 0 on its own).
constexpr int cEx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
constexpr int cEy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Device-global memory, said so explicitly.  Pointers that the compiler
// cannot trace to a kernel argument (a batched launch reads its members'
// pointers from their records) would otherwise be accessed with flat
// instructions, whose outstanding loads also hold up every wait on LDS and
// scalar results.
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
using gmem = __attribute__((address_space(1))) T;
#else
template <typename T>
using gmem = T;   // the host pass only parses device code
#endif
template <typename T>
__device__ __forceinline__ const gmem<T> *gin(const T *p)
{
    return (const gmem<T> *)p;
}
template <typename T>
__device__ __forceinline__ gmem<T> *gout(T *p)
{
    return (gmem<T> *)p;
}

// Buffers of a batch member at a launch of the given parity.
__device__ __forceinline__ DevState batch_state(const BatchInst &in, int parity)
{
    const bool sw = ((in.parity0 ^ parity) & 1) != 0;
    void *const f0 = in.f[0], *const f1 = in.f[1];
    double *const W0 = in.W[0], *const W1 = in.W[1], *const G0 = in.G[0], *const G1 = in.G[1];
    DevState s;
    s.W = sw ? W1 : W0; s.G = sw ? G1 : G0; s.Wo = sw ? W0 : W1; s.Go = sw ? G0 : G1;
    void *const fi = sw ? f1 : f0, *const fo = sw ? f0 : f1;
    s.f = reinterpret_cast<const double *>(fi);
    s.fo = reinterpret_cast<double *>(fo);
    s.f32 = reinterpret_cast<const float *>(fi);
    s.fo32 = reinterpret_cast<float *>(fo);
    return s;
}

// c x for c in {-1, 0, 1}
template <int C, typename T>
__device__ __forceinline__ T cmul(T x)
{
    if constexpr (C == 0) return T(0);
    else if constexpr (C > 0) return x;
    else return -x;
}
// a x + b y for a, b in {-1, 0, 1}, one rounding at most
template <int A, int B, typename T>
__device__ __forceinline__ T cdot(T x, T y)
{
    if constexpr (A == 0) return cmul<B>(y);
    else if constexpr (B == 0) return cmul<A>(x);
    else if constexpr (A > 0 && B > 0) return x + y;
    else if constexpr (A > 0) return x - y;
    else if constexpr (B > 0) return y - x;
    else return -(x + y);
}

}  // namespace
}  // namespace sdg
