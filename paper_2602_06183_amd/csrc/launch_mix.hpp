// Launches of the tile kernels.  A unit is one contraction: a device function over (LDS, workgroup id, number of workgroups, arguments) with its
// thread count and LDS size.  launch_units puts one unit, or several independent ones of the same thread count, into a single launch: the
// workgroups of the first unit come first, so units are listed by the length of their tiles.
#pragma once
#include <hip/hip_runtime.h>

namespace sffn {

constexpr int lds_max(int a, int b) { return a > b ? a : b; }

template <class U>
__global__ void __launch_bounds__(U::THREADS, U::THREADS == 256 && U::LDS > 80 * 1024 ? 1 : U::THREADS < 256 ? 1 : 2) unit_kernel(typename U::Args a) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[U::LDS];
    U::run(smem, blockIdx.x, gridDim.x, a);
}
template <class U>
hipError_t launch_units(hipStream_t s, const typename U::Args& args) {
    const unsigned n = U::count(args);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL((unit_kernel<U>), dim3(n), dim3(U::THREADS), 0, s, U::args(args));
    return hipGetLastError();
}

// Two or three units in one launch, the workgroups of the first unit first or, `swap`, those of the second before them: units are listed by the length of their
// tiles, which can depend on sizes.  Every unit's range of workgroups starts at a multiple of 8 (s0, s1, s2), so that a unit's own workgroup ids still say
// which XCD they run on.
constexpr unsigned round8(unsigned n) { return (n + 7) & ~7u; }
template <class U0, class U1>
__global__ void __launch_bounds__(U0::THREADS, lds_max(U0::LDS, U1::LDS) > 80 * 1024 ? 1 : 2)
    unit_kernel2(typename U0::Args a0, typename U1::Args a1, int n0, int n1, int s0, int s1) {
    static_assert(U0::THREADS == U1::THREADS, "units of one launch have the same workgroup size");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[lds_max(U0::LDS, U1::LDS)];
    const int p0 = (int)blockIdx.x - s0, p1 = (int)blockIdx.x - s1;
    if (p0 >= 0 && p0 < n0) U0::run(smem, p0, n0, a0);
    else if (p1 >= 0 && p1 < n1) U1::run(smem, p1, n1, a1);
}
template <class U0, class U1>
hipError_t launch_units(hipStream_t s, const typename U0::Args& a0, const typename U1::Args& a1, bool swap = false) {
    const unsigned n0 = U0::count(a0), n1 = U1::count(a1);
    if (n0 + n1 == 0) return hipSuccess;
    const unsigned s0 = swap ? round8(n1) : 0, s1 = swap ? 0 : round8(n0);
    hipLaunchKernelGGL((unit_kernel2<U0, U1>), dim3(swap ? s0 + n0 : s1 + n1), dim3(U0::THREADS), 0, s, U0::args(a0), U1::args(a1), (int)n0, (int)n1, (int)s0, (int)s1);
    return hipGetLastError();
}
template <class U0, class U1, class U2>
__global__ void __launch_bounds__(U0::THREADS, lds_max(U0::LDS, lds_max(U1::LDS, U2::LDS)) > 80 * 1024 ? 1 : 2)
    unit_kernel3(typename U0::Args a0, typename U1::Args a1, typename U2::Args a2, int n0, int n1, int n2, int s0, int s1, int s2) {
    static_assert(U0::THREADS == U1::THREADS && U0::THREADS == U2::THREADS, "units of one launch have the same workgroup size");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[lds_max(U0::LDS, lds_max(U1::LDS, U2::LDS))];
    const int p0 = (int)blockIdx.x - s0, p1 = (int)blockIdx.x - s1, p2 = (int)blockIdx.x - s2;
    if (p0 >= 0 && p0 < n0) U0::run(smem, p0, n0, a0);
    else if (p1 >= 0 && p1 < n1) U1::run(smem, p1, n1, a1);
    else if (p2 >= 0 && p2 < n2) U2::run(smem, p2, n2, a2);
}
template <class U0, class U1, class U2>
hipError_t launch_units(hipStream_t s, const typename U0::Args& a0, const typename U1::Args& a1, const typename U2::Args& a2, bool swap = false) {
    const unsigned n0 = U0::count(a0), n1 = U1::count(a1), n2 = U2::count(a2);
    if (n0 + n1 + n2 == 0) return hipSuccess;
    const unsigned s0 = swap ? round8(n1) : 0, s1 = swap ? 0 : round8(n0), s2 = round8(n0) + round8(n1);
    hipLaunchKernelGGL((unit_kernel3<U0, U1, U2>), dim3(s2 + n2), dim3(U0::THREADS), 0, s, U0::args(a0), U1::args(a1), U2::args(a2), (int)n0, (int)n1, (int)n2,
                       (int)s0, (int)s1, (int)s2);
    return hipGetLastError();
}

}  // namespace sffn
