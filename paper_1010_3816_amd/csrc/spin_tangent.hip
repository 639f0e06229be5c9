// gfx950 forward-mode derivative of the Lax-Wendroff step (arXiv:1010.3816,
// Eqs. (lw1)-(lw2) with the boundary conditions) with respect to the spin a:
// the state and its a-derivative advance together, one pass per step.
#include "adjoint_common.hpp"

namespace teuk {
namespace {

// Forward-mode derivative with respect to the spin: one step of the state,
// u^{m+1} = A u^m, and of its a-derivative v = du/da,
//   v^{m+1} = A v^m + (dA/da) u^m.
// Stage 2 is linear in the stage-1 values, so with W = S1(v) + (dS1/da) u
// (the a-derivative of the stage-1 result along the trajectory)
//   v^{m+1} = v^m - dt [D' dh/dr + D dW/dr - S'(hbar) - S(Wbar)],
// the tangent step's T with W in place of d(h) and v^m added.  The sweep,
// tiles and u^{m+1} are those of lw_tangent_kernel (bit for bit); the
// samples of u^m and v^m at the tile's (at most one) extraction point are
// fused as in the forward kernels.
template <int KEEP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
    lw_spin_tangent_kernel(const double2* __restrict__ u_in, const double2* __restrict__ v_in,
                           double2* __restrict__ u_out, double2* __restrict__ v_out, const double* __restrict__ rad,
                           const double* __restrict__ rad_da, const double* __restrict__ ang,
                           const ExtPoint* __restrict__ ext, double2* __restrict__ series_u,
                           double2* __restrict__ series_v, AdjScalars A) {
    extern __shared__ double rad_s[];
    tangent_tile<true, KEEP>(u_in, v_in, u_out, v_out, rad, rad_da, ang, ext, series_u, series_v, A, rad_s);
}

// *out += sum_i Re(conj(g_i) t_i) over count complex values (one workgroup:
// a fixed summation order, so the result does not depend on the launch).
__global__ void __launch_bounds__(256) series_dot_kernel(const double2* __restrict__ g, const double2* __restrict__ t,
                                                         int64_t count, double* __restrict__ out) {
    __shared__ double part[256];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < count; i += blockDim.x) s = fma(g[i].x, t[i].x, fma(g[i].y, t[i].y, s));
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = blockDim.x / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out += part[0];
}

}  // namespace

hipError_t launch_series_dot(const double2* g, const double2* t, int64_t count, double* out, hipStream_t s) {
    hipLaunchKernelGGL(series_dot_kernel, dim3(1), dim3(256), 0, s, g, t, count, out);
    return hipGetLastError();
}

hipError_t launch_spin_tangent(const double2* u_in, const double2* v_in, double2* u_out, double2* v_out,
                               double2* series_u, double2* series_v, const AdjArgs& a, int waves_per_block,
                               hipStream_t s) {
    dim3 grid, block;
    size_t lds;
    adjoint_launch_shape(a.k, waves_per_block, 4 * kNumSRad, &grid, &block, &lds, kTanSlots * sizeof(double2));
    hipLaunchKernelGGL(a.k.keep ? lw_spin_tangent_kernel<1> : lw_spin_tangent_kernel<0>, grid, block, lds, s, u_in,
                       v_in, u_out, v_out, a.rad, a.rad_da, a.ang, a.ext, series_u, series_v, a.k);
    return hipGetLastError();
}

}  // namespace teuk
