// The 1-D coefficient tables of a grid (arXiv:1010.3816, Sec. 3), one thread
// per position: the tortoise inversion by safeguarded Newton steps, the radial
// factors, their a-derivatives (dual numbers), and the angular factors.  On
// the host these took 0.8 us a position, 10.7 ms on a grid of 6400 columns
// (12,799 positions); here every position has its own thread, bound by the
// latency of one position's Newton steps (logarithm, exponential, division in
// sequence).
#include "geometry.hpp"

namespace teuk {
namespace {

// x = r - r_+ and the radial factors of both kinds of position (blockIdx.y).
// *failed becomes 1 if an inversion does not converge.
__global__ void radial_table_kernel(TableArgs A, double* __restrict__ x_tab, double* __restrict__ rad, int* failed) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, kind = blockIdx.y;
    if (i >= A.pitch) return;
    double R[kNumSRad] = {};
    double x = 0.0;
    if (i < A.nr - kind) {
        if (!tortoise_inverse(A.a, A.rmin + (i + 0.5 * kind) * A.dr, &x)) *failed = 1;
        stage_fields<double>(A.a, A.s, A.m, x, A.dth, A.d[kind], A.t[kind], R);
    }
    x_tab[(size_t)kind * A.pitch + i] = x;
    for (int f = 0; f < kNumSRad; ++f) rad[((size_t)f * 2 + kind) * A.pitch + i] = R[f];
}

// d/da of the radial factors at fixed r*, from the x of radial_table_kernel.
__global__ void radial_table_da_kernel(TableArgs A, const double* __restrict__ x_tab, double* __restrict__ da) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, kind = blockIdx.y;
    if (i >= A.pitch) return;
    Dual R[kNumSRad];
    if (i < A.nr - kind) {
        const Dual x = tortoise_x_dual(A.a, x_tab[(size_t)kind * A.pitch + i]);
        stage_fields<Dual>(Dual(A.a, 1.0), A.s, A.m, x, A.dth, A.d[kind], A.t[kind], R);
    }
    for (int f = 0; f < kNumSRad; ++f) da[((size_t)f * 2 + kind) * A.pitch + i] = R[f].d;
}

__global__ void angular_table_kernel(TableArgs A, double* __restrict__ ang) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < A.nth) angular_fields(A.s, A.m, j, A.dth, ang + (size_t)j * kNumAng);
}

}  // namespace

hipError_t launch_tables(const TableArgs& a, double* x_tab, double* rad, double* ang, int* failed, hipStream_t s) {
    if (rad != nullptr)
        hipLaunchKernelGGL(radial_table_kernel, dim3((a.pitch + 63) / 64, 2), dim3(64), 0, s, a, x_tab, rad, failed);
    hipLaunchKernelGGL(angular_table_kernel, dim3((a.nth + 63) / 64), dim3(64), 0, s, a, ang);
    return hipGetLastError();
}

hipError_t launch_tables_da(const TableArgs& a, const double* x_tab, double* da, hipStream_t s) {
    hipLaunchKernelGGL(radial_table_da_kernel, dim3((a.pitch + 63) / 64, 2), dim3(64), 0, s, a, x_tab, da);
    return hipGetLastError();
}

}  // namespace teuk
