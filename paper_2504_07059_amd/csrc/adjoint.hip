// Adjoint launchers: dispatch on the lattice to the kernels compiled in
// adjoint_d2q9.hip and adjoint_d3q19.hip, and the fixed-order FP64 sum of the
// gradient partials.
#include <hip/hip_runtime.h>

#include "common.hpp"

namespace lbmmc {

template <int LAT>
hipError_t launch_adjoint_lat(int ns, const Launch& L, const float* lam_in, float* mu,
                              double* gpart);
template <int LAT>
hipError_t launch_adjoint_fused_lat(int ns, const Launch& L, const float* mu_in, float* mu_out,
                                    double* gpart);
template <int LAT>
hipError_t launch_adjoint_stream_lat(int ns, const Launch& L, const float* mu, float* lam_out);
template <int LAT>
hipError_t launch_adjoint_init_lat(int ns, const LatParams* lp, const LatParams& h,
                                   const double* x0, const float* lam0, double* gpart,
                                   int nblocks, hipStream_t s);

extern template hipError_t launch_adjoint_lat<0>(int, const Launch&, const float*, float*,
                                                  double*);
extern template hipError_t launch_adjoint_fused_lat<0>(int, const Launch&, const float*, float*,
                                                        double*);
extern template hipError_t launch_adjoint_stream_lat<0>(int, const Launch&, const float*, float*);
extern template hipError_t launch_adjoint_init_lat<0>(int, const LatParams*, const LatParams&,
                                                       const double*, const float*, double*, int,
                                                       hipStream_t);
extern template hipError_t launch_adjoint_lat<1>(int, const Launch&, const float*, float*,
                                                  double*);
extern template hipError_t launch_adjoint_fused_lat<1>(int, const Launch&, const float*, float*,
                                                        double*);
extern template hipError_t launch_adjoint_stream_lat<1>(int, const Launch&, const float*, float*);
extern template hipError_t launch_adjoint_init_lat<1>(int, const LatParams*, const LatParams&,
                                                       const double*, const float*, double*, int,
                                                       hipStream_t);

hipError_t launch_adjoint(int lattice, int ns, const Launch& L, const float* lam_in, float* mu,
                          double* gpart, int) {
    return lattice == 0 ? launch_adjoint_lat<0>(ns, L, lam_in, mu, gpart)
                        : launch_adjoint_lat<1>(ns, L, lam_in, mu, gpart);
}

hipError_t launch_adjoint_fused(int lattice, int ns, const Launch& L, const float* mu_in,
                                float* mu_out, double* gpart) {
    return lattice == 0 ? launch_adjoint_fused_lat<0>(ns, L, mu_in, mu_out, gpart)
                        : launch_adjoint_fused_lat<1>(ns, L, mu_in, mu_out, gpart);
}

hipError_t launch_adjoint_stream(int lattice, int ns, const Launch& L, const float* mu,
                                 float* lam_out) {
    return lattice == 0 ? launch_adjoint_stream_lat<0>(ns, L, mu, lam_out)
                        : launch_adjoint_stream_lat<1>(ns, L, mu, lam_out);
}

hipError_t launch_adjoint_init(int lattice, int ns, const LatParams* lp, const LatParams& h,
                               const double* x0, const float* lam0, double* gpart, int nblocks,
                               hipStream_t s) {
    return lattice == 0 ? launch_adjoint_init_lat<0>(ns, lp, h, x0, lam0, gpart, nblocks, s)
                        : launch_adjoint_init_lat<1>(ns, lp, h, x0, lam0, gpart, nblocks, s);
}

// Fixed-order sum of the per-block partials (one work-group of 256 threads:
// thread t takes blocks t, t+256, ...; then a fixed shuffle and LDS tree), with
// d/dK converted to d/dD (dK_ij/dD_ij = 6 M_i M_j), added into grad.
__global__ void __launch_bounds__(256) k_grad_reduce(const LatParams* __restrict__ lps,
                                                     const double* __restrict__ gpart,
                                                     int nblocks, int ng, int ns,
                                                     double* __restrict__ grad) {
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int npair = ns * (ns - 1) / 2;
    for (int q = 0; q < ng; ++q) {
        double v = 0.0;
        for (int b = tid; b < nblocks; b += 256) v += gpart[(int64_t)b * ng + q];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) red[wave] = v;
        __syncthreads();
        if (tid == 0) {
            double s = (red[0] + red[1]) + (red[2] + red[3]);
            if (q < npair) {
                int k = 0;
                for (int i = 0; i < ns; ++i)
                    for (int j = i + 1; j < ns; ++j, ++k)
                        if (k == q) s *= lps[0].dscale[i][j];
            }
            grad[q] += s;
        }
        __syncthreads();
    }
}

hipError_t launch_grad_reduce(const LatParams* lp, const double* gpart, int nblocks, int ng,
                              int ns, double* grad, hipStream_t s) {
    hipLaunchKernelGGL(k_grad_reduce, dim3(1), dim3(256), 0, s, lp, gpart, nblocks, ng, ns, grad);
    return hipGetLastError();
}

}  // namespace lbmmc
