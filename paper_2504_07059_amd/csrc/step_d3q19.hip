// The fused step of the D3Q19 lattice for two species, its initial state and observables.
#include "step_impl.hpp"

namespace lbmmc {
template hipError_t launch_step_ns<1, 2>(const Launch&);
template hipError_t launch_init_lat<1>(int, const LatParams*, int, const LatParams&, const double*,
                                        const float*, float*, float*, unsigned*, hipStream_t);
template hipError_t launch_moments_lat<1>(int, const Launch&, int, float*, float*, float*, float*,
                                           float*, double*, int);
}  // namespace lbmmc
