// The fused step of the D2Q9 lattice, its initial state and observables.
#include "step_impl.hpp"

namespace lbmmc {
template hipError_t launch_step_ns<0, 2>(const Launch&);
template hipError_t launch_step_ns<0, 3>(const Launch&);
template hipError_t launch_step_ns<0, 4>(const Launch&);
template hipError_t launch_init_lat<0>(int, const LatParams*, int, const LatParams&, const double*,
                                        const float*, float*, float*, unsigned*, hipStream_t);
template hipError_t launch_moments_lat<0>(int, const Launch&, int, float*, float*, float*, float*,
                                           float*, double*, int);
}  // namespace lbmmc
