// The adjoint kernels of the D3Q19 lattice.
#include "adjoint_impl.hpp"

namespace lbmmc {
template hipError_t launch_adjoint_lat<1>(int, const Launch&, const float*, float*, double*);
template hipError_t launch_adjoint_fused_lat<1>(int, const Launch&, const float*, float*,
                                                 double*);
template hipError_t launch_adjoint_stream_lat<1>(int, const Launch&, const float*, float*);
template hipError_t launch_adjoint_init_lat<1>(int, const LatParams*, const LatParams&,
                                                const double*, const float*, double*, int,
                                                hipStream_t);
}  // namespace lbmmc
