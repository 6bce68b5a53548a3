// The fused step of the D3Q19 lattice for three species.
#include "step_impl.hpp"

namespace lbmmc {
template hipError_t launch_step_ns<1, 3>(const Launch&);
}  // namespace lbmmc
