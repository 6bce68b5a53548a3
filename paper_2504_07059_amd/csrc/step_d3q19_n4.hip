// The fused step of the D3Q19 lattice for four species.
#include "step_impl.hpp"

namespace lbmmc {
template hipError_t launch_step_ns<1, 4>(const Launch&);
}  // namespace lbmmc
