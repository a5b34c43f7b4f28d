// The two-step adjoint sweeps, compiled as tile.hip is.
#include "adjoint_tile.hpp"

namespace ltne {

template <typename Lm, typename C, typename R>
hipError_t launch_adjoint2(const Adjoint2Launch& a) {
  hipLaunchKernelGGL((adjoint2_kernel<Lm, C, R>), dim3(kXcds * a.grid.per_xcd), dim3(AdjTileForm<Lm>::Block), 0,
                     a.stream, *static_cast<const StepConsts<C>*>(a.consts), static_cast<const Lm*>(a.lam_in),
                     static_cast<Lm*>(a.lam_out), static_cast<const R*>(a.rec1), static_cast<const R*>(a.rec0),
                     static_cast<const R*>(a.phi), static_cast<const R*>(a.hv), a.gphi, a.ghv, a.grid, a.lplane);
  return hipGetLastError();
}

template hipError_t launch_adjoint2<double, double, double>(const Adjoint2Launch& a);
template hipError_t launch_adjoint2<float, float, double>(const Adjoint2Launch& a);
template hipError_t launch_adjoint2<float, float, float>(const Adjoint2Launch& a);

}  // namespace ltne
