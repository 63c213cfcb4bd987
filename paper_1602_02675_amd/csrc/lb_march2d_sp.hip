// Square-lattice step as a column march with two gases: the plain form's
// instances that carry the species moment rho chi.  The kernel templates are
// in lb_march2d.hpp; the instances are spread over translation units of their
// own (lb_march2d.hip, lb_pool2d.hip, lb_pool2d_sp.hip) that compile in
// parallel.
#include "lb_march2d.hpp"

namespace lbsd {

template <typename T>
int march2d_blocks_per_cu_species(bool lean, bool rest)
{
    return rest ? march_resident<T, true, true, false>(lean) : march_resident<T, false, true, false>(lean);
}
template int march2d_blocks_per_cu_species<double>(bool, bool);
template int march2d_blocks_per_cu_species<float>(bool, bool);

template <typename T>
hipError_t launch_march2d_species(const T* Y, T* Yn, const Grid& g, const MarchGeom& m, const Consts& k,
                                  StepCtl* ctl, double* partials, const MarchWords& w, long long step,
                                  hipStream_t stream)
{
    return k.rest ? launch_march2d_w<T, true, true>(Y, Yn, g, m, k, ctl, partials, w, step, stream)
                          : launch_march2d_w<T, false, true>(Y, Yn, g, m, k, ctl, partials, w, step, stream);
}

template <typename T>
hipError_t launch_lanes_species(const T* Y, const Grid& g, const Consts& k, int32_t* fx, int32_t* fy, int32_t* c1,
                                hipStream_t stream)
{
    return k.rest ? launch_lanes_w<T, true, true>(Y, g, k, fx, fy, c1, stream)
                          : launch_lanes_w<T, false, true>(Y, g, k, fx, fy, c1, stream);
}

template hipError_t launch_lanes_species<double>(const double*, const Grid&, const Consts&, int32_t*, int32_t*,
                                                 int32_t*, hipStream_t);
template hipError_t launch_lanes_species<float>(const float*, const Grid&, const Consts&, int32_t*, int32_t*, int32_t*,
                                                hipStream_t);
template hipError_t launch_march2d_species<double>(const double*, double*, const Grid&, const MarchGeom&,
                                                   const Consts&, StepCtl*, double*, const MarchWords&, long long,
                                                   hipStream_t);
template hipError_t launch_march2d_species<float>(const float*, float*, const Grid&, const MarchGeom&,
                                                  const Consts&, StepCtl*, double*, const MarchWords&, long long,
                                                  hipStream_t);

}  // namespace lbsd
