// Square-lattice pool form with two gases: the pool kernels' instances that
// carry the species moment rho chi (kernel templates in lb_march2d.hpp; a
// translation unit of its own so that it compiles in parallel).
#include "lb_march2d.hpp"

namespace lbsd {

template <typename T>
int pool2d_blocks_per_cu_species(bool lean, bool rest)
{
    return rest ? march_resident<T, true, true, true>(lean) : march_resident<T, false, true, true>(lean);
}
template int pool2d_blocks_per_cu_species<double>(bool, bool);
template int pool2d_blocks_per_cu_species<float>(bool, bool);

template <typename T>
hipError_t launch_pool2d_species(const PoolView& v, const Consts& k, int nblocks_lean, int nblocks,
                                 hipStream_t stream)
{
    return k.rest ? launch_pool2d_w<T, true, true>(v, k, nblocks_lean, nblocks, stream)
                          : launch_pool2d_w<T, false, true>(v, k, nblocks_lean, nblocks, stream);
}

template hipError_t launch_pool2d_species<double>(const PoolView&, const Consts&, int, int, hipStream_t);
template hipError_t launch_pool2d_species<float>(const PoolView&, const Consts&, int, int, hipStream_t);

}  // namespace lbsd
