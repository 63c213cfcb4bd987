// Square-lattice pool form (many grids per launch over a tile table): the
// one-gas kernel instances (kernel templates in lb_march2d.hpp; a translation
// unit of its own so that it compiles in parallel with the plain form's).
#include "lb_march2d.hpp"

namespace lbsd {

template <typename T>
int pool2d_blocks_per_cu(bool lean, bool rest, bool species)
{
    if (species) return pool2d_blocks_per_cu_species<T>(lean, rest);
    return rest ? march_resident<T, true, false, true>(lean) : march_resident<T, false, false, true>(lean);
}

template <typename T>
hipError_t launch_pool2d(const PoolView& v, const Consts& k, int nblocks_lean, int nblocks, hipStream_t stream)
{
    if (k.species) return launch_pool2d_species<T>(v, k, nblocks_lean, nblocks, stream);
    return k.rest ? launch_pool2d_w<T, true, false>(v, k, nblocks_lean, nblocks, stream)
                          : launch_pool2d_w<T, false, false>(v, k, nblocks_lean, nblocks, stream);
}

template int pool2d_blocks_per_cu<double>(bool, bool, bool);
template int pool2d_blocks_per_cu<float>(bool, bool, bool);
template hipError_t launch_pool2d<double>(const PoolView&, const Consts&, int, int, hipStream_t);
template hipError_t launch_pool2d<float>(const PoolView&, const Consts&, int, int, hipStream_t);

}  // namespace lbsd
