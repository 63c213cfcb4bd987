// Square-lattice step as a column march: the one-gas instances of the plain
// form and the launch geometry (the kernel templates and how the march works
// are in lb_march2d.hpp; the pool form's one-gas instances are in
// lb_pool2d.hip, the two-gas instances in lb_march2d_sp.hip and
// lb_pool2d_sp.hip).
#include <algorithm>

#include "lb_march2d.hpp"

namespace lbsd {

namespace {

int64_t x_strips(const Grid& g) { return (g.nx + kMCols - 1) / kMCols; }

// Smallest strip height.  A lean tile marches 4 halo rows besides its own (a
// general one 10), so low strips repeat work; but a small grid leaves most of the
// chip idle, and its step lasts as long as one tile's march.  So 2 or 4 rows where
// that makes less than 1024 or 2048 tiles (more cost the reduction of their rows
// what they save): us per planar step in FP64 with 8 rows / fewer, 400 x 100 26.2 /
// 19.4 (2 rows), 800 x 200 28.9 / 24.9 (4; with 2 26.3), 1200 x 300 30.9 / 27.9 (4),
// 500 x 500 30.0 / 29.6 (4; 2500 tiles of 4 rows and more: 28 to 31 either way);
// four states on 200 x 200 231 / 182.
constexpr int kMinRows = 8;
int64_t min_rows(const Grid& g)
{
    for (int64_t r = 2; r < kMinRows; r *= 2)
        if (x_strips(g) * ((g.ny + r - 1) / r) < 512 * r) return r;
    return kMinRows;
}

}  // namespace

// About one tile per resident wavefront of the lean pass, which does the whole
// of a planar step: taller tiles march fewer halo rows again, and tiles beyond
// the resident wavefronts would start a second round.
MarchGeom march2d_geometry(const Grid& g, int cus, int per_cu, int per_cu_lean)
{
    MarchGeom m;
    const int64_t xs = x_strips(g);
    const int64_t resident = (int64_t)(cus > 0 ? cus : 1) * (per_cu > 0 ? per_cu : 1);
    const int64_t resident_lean = (int64_t)(cus > 0 ? cus : 1) * (per_cu_lean > 0 ? per_cu_lean : 1);
    const int64_t chunks = std::max<int64_t>(1, resident_lean * kMNW / xs);
    const int64_t sy = std::max<int64_t>((g.ny + chunks - 1) / chunks, min_rows(g));
    m.sy = (int)sy;
    m.grid_x = xs;
    m.grid_y = (g.ny + sy - 1) / sy;
    const int64_t nt = m.blocks();
    m.nblocks_lean = (int)std::min<int64_t>(resident_lean, (nt + kMNW - 1) / kMNW);
    m.nblocks = (int)std::min<int64_t>(resident, (nt * kSplitMax + kMNW - 1) / kMNW);
    return m;
}

int64_t march2d_max_blocks(const Grid& g)
{
    const int64_t r = min_rows(g);
    return x_strips(g) * ((g.ny + r - 1) / r);
}

template <typename T>
int march2d_blocks_per_cu(bool lean, bool rest, bool species)
{
    if (species) return march2d_blocks_per_cu_species<T>(lean, rest);
    return rest ? march_resident<T, true, false, false>(lean) : march_resident<T, false, false, false>(lean);
}

// The dual-level set runs the instances without the rest group.
template <typename T>
hipError_t launch_march2d(const T* Y, T* Yn, const Grid& g, const MarchGeom& m, const Consts& k,
                          StepCtl* ctl, double* partials, const MarchWords& w, long long step, hipStream_t stream)
{
    if (k.species) return launch_march2d_species<T>(Y, Yn, g, m, k, ctl, partials, w, step, stream);
    return k.rest ? launch_march2d_w<T, true, false>(Y, Yn, g, m, k, ctl, partials, w, step, stream)
                          : launch_march2d_w<T, false, false>(Y, Yn, g, m, k, ctl, partials, w, step, stream);
}

template <typename T>
hipError_t launch_lanes_march(const T* Y, const Grid& g, const Consts& k, int32_t* fx, int32_t* fy, int32_t* c1,
                              hipStream_t stream)
{
    if (k.species) return launch_lanes_species<T>(Y, g, k, fx, fy, c1, stream);
    return k.rest ? launch_lanes_w<T, true, false>(Y, g, k, fx, fy, c1, stream)
                          : launch_lanes_w<T, false, false>(Y, g, k, fx, fy, c1, stream);
}

template int march2d_blocks_per_cu<double>(bool, bool, bool);
template int march2d_blocks_per_cu<float>(bool, bool, bool);
template hipError_t launch_march2d<double>(const double*, double*, const Grid&, const MarchGeom&, const Consts&,
                                           StepCtl*, double*, const MarchWords&, long long, hipStream_t);
template hipError_t launch_march2d<float>(const float*, float*, const Grid&, const MarchGeom&, const Consts&,
                                          StepCtl*, double*, const MarchWords&, long long, hipStream_t);
template hipError_t launch_lanes_march<double>(const double*, const Grid&, const Consts&, int32_t*, int32_t*, int32_t*,
                                               hipStream_t);
template hipError_t launch_lanes_march<float>(const float*, const Grid&, const Consts&, int32_t*, int32_t*, int32_t*,
                                              hipStream_t);

}  // namespace lbsd
