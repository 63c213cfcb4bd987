// Kernel-side interface shared by the step kernels and the host runtime.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lb_device.hpp"

namespace lbsd {

constexpr int kErrReach = 1;  // a packet would travel further than the halo
constexpr int kErrState = 2;  // rho <= 0 or a non-finite moment

// Tiles the square lattice's lean pass gave up are counted in kGivenUp words
// a cache line apart: on general flows every wavefront of the pass counts one
// at about the same time, and one word takes them one after another.
constexpr int kGivenUp = 16, kGivenUpStride = 32;

// Per-solver control block in device memory (written by the step kernels).
struct StepCtl {
    int next[5];            // square lattice: tile claim counters of the two passes (reset by finalize)
    int err_code;           // kErr* bits of the first failed step
    long long err_step;     // first failed step (LLONG_MAX if none)
    long long totals_step;  // step whose totals are in `totals`
    double totals[4];       // interior sums of the moment fields (lattice units)
    int max_reach;          // largest reach seen in the latest step
    int err_buf;            // moment set (0 or 1) that holds the last good state after a failed step
    double totals_sp;       // square lattice with two gases: interior sum of rho chi
    long long fail_step0;   // 1-D: the launch a step of which failed: its first step,
    int fail_steps, fail_in;  // its steps and the set it read (which it leaves intact)
    int given_up[kGivenUp * kGivenUpStride];  // square lattice: see kGivenUp (cleared by finalize)
};

// Per-block partial results: 4 field sums, reach, error bits; the square
// lattice with two gases puts the sum of rho chi at index 6.
constexpr int kPartialStride = 8;

struct Grid {
    int64_t nx, ny;  // ny = 1 in 1-D
    int bc_x, bc_y;
};

// 1-D: `steps` <= tube_group steps in one launch, step0 the first, from the
// moment set Y (set in_buf) to Yn (SoA [nf][nx] of T).
template <typename T>
hipError_t launch_tube(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, double* partials,
                       long long step0, int steps, int in_buf, hipStream_t stream);
// Behind the launches of a call, the last of them `steps` steps from step0: the
// reduction of its partial rows (step_blocks_1d of them at most) and, if a step of
// any of the launches failed, its error and the set that ctl then names, which
// holds the last good state once launch_tube_again has made it.
hipError_t launch_tube_finalize(const Grid& g, const Consts& k, bool fp64, StepCtl* ctl, double* partials,
                                long long step0, int steps, hipStream_t stream);
// The `steps` good steps of a failed launch of K again, from its input Y to Yn, and
// the failing step's largest reach over all nodes.
template <typename T>
hipError_t launch_tube_again(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, int K, int steps,
                             hipStream_t stream);
int tube_group(const Grid& g, const Consts& k, bool fp64);
int64_t step_blocks_1d(const Grid& g);

// Square lattice, column-march kernels (lb_march2d.hpp).  The grid is cut into
// tiles (strips of kMarchCols columns x row chunks) that the device's resident
// wavefronts take.
constexpr int kHalo = 5;
constexpr int kMarchCols = 64 - 2 * kHalo;
struct MarchGeom {
    int sy;                   // destination rows per tile
    int64_t grid_x, grid_y;   // tiles along x (column strips) and y (row chunks)
    int nblocks;              // blocks (of four wavefronts) of the general pass, resident at once
    int nblocks_lean;         // blocks of the lean pass
    int64_t blocks() const { return grid_x * grid_y; }  // tiles (= rows of partials)
};
// cus: compute units; per_cu / per_cu_lean: resident blocks per CU of the
// general and the lean pass (march2d_blocks_per_cu).
MarchGeom march2d_geometry(const Grid& g, int cus, int per_cu, int per_cu_lean);
int64_t march2d_max_blocks(const Grid& g);
// Resident blocks per CU of the general pass (lean = false) or the lean pass, of
// the instance with or without a rest level and a second gas.
template <typename T>
int march2d_blocks_per_cu(bool lean, bool rest, bool species);
// Per-tile words of the two passes (device memory), and the row chunks the
// general pass may cut a tile into (it then writes smax partial rows per tile).
struct MarchWords {
    int* flags;  // this step's lean pass gave the tile up
    int* keep;   // the next step's lean pass will (zero at the start; nullptr: not kept between steps)
    int* nch;    // partial rows the tile has this step (row p at p * tiles + tile)
    int smax;
};
constexpr int kSplitMax = 8;
// Bytes of the three words per tile.
inline size_t march2d_word_bytes(int64_t ntiles) { return (size_t)3 * ntiles * 4; }
inline MarchWords march2d_words(int* w, int64_t ntiles, int smax, bool keep)
{
    return MarchWords{w, keep ? w + ntiles : nullptr, w + 2 * ntiles, smax};
}
// One step: the lean pass over every tile, then the general pass over the
// tiles it gave up and the row-chunk neighbours their sources can reach (it
// returns at once when there are none).
template <typename T>
hipError_t launch_march2d(const T* Y, T* Yn, const Grid& g, const MarchGeom& m, const Consts& k,
                          StepCtl* ctl, double* partials, const MarchWords& w, long long step, hipStream_t stream);

// Hexagonal lattice (lb_hex.hip): hex_blocks(g) blocks and partial rows per step.
template <typename T>
hipError_t launch_hex(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, double* partials,
                      long long step, hipStream_t stream);
int64_t hex_blocks(const Grid& g);

// Reduce nb per-block partial rows of one step into ctl (fixed order);
// species2d: also the rho chi sums of the square lattice with two gases; nch:
// rows per tile where a tile may have several (MarchWords::nch), else nullptr.
// in_buf: the moment set (0 or 1) the step read.
hipError_t launch_finalize(double* partials, int64_t nb, StepCtl* ctl, long long step, int in_buf,
                           hipStream_t stream, bool species2d = false, const int* nch = nullptr);

// Riemann initial state: node i (cell centre x_lo + (i + 1/2) dx) takes the
// left moments when x < x_d, else the right ones (lattice units; left and
// right hold 5 values, of which the first nf are used).
template <typename T>
hipError_t launch_init_riemann(T* Y, const Grid& g, int nf, double x_lo, double dx, double x_d,
                               const double* left, const double* right, hipStream_t stream);

// Lattice-unit state -> FP64 physical moments (divide by scale[f]; 5 values).
// which (device memory, may be null): Y1 holds the state where *which != 0.
template <typename T>
hipError_t launch_export(const T* Y, double* out, int64_t nn, int nf, const double* scale,
                         hipStream_t stream, const T* Y1 = nullptr, const int32_t* which = nullptr);

// Per-node (f_x, f_y, c'_1) by the node functions of each lattice's step (a
// wavefront of 64 consecutive nodes takes the tame or the general form for all).
template <typename T>
hipError_t launch_lanes_tube(const T* Y, const Grid& g, const Consts& k, int32_t* fx, int32_t* fy, int32_t* c1,
                             hipStream_t stream);
template <typename T>
hipError_t launch_lanes_march(const T* Y, const Grid& g, const Consts& k, int32_t* fx, int32_t* fy, int32_t* c1,
                              hipStream_t stream);
template <typename T>
hipError_t launch_lanes_hex(const T* Y, const Grid& g, const Consts& k, int32_t* fa, int32_t* fb, int32_t* c1,
                            hipStream_t stream);

hipError_t launch_reset_ctl(StepCtl* ctl, hipStream_t stream);

// p[0 .. n) := v (a kernel, not a memset: it may be captured into a graph).
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t stream);

// *out := the outcome of the step(s) recorded in ctl: kStatusOk, or the
// status code of the first failure (the values of LB_OK, LB_ESTATE, LB_EREACH).
constexpr int kStatusOk = 0, kStatusState = -4, kStatusReach = -5;
hipError_t launch_status(const StepCtl* ctl, int32_t* out, hipStream_t stream);

// ---- pools: many independent problems advanced together by launches over a
// device-resident tile table (lb_pool.hip) ----

struct PoolProb {       // one slot, written by the host between launches
    int64_t off[2];     // element offsets of the two SoA moment sets in the arena
    int64_t nx, ny;
    int32_t bc_x, bc_y;
    int32_t active;     // 0: free slot (it owns no tiles)
    int32_t pad;
    int64_t target;     // the problem stops after this many good steps
    int64_t t0, t1;     // its tiles [t0, t1) in the tile table
};

struct PoolState {      // one slot, written by the device, read by the host after a sync
    int64_t done;       // good steps so far
    int64_t err_step;   // step that failed (0: none); the problem then stops
    int32_t err_code;   // kErr* bits
    int32_t max_reach;  // largest reach of its latest step
    int64_t totals_step;
    double totals[4];   // interior sums after step totals_step (lattice units)
    int32_t set;        // moment set that holds the moments
    int32_t pad;
};

struct PoolTile {        // one tile, with a copy of its slot's grid so a block reads one record
    int32_t prob, rows;  // slot; destination rows (square lattice; 1 in 1-D)
    int64_t x0, y0;      // first destination column / row
    int64_t off[2];      // the slot's two moment sets (element offsets in the arena)
    int64_t nx, ny;
    int32_t bc_x, bc_y;
};

// Per-tile word kept by the per-slot reduction: bit 0 = the set holding the
// slot's current moments, bit 1 = the slot still steps; 1-D: from bit 8 the
// steps it has left (at most kTileLeftMax), or, with bit 2, the good steps of a
// failed launch that are to be made again.
constexpr int kTileSet = 1, kTileLive = 2, kTileAgain = 4, kTileLeftShift = 8, kTileLeftMax = 1 << 20;

struct PoolView {
    const PoolProb* probs;
    PoolState* state;
    const PoolTile* tiles;
    int32_t* tstate;        // kTileSet | kTileLive per tile
    const int32_t* ntiles;  // tiles in the table (read by the kernels, so admissions need no new launch shape)
    double* partials;       // kPartialStride doubles per tile
    int32_t* flags;         // square lattice: per tile, the next step's lean pass will give it up
    int32_t* flags_lean;    // square lattice: per tile, this step's lean pass gave it up
    int32_t* next;          // 5 counters, as StepCtl::next; reset by finalize
    void* arena;            // moment sets of all slots (T elements)
};

// Tile shapes of the 1-D pool kernel: the steps a launch makes (a tile is then
// the tube_cols nodes that a wavefront can bring that far on its own).
constexpr int kPool1Shapes = 5;
constexpr int kPool1Steps[kPool1Shapes] = {1, 2, 4, 6, 8};
// Nodes per lane of a long tube and of the pools' (see lb_tube.hpp): five, or
// three for two gases in FP64, which would otherwise take 390 registers.
constexpr int tube_lanes(bool species, bool fp64) { return species && fp64 ? 3 : 5; }
constexpr int tube_lost(int J) { return (kHalo + J - 1) / J; }                      // halo lanes a step costs
constexpr int tube_cols(int J, int K) { return (64 - 2 * K * tube_lost(J)) * J; }  // nodes a wavefront stores

// Square-lattice pool tiles: the strip height is chosen so that the live
// problems make about kPool2TilesPerBlock[shape] tiles per resident block
// (claim-order balance against the 2L halo rows each tile marches again), and
// is at least kPool2MinRows.
constexpr int kPool2Shapes = 5;
constexpr int kPool2TilesPerBlock[kPool2Shapes] = {2, 3, 4, 6, 8};
constexpr int kPool2MinRows = 16;
constexpr int kPool2Cols = kMarchCols;  // destination columns per square-lattice tile

// 1-D: up to `steps` <= halo steps of every live slot (nblocks: a wavefront per
// tile, four per block) and the per-slot reduction, which commits them if
// commit != 0.
template <typename T>
hipError_t launch_pool1d(const PoolView& v, const Consts& k, int halo, int steps, int nblocks, int nslots, int commit,
                         hipStream_t stream);
// Behind a call's launches: the good steps of those that failed, made again.
template <typename T>
hipError_t launch_pool1d_again(const PoolView& v, const Consts& k, int halo, int nblocks, hipStream_t stream);
// Square lattice, one step of every live tile: the lean pass, then the general
// pass over what it left (resident wavefronts take the tiles).
template <typename T>
hipError_t launch_pool2d(const PoolView& v, const Consts& k, int nblocks_lean, int nblocks, hipStream_t stream);
// Resident blocks per CU of the pool's general pass (lean = false) or lean pass.
template <typename T>
int pool2d_blocks_per_cu(bool lean, bool rest, bool species);
// Per slot of a square-lattice pool: reduce its tiles' partial rows (fixed
// order) into its state and, when commit != 0 and the step succeeded, count the
// step.
hipError_t launch_pool2d_finalize(const PoolView& v, int nslots, int commit, hipStream_t stream);

}  // namespace lbsd
