// The 1-D step kernels (how a wavefront makes its steps is in lb_tube.hpp) and
// the per-step reductions, of which the square and hexagonal lattices use the
// plain one.  Steps write one row of partial results per block; a one-block
// kernel then adds the rows in a fixed order (deterministic totals) and records
// the reach (halo overflow) and state checks.  No atomics or device-scope fences
// in the step kernels: the kernel boundary orders the rows.
#include "lb_tube.hpp"

namespace lbsd {

namespace {

// First stage of the reduction of many partial rows (too many for one block to
// read quickly; with nch, tile b has nch[b] rows, i nb + b): block g folds tiles
// [g kChunk, (g + 1) kChunk) in a fixed order (sums, largest reach, error bits)
// into row g kChunk, the first of its own chunk, so that blocks never touch each
// other's rows.
constexpr int kChunk = 256;
__global__ void __launch_bounds__(kChunk)
partials_chunk_kernel(double* __restrict__ partials, int64_t nb, const StepCtl* __restrict__ ctl, long long step,
                      const int* __restrict__ nch)
{
    __shared__ double s_sum[kChunk / 64][5];
    __shared__ int s_ir[kChunk / 64][2];
    if (ctl->err_step < step) return;  // an earlier step failed: the rows are not this step's
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t b0 = (int64_t)blockIdx.x * kChunk, b = b0 + tid;
    double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    int reach = 0, err = 0;
    const int rows = b < nb ? (nch ? nch[b] : 1) : 0;
    for (int i = 0; i < rows; ++i) {
        const double* p = partials + ((int64_t)i * nb + b) * kPartialStride;
#pragma unroll
        for (int f = 0; f < 4; ++f) s[f] += p[f];
        s[4] += p[6];
        reach = max(reach, (int)p[4]);
        err |= (int)p[5];
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) s[f] = wave_sum(s[f]);
    reach = wave_max(reach);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) err |= __shfl_xor(err, o, 64);
    if (lane == 0) {
#pragma unroll
        for (int f = 0; f < 5; ++f) s_sum[wid][f] = s[f];
        s_ir[wid][0] = reach;
        s_ir[wid][1] = err;
    }
    __syncthreads();
    if (tid == 0) {
        double* q = partials + b0 * kPartialStride;
        for (int f = 0; f < 5; ++f) {
            double t = s_sum[0][f];
            for (int w = 1; w < kChunk / 64; ++w) t += s_sum[w][f];
            q[f < 4 ? f : 6] = t;
        }
        int r = s_ir[0][0], e = s_ir[0][1];
        for (int w = 1; w < kChunk / 64; ++w) { r = max(r, s_ir[w][0]); e |= s_ir[w][1]; }
        q[4] = (double)r;
        q[5] = (double)e;
    }
}

// Sum the per-block partials of one step in a fixed order (deterministic),
// record the totals, the largest reach and the first failed step.  Rows b
// stride for b < nb (stride > 1: the chunk heads of partials_chunk_kernel).
// A thread's rows are read one after another: 1024 threads from kFinManyRows
// rows on (4096 rows took 14 us with 256 threads, 10 with 1024; but a step of a
// few rows, whose latency counts, 3 us more).
constexpr int kFinTPB = 256, kFinMaxTPB = 1024, kFinManyRows = 1024;
template <int TPB>
__global__ void __launch_bounds__(TPB)
finalize_kernel(const double* __restrict__ partials, int64_t nb, int64_t stride, StepCtl* __restrict__ ctl,
                long long step, int sp2, const int* __restrict__ nch, int in_buf)
{
    __shared__ double s_sum[TPB / 64][5];
    __shared__ int s_ir[TPB / 64][2];
    if (threadIdx.x == 0) {  // the step kernels of this step are done with their counters
        for (int i = 0; i < 5; ++i) ctl->next[i] = 0;
    }
    if (threadIdx.x < kGivenUp) ctl->given_up[threadIdx.x * kGivenUpStride] = 0;
    if (ctl->err_step < step) return;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    int reach = 0, err = 0;
    for (int64_t b = tid; b < nb; b += TPB) {
        const int rows = nch ? nch[b] : 1;  // (at least 1: the first row need not wait for it)
        int i = 0;
        do {
            const double* p = partials + ((int64_t)i * nb + b) * stride * kPartialStride;
#pragma unroll
            for (int f = 0; f < 4; ++f) s[f] += p[f];
            if (sp2) s[4] += p[6];  // rho chi (square lattice, two gases)
            reach = max(reach, (int)p[4]);
            err |= (int)p[5];
        } while (++i < rows);
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) s[f] = wave_sum(s[f]);
    reach = wave_max(reach);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) err |= __shfl_xor(err, o, 64);
    if (lane == 0) {
#pragma unroll
        for (int f = 0; f < 5; ++f) s_sum[wid][f] = s[f];
        s_ir[wid][0] = reach;
        s_ir[wid][1] = err;
    }
    __syncthreads();
    if (tid == 0) {
        for (int f = 0; f < 5; ++f) {
            double t = s_sum[0][f];
            for (int w = 1; w < TPB / 64; ++w) t += s_sum[w][f];
            if (f < 4) ctl->totals[f] = t;
            else ctl->totals_sp = t;
        }
        int r = s_ir[0][0], e = s_ir[0][1];
        for (int w = 1; w < TPB / 64; ++w) { r = max(r, s_ir[w][0]); e |= s_ir[w][1]; }
        ctl->max_reach = r;
        ctl->totals_step = step;
        if (e) {
            ctl->err_code = e;
            ctl->err_step = step;
            ctl->err_buf = in_buf;  // its input, which it left intact
        }
    }
}

// ------------------------------------------------------------------ 1-D ----

// Outcomes of wavefronts or blocks combined: the earliest failing step counts,
// then its error bits and largest reach.
__device__ __forceinline__ TubeOut worse(const TubeOut& a, const TubeOut& b)
{
    const int ea = a.errsub ? a.errsub : INT_MAX, eb = b.errsub ? b.errsub : INT_MAX;
    if (ea < eb) return a;
    if (eb < ea) return b;
    return TubeOut{max(a.reach, b.reach), a.err | b.err, a.errsub};
}
__device__ __forceinline__ TubeOut wave_worse(TubeOut o)
{
#pragma unroll
    for (int m = 32; m > 0; m >>= 1)
        o = worse(o, TubeOut{__shfl_xor(o.reach, m, 64), __shfl_xor(o.err, m, 64), __shfl_xor(o.errsub, m, 64)});
    return o;
}

// A row of partials of the 1-D kernels: sums, reach and error bits as
// elsewhere; index 7 the failing step of the launch (TubeOut::errsub).
__device__ __forceinline__ void put_row(double* __restrict__ row, const double (&s)[4], const TubeOut& o)
{
#pragma unroll
    for (int f = 0; f < 4; ++f) row[f] = s[f];
    row[4] = (double)o.reach;
    row[5] = (double)o.err;
    row[6] = 0.0;
    row[7] = (double)o.errsub;
}
__device__ __forceinline__ TubeOut row_out(const double* __restrict__ row)
{
    return TubeOut{(int)row[4], (int)row[5], (int)row[7]};
}

// The block's sums and outcome, in wavefront order, in every thread.
template <int NW>
__device__ __forceinline__ TubeOut block_rows(double (&s)[4], TubeOut o)
{
    __shared__ double s_sum[NW][4];
    __shared__ TubeOut s_out[NW];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int f = 0; f < 4; ++f) s[f] = wave_sum(s[f]);
    o = wave_worse(o);
    __syncthreads();
    if (lane == 0) {
#pragma unroll
        for (int f = 0; f < 4; ++f) s_sum[wid][f] = s[f];
        s_out[wid] = o;
    }
    __syncthreads();
    const int nw = min(NW, (int)(blockDim.x >> 6));
    o = s_out[0];
#pragma unroll
    for (int f = 0; f < 4; ++f) s[f] = s_sum[0][f];
    for (int w = 1; w < nw; ++w) {
        o = worse(o, s_out[w]);
#pragma unroll
        for (int f = 0; f < 4; ++f) s[f] += s_sum[w][f];
    }
    return o;
}

constexpr int kTubeTPB = 256, kTubeNW = kTubeTPB / 64;
// Wavefronts per SIMD.  Five nodes per lane take 240 registers in FP64 and with
// two gases; one gas in FP32 fits three wavefronts with 20 registers spilled
// (2^24 nodes 92 us per step, two wavefronts without spills 105).
template <typename T, bool SP, int J>
constexpr int kTubeWpe = J > 2 && sizeof(T) == 4 && !SP ? 3 : 2;

// `steps` steps, step0 the first: one tile per wavefront, one row of partials
// per block.  A failure is entered in ctl at once, so that the launches queued
// behind return without touching the failed launch's input.
template <typename T, bool SP, int J>
__global__ void __launch_bounds__(kTubeTPB) __attribute__((amdgpu_waves_per_eu(kTubeWpe<T, SP, J>)))
tube_kernel(const T* __restrict__ Y, T* __restrict__ Yn, int64_t nx, int bc, Consts k, StepCtl* __restrict__ ctl,
            double* __restrict__ partials, long long step0, int steps, int64_t ntiles, int in_buf)
{
    __shared__ TubeEdges<T> s_edges[kTubeNW];
    __shared__ TubeStash<T, SP, J> s_stash[kTubeNW];
    if (ctl->err_step < step0) return;  // an earlier step failed: keep its input intact
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t tile = (int64_t)blockIdx.x * kTubeNW + wid;
    double tot[SP ? 4 : 3] = {};
    TubeOut o{0, 0, 0};
    if (tile < ntiles)
        o = tube_run<T, SP, J>(Y, Yn, nx, bc, tile * tube_cols(J, steps), steps, steps, k, s_edges[wid], s_stash[wid],
                               tot);
    double s[4] = {tot[0], tot[1], tot[2], SP ? tot[SP ? 3 : 0] : 0.0};
    o = block_rows<kTubeNW>(s, o);
    if (threadIdx.x == 0) {
        put_row(partials + (int64_t)blockIdx.x * kPartialStride, s, o);
        if (o.errsub) {
            atomicMin((unsigned long long*)&ctl->err_step, (unsigned long long)(step0 + o.errsub - 1));
            ctl->fail_step0 = step0;  // (every failing block of the launch writes the same)
            ctl->fail_steps = steps;
            ctl->fail_in = in_buf;
        }
    }
}

// Many rows: block g folds rows [g kChunk, (g + 1) kChunk) into the first.
__global__ void __launch_bounds__(kChunk)
tube_chunk_kernel(double* __restrict__ partials, int64_t nb, const StepCtl* __restrict__ ctl)
{
    if (ctl->err_step != LLONG_MAX) return;  // the rows of a failed launch are read one by one
    const int64_t b0 = (int64_t)blockIdx.x * kChunk, b = b0 + threadIdx.x;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    TubeOut o{0, 0, 0};
    if (b < nb) {
        const double* p = partials + b * kPartialStride;
#pragma unroll
        for (int f = 0; f < 4; ++f) s[f] = p[f];
        o = row_out(p);
    }
    o = block_rows<kChunk / 64>(s, o);
    if (threadIdx.x == 0) put_row(partials + b0 * kPartialStride, s, o);
}

__host__ __device__ constexpr int64_t tube_tiles(int64_t nx, int J, int K) { return (nx + tube_cols(J, K) - 1) / tube_cols(J, K); }
__host__ __device__ constexpr int64_t tube_blocks(int64_t nx, int J, int K)
{
    return (tube_tiles(nx, J, K) + kTubeNW - 1) / kTubeNW;
}

// Behind the launches of one call, the last of them `steps` steps from step0, of J
// nodes per lane: its rows (stride as in finalize_kernel) -> totals and reach.
// Where a step of any of the launches failed, its error: the first of its rows'.
template <int TPB>
__global__ void __launch_bounds__(TPB)
tube_finalize_kernel(const double* __restrict__ partials, int64_t nb, int64_t stride, StepCtl* __restrict__ ctl,
                     long long step0, int steps, int64_t nx, int J)
{
    if (ctl->err_code) return;  // a failure that is dealt with
    const bool failed = ctl->err_step != LLONG_MAX;
    const int in = ctl->fail_in;
    if (failed) {
        nb = tube_blocks(nx, J, ctl->fail_steps);
        stride = 1;
    }
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    TubeOut o{0, 0, 0};
    for (int64_t b = threadIdx.x; b < nb; b += TPB) {
        const double* p = partials + b * stride * kPartialStride;
#pragma unroll
        for (int f = 0; f < 4; ++f) s[f] += p[f];
        o = worse(o, row_out(p));
    }
    o = block_rows<TPB / 64>(s, o);
    if (threadIdx.x != 0) return;
    ctl->max_reach = o.reach;
    if (failed) {
        ctl->err_code = o.err;
        ctl->err_buf = o.errsub > 1 ? in ^ 1 : in;
    } else {
        for (int f = 0; f < 4; ++f) ctl->totals[f] = s[f];
        ctl->totals_sp = 0.0;
        ctl->totals_step = step0 + steps - 1;
    }
}

// After a failed launch of K-step tiles: makes the `steps` good steps before the
// failing one again, from Y to Yn, and the failing one for its largest reach.
template <typename T, bool SP, int J>
__global__ void __launch_bounds__(kTubeTPB) __attribute__((amdgpu_waves_per_eu(kTubeWpe<T, SP, J>)))
tube_again_kernel(const T* __restrict__ Y, T* __restrict__ Yn, int64_t nx, int bc, Consts k, StepCtl* __restrict__ ctl,
                  int64_t ntiles, int K, int steps)
{
    __shared__ TubeEdges<T> s_edges[kTubeNW];
    __shared__ TubeStash<T, SP, J> s_stash[kTubeNW];
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t tile = (int64_t)blockIdx.x * kTubeNW + wid, X0 = tile * tube_cols(J, K);
    if (tile >= ntiles) return;
    double tot[SP ? 4 : 3] = {};
    const TubeOut o = tube_run<T, SP, J, true>(Y, Yn, nx, bc, X0, K, steps + 1, k, s_edges[wid], s_stash[wid], tot);
    if ((threadIdx.x & 63) == 0) atomicMax(&ctl->max_reach, o.reach);
}

// floor(v) and c'_1 of every node (a spare lane repeats the last node).
template <typename T, bool SP>
__global__ void __launch_bounds__(kTubeTPB)
tube_lanes_kernel(const T* __restrict__ Y, int64_t nx, Consts k, int32_t* __restrict__ fx, int32_t* __restrict__ fy,
                  int32_t* __restrict__ c1)
{
    const int64_t q = (int64_t)blockIdx.x * kTubeTPB + threadIdx.x, x = min(q, nx - 1);
    T y[SP ? 4 : 3][1];
    static_for<(SP ? 4 : 3)>([&](auto f) { y[f][0] = Y[f * nx + x]; });
    int f, c;
    tube_decisions<T, SP>(y, k, &f, &c);
    if (q >= nx) return;
    fx[q] = f;
    fy[q] = 0;
    c1[q] = c;
}

// Pool form: one wavefront per tile of the tile table.  A tile belongs to one
// slot; its word says whether the slot still steps, how many steps it has left
// and which moment set holds its state.
template <typename T, bool SP, int J>
__global__ void __launch_bounds__(kTubeTPB) __attribute__((amdgpu_waves_per_eu(kTubeWpe<T, SP, J>)))
pool_tube_kernel(PoolView v, Consts k, int K, int steps, int commit)
{
    __shared__ TubeEdges<T> s_edges[kTubeNW];
    __shared__ TubeStash<T, SP, J> s_stash[kTubeNW];
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int t = blockIdx.x * kTubeNW + wid;
    if (t >= *v.ntiles) return;
    const int ts = v.tstate[t];
    if (!(ts & kTileLive)) return;
    T* arena = (T*)v.arena;
    const PoolTile& tl = v.tiles[t];
    const int64_t o0 = tl.off[0], o1 = tl.off[1];
    const int64_t from = (ts & kTileSet) ? o1 : o0, to = (ts & kTileSet) ? o0 : o1;
    double tot[SP ? 4 : 3] = {};
    // (a trial launch, whose steps do not count, makes all of them)
    const int n = commit ? min(steps, ts >> kTileLeftShift) : steps;
    const TubeOut o = tube_run<T, SP, J>(arena + from, arena + to, tl.nx, tl.bc_x, tl.x0, K, n, k, s_edges[wid],
                                      s_stash[wid], tot);
    double s[4] = {tot[0], tot[1], tot[2], SP ? tot[SP ? 3 : 0] : 0.0};
#pragma unroll
    for (int f = 0; f < 4; ++f) s[f] = wave_sum(s[f]);
    if ((threadIdx.x & 63) == 0) put_row(v.partials + (int64_t)t * kPartialStride, s, o);
}

// Per slot of a 1-D pool (one block each): the reduction of tube_finalize_kernel
// over the slot's tiles; commits the launch's steps.  A step that failed after good
// ones of its launch leaves the slot's tiles marked for pool_tube_again_kernel.
__global__ void __launch_bounds__(kFinTPB) pool_tube_finalize_kernel(PoolView v, int steps, int commit)
{
    const PoolProb& P = v.probs[blockIdx.x];
    PoolState& S = v.state[blockIdx.x];
    const int64_t done = S.done;
    const int set = S.set;
    if (!commit || !P.active || done >= P.target || S.err_step != 0) return;
    const int n = (int)min((int64_t)steps, P.target - done);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    TubeOut o{0, 0, 0};
    for (int64_t b = P.t0 + threadIdx.x; b < P.t1; b += kFinTPB) {
        const double* p = v.partials + b * kPartialStride;
#pragma unroll
        for (int f = 0; f < 4; ++f) s[f] += p[f];
        o = worse(o, row_out(p));
    }
    o = block_rows<kFinTPB / 64>(s, o);
    const int good = o.errsub ? o.errsub - 1 : n;
    const int64_t now = done + good;
    const int nset = good > 0 ? set ^ 1 : set;
    const int64_t left = P.target - now;
    int word = nset;
    if (o.errsub && good > 0) word |= kTileAgain | good << kTileLeftShift;
    if (!o.errsub && left > 0) word |= kTileLive | (int)min(left, (int64_t)kTileLeftMax) << kTileLeftShift;
    for (int64_t t = P.t0 + threadIdx.x; t < P.t1; t += kFinTPB) v.tstate[t] = word;
    if (threadIdx.x != 0) return;
    for (int f = 0; f < 4; ++f) S.totals[f] = s[f];
    S.max_reach = o.reach;
    S.totals_step = done + n;
    S.done = now;
    S.set = nset;
    if (o.errsub) {
        S.err_code = o.err;
        S.err_step = now + 1;
        if (good > 0) atomicAdd(&v.next[0], 1);
    }
}

// Behind the launches of one call, some of more than one step: the good steps of
// launches that failed, made again.  (next[0] says whether there may be any; the
// next upload of the tables clears it.)
template <typename T, bool SP, int J>
__global__ void __launch_bounds__(kTubeTPB) __attribute__((amdgpu_waves_per_eu(kTubeWpe<T, SP, J>)))
pool_tube_again_kernel(PoolView v, Consts k, int K)
{
    __shared__ TubeEdges<T> s_edges[kTubeNW];
    __shared__ TubeStash<T, SP, J> s_stash[kTubeNW];
    if (v.next[0] == 0) return;
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int t = blockIdx.x * kTubeNW + wid;
    if (t >= *v.ntiles) return;
    const int ts = v.tstate[t];
    if (!(ts & kTileAgain)) return;
    T* arena = (T*)v.arena;
    const PoolTile& tl = v.tiles[t];
    const int64_t o0 = tl.off[0], o1 = tl.off[1];
    const int64_t from = (ts & kTileSet) ? o0 : o1, to = (ts & kTileSet) ? o1 : o0;  // (the word has the new set)
    double tot[SP ? 4 : 3] = {};
    tube_run<T, SP, J>(arena + from, arena + to, tl.nx, tl.bc_x, tl.x0, K, ts >> kTileLeftShift, k, s_edges[wid],
                       s_stash[wid], tot);
    if ((threadIdx.x & 63) == 0) v.tstate[t] = ts & kTileSet;
}

// Per slot of a square-lattice pool (one block each): the same fixed-order
// reduction as finalize_kernel over the slot's tile rows.
__global__ void __launch_bounds__(kFinTPB) pool_finalize_kernel(PoolView v, int commit)
{
    __shared__ double s_sum[kFinTPB / 64][4];
    __shared__ int s_ir[kFinTPB / 64][2];
    const int p = blockIdx.x;
    if (p == 0 && threadIdx.x == 0) {  // the step kernels of this step are done with their counters
        for (int i = 0; i < 5; ++i) v.next[i] = 0;
    }
    const PoolProb& P = v.probs[p];
    PoolState& S = v.state[p];
    if (!P.active || S.done >= P.target || S.err_step != 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int reach = 0, err = 0;
    for (int64_t b = P.t0 + tid; b < P.t1; b += kFinTPB) {
        const double* q = v.partials + b * kPartialStride;
#pragma unroll
        for (int f = 0; f < 4; ++f) s[f] += q[f];
        reach = max(reach, (int)q[4]);
        err |= (int)q[5];
    }
#pragma unroll
    for (int f = 0; f < 4; ++f) s[f] = wave_sum(s[f]);
    reach = wave_max(reach);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) err |= __shfl_xor(err, o, 64);
    if (lane == 0) {
#pragma unroll
        for (int f = 0; f < 4; ++f) s_sum[wid][f] = s[f];
        s_ir[wid][0] = reach;
        s_ir[wid][1] = err;
    }
    __shared__ int s_word;
    __syncthreads();
    if (tid == 0 && commit) {
        const int64_t step = S.done + 1;
        for (int f = 0; f < 4; ++f) {
            double t = s_sum[0][f];
            for (int w = 1; w < kFinTPB / 64; ++w) t += s_sum[w][f];
            S.totals[f] = t;
        }
        int r = s_ir[0][0], e = s_ir[0][1];
        for (int w = 1; w < kFinTPB / 64; ++w) { r = max(r, s_ir[w][0]); e |= s_ir[w][1]; }
        S.max_reach = r;
        S.totals_step = step;
        if (e) {
            S.err_code = e;
            S.err_step = step;
        } else {
            S.done = step;
            S.set ^= 1;
        }
        s_word = S.set | (!e && S.done < P.target ? kTileLive : 0);
    }
    __syncthreads();
    if (commit)
        for (int64_t t = P.t0 + tid; t < P.t1; t += kFinTPB) v.tstate[t] = s_word;
}

}  // namespace

namespace {

// Nodes per lane and steps per launch of a tube.  Where the chip is idle a launch
// lasts as long as a wavefront's steps, so short tubes take two nodes per lane
// and as many steps as leave a wavefront on most SIMDs (32, 56 or 80 nodes per
// wavefront for 8, 6 or 4 steps); beyond that five nodes per lane, whose halo is
// the smallest share.  Two gases in FP64 take three (five would need 390
// registers, one wavefront per SIMD).  The line between the two, us per step
// with two nodes per lane / with more: FP64 200 000 nodes 3.8 / 5.2 (two gases
// 6.0 / 6.3), 300 000 5.1 / 5.3 (7.1 / 6.6); FP32 300 000 4.0 / 6.7, 400 000
// 4.7 / 6.8 (6.1 / 7.5).  Six steps of five nodes: 2^24 nodes of one gas in FP64
// take 600 us where one step per launch took 1116 (HBM-bound); 16384 nodes 2.7 us
// per step where a launch per step took 14.
struct TubeShape {
    int J, K;
};
constexpr int64_t kTubeShort64 = 200000, kTubeShort32 = 400000;
TubeShape tube_shape(int64_t nx, bool species, bool fp64)
{
    if (nx <= 32 * 1024) return {2, 8};
    if (nx <= 56 * 1024) return {2, 6};
    if (nx <= (fp64 ? kTubeShort64 : kTubeShort32)) return {2, 4};
    return species && fp64 ? TubeShape{3, 3} : TubeShape{5, 6};
}
template <typename T, bool SP>
constexpr int kLongJ = tube_lanes(SP, sizeof(T) == 8);

}  // namespace

int64_t step_blocks_1d(const Grid& g)
{
    // (the fewest nodes per wavefront of each: 8 steps of J = 2; 6 of J = 5, 3 of J = 3)
    return g.nx <= kTubeShort32 ? tube_blocks(g.nx, 2, 8) : tube_blocks(g.nx, 3, 3);
}

int tube_group(const Grid& g, const Consts& k, bool fp64) { return tube_shape(g.nx, k.species, fp64).K; }

template <typename T, bool SP, int J>
static hipError_t launch_tube_j(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, double* partials,
                                long long step0, int steps, int in_buf, hipStream_t stream)
{
    tube_kernel<T, SP, J><<<(unsigned)tube_blocks(g.nx, J, steps), kTubeTPB, 0, stream>>>(
        Y, Yn, g.nx, g.bc_x, k, ctl, partials, step0, steps, tube_tiles(g.nx, J, steps), in_buf);
    return hipGetLastError();
}

template <typename T, bool SP, int J>
static hipError_t launch_tube_again_j(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, int K, int steps,
                                      hipStream_t stream)
{
    tube_again_kernel<T, SP, J><<<(unsigned)tube_blocks(g.nx, J, K), kTubeTPB, 0, stream>>>(
        Y, Yn, g.nx, g.bc_x, k, ctl, tube_tiles(g.nx, J, K), K, steps);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tube(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, double* partials,
                       long long step0, int steps, int in_buf, hipStream_t stream)
{
    const bool shrt = tube_shape(g.nx, k.species, sizeof(T) == 8).J == 2;
    if (k.species)
        return shrt ? launch_tube_j<T, true, 2>(Y, Yn, g, k, ctl, partials, step0, steps, in_buf, stream)
                    : launch_tube_j<T, true, kLongJ<T, true>>(Y, Yn, g, k, ctl, partials, step0, steps, in_buf, stream);
    return shrt ? launch_tube_j<T, false, 2>(Y, Yn, g, k, ctl, partials, step0, steps, in_buf, stream)
                : launch_tube_j<T, false, kLongJ<T, false>>(Y, Yn, g, k, ctl, partials, step0, steps, in_buf, stream);
}

template <typename T>
hipError_t launch_tube_again(const T* Y, T* Yn, const Grid& g, const Consts& k, StepCtl* ctl, int K, int steps,
                             hipStream_t stream)
{
    const bool shrt = tube_shape(g.nx, k.species, sizeof(T) == 8).J == 2;
    if (k.species)
        return shrt ? launch_tube_again_j<T, true, 2>(Y, Yn, g, k, ctl, K, steps, stream)
                    : launch_tube_again_j<T, true, kLongJ<T, true>>(Y, Yn, g, k, ctl, K, steps, stream);
    return shrt ? launch_tube_again_j<T, false, 2>(Y, Yn, g, k, ctl, K, steps, stream)
                : launch_tube_again_j<T, false, kLongJ<T, false>>(Y, Yn, g, k, ctl, K, steps, stream);
}

hipError_t launch_tube_finalize(const Grid& g, const Consts& k, bool fp64, StepCtl* ctl, double* partials,
                                long long step0, int steps, hipStream_t stream)
{
    const int J = tube_shape(g.nx, k.species, fp64).J;
    int64_t nb = tube_blocks(g.nx, J, steps), stride = 1;
    if (nb > 16 * kChunk) {  // many rows: fold each chunk first, on many CUs
        const int64_t n = (nb + kChunk - 1) / kChunk;
        tube_chunk_kernel<<<(unsigned)n, kChunk, 0, stream>>>(partials, nb, ctl);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        nb = n;
        stride = kChunk;
    }
    if (nb >= kFinManyRows)
        tube_finalize_kernel<kFinMaxTPB><<<1, kFinMaxTPB, 0, stream>>>(partials, nb, stride, ctl, step0, steps, g.nx, J);
    else
        tube_finalize_kernel<kFinTPB><<<1, kFinTPB, 0, stream>>>(partials, nb, stride, ctl, step0, steps, g.nx, J);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_lanes_tube(const T* Y, const Grid& g, const Consts& k, int32_t* fx, int32_t* fy, int32_t* c1,
                             hipStream_t stream)
{
    const unsigned nb = (unsigned)((g.nx + kTubeTPB - 1) / kTubeTPB);
    if (k.species) tube_lanes_kernel<T, true><<<nb, kTubeTPB, 0, stream>>>(Y, g.nx, k, fx, fy, c1);
    else tube_lanes_kernel<T, false><<<nb, kTubeTPB, 0, stream>>>(Y, g.nx, k, fx, fy, c1);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pool1d(const PoolView& v, const Consts& k, int K, int steps, int nblocks, int nslots, int commit,
                         hipStream_t stream)
{
    constexpr int J = kLongJ<T, false>, JS = kLongJ<T, true>;
    if (k.species) pool_tube_kernel<T, true, JS><<<nblocks, kTubeTPB, 0, stream>>>(v, k, K, steps, commit);
    else pool_tube_kernel<T, false, J><<<nblocks, kTubeTPB, 0, stream>>>(v, k, K, steps, commit);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    pool_tube_finalize_kernel<<<nslots, kFinTPB, 0, stream>>>(v, steps, commit);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_pool1d_again(const PoolView& v, const Consts& k, int K, int nblocks, hipStream_t stream)
{
    constexpr int J = kLongJ<T, false>, JS = kLongJ<T, true>;
    if (k.species) pool_tube_again_kernel<T, true, JS><<<nblocks, kTubeTPB, 0, stream>>>(v, k, K);
    else pool_tube_again_kernel<T, false, J><<<nblocks, kTubeTPB, 0, stream>>>(v, k, K);
    return hipGetLastError();
}

hipError_t launch_pool2d_finalize(const PoolView& v, int nslots, int commit, hipStream_t stream)
{
    pool_finalize_kernel<<<nslots, kFinTPB, 0, stream>>>(v, commit);
    return hipGetLastError();
}

hipError_t launch_finalize(double* partials, int64_t nb, StepCtl* ctl, long long step, int in_buf,
                           hipStream_t stream, bool species2d, const int* nch)
{
    const int sp2 = species2d ? 1 : 0;
    if (nb > 16 * kChunk) {  // many rows: fold each chunk first, on many CUs
        const int64_t g = (nb + kChunk - 1) / kChunk;
        partials_chunk_kernel<<<(unsigned)g, kChunk, 0, stream>>>(partials, nb, ctl, step, nch);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        finalize_kernel<kFinTPB><<<1, kFinTPB, 0, stream>>>(partials, g, kChunk, ctl, step, sp2, nullptr, in_buf);
        return hipGetLastError();
    }
    if (nb >= kFinManyRows)
        finalize_kernel<kFinMaxTPB><<<1, kFinMaxTPB, 0, stream>>>(partials, nb, 1, ctl, step, sp2, nch, in_buf);
    else
        finalize_kernel<kFinTPB><<<1, kFinTPB, 0, stream>>>(partials, nb, 1, ctl, step, sp2, nch, in_buf);
    return hipGetLastError();
}

template hipError_t launch_tube<double>(const double*, double*, const Grid&, const Consts&, StepCtl*, double*, long long,
                                        int, int, hipStream_t);
template hipError_t launch_tube<float>(const float*, float*, const Grid&, const Consts&, StepCtl*, double*, long long,
                                       int, int, hipStream_t);
template hipError_t launch_tube_again<double>(const double*, double*, const Grid&, const Consts&, StepCtl*, int, int,
                                              hipStream_t);
template hipError_t launch_tube_again<float>(const float*, float*, const Grid&, const Consts&, StepCtl*, int, int,
                                             hipStream_t);
template hipError_t launch_lanes_tube<double>(const double*, const Grid&, const Consts&, int32_t*, int32_t*, int32_t*,
                                              hipStream_t);
template hipError_t launch_lanes_tube<float>(const float*, const Grid&, const Consts&, int32_t*, int32_t*, int32_t*,
                                             hipStream_t);
template hipError_t launch_pool1d<double>(const PoolView&, const Consts&, int, int, int, int, int, hipStream_t);
template hipError_t launch_pool1d<float>(const PoolView&, const Consts&, int, int, int, int, int, hipStream_t);
template hipError_t launch_pool1d_again<double>(const PoolView&, const Consts&, int, int, hipStream_t);
template hipError_t launch_pool1d_again<float>(const PoolView&, const Consts&, int, int, hipStream_t);

}  // namespace lbsd
