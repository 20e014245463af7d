// pm_kernels.hip -- gfx950 kernels of the MRT lattice Boltzmann update for
// power-law natural convection in a porous cavity (arXiv:2011.15073).
//
// One time step is one fused kernel over all nodes: gather the 9 + 5
// populations, collide (D2Q9 MRT with buoyancy and porous drag, Eq. 12;
// local power-law viscosity, Eqs. 21-23; D2Q5 MRT, Eq. 18) and scatter.
// Memory follows the AA pattern: a single copy of the populations, updated in
// place.
//   even step: node x reads its own slots f_q(x), writes f*_q to slot opp(q)
//              of the same node (no streaming);
//   odd step:  node x pulls f_q from slot opp(q) of node x - e_q and pushes
//              f*_q to slot q of node x + e_q, which completes the streaming
//              of both steps.
// Each node reads and writes exactly the same 14 addresses in a step, so the
// update is race-free without a second buffer; the walls (halfway
// bounce-back, thermal anti-bounce-back) are applied on the odd step's pull
// and push.  Every population is read once and written once per step: the
// algorithmic traffic is 14 * 2 * sizeof(T) bytes per node update.
//
// Each grid row stores its 9 + 5 population rows one after the other (x
// fastest, rows padded to 64 elements), so a node update touches one
// contiguous block per grid row; one workgroup covers a row segment of 64,
// 128 or 256 nodes (chosen by the host from the grid size and dtype), one
// lane per node, so every load and store of a wave is a contiguous 256 B
// (FP32) run; workgroups run in row-major tile order (in XCD bands, with
// cached loads, while the state fits the last-level cache: NEAR).  The
// streaming hint is used on every access that is not shifted along x (those
// lines are touched exactly once per step); the x-shifted accesses of the odd
// step straddle lines that the neighbouring wave also touches, so they keep
// the default caching.
#include "pm_device.h"

#include <algorithm>
#include <type_traits>

namespace pm {
namespace {

using namespace pm::dev;

// One workgroup per row segment of blockDim.x nodes (64, 128 or 256).
// NEAR (the state fits the last-level cache, NEAR_BYTES): tiles in XCD bands
// and cached loads; otherwise launch order and streaming loads.  us per step,
// streaming / near: FP32 64^2 3.6 / 3.2, 256^2 4.5 / 3.8, 1024^2 21.4 / 20.3,
// 2048^2 72.5 / 66.7 (3000^2 164 / 182); FP64 160^2 5.4 / 4.7, 512^2 13.0 /
// 12.0, 1500^2 86.5 / 80.3 (2048^2 159 / 166); FP16 storage 256^2 4.0 / 3.5,
// 1024^2 17.0 / 15.4, 3000^2 111 / 101 (4096^2 207 / 211).
template <typename T, bool ODD, bool POW, bool LOGDA, bool SR, bool NEAR, typename S>
__global__ __launch_bounds__(TILE) void k_step(KParams<T, S> p, int tiles_x, int ntiles) {
  const int tile = NEAR ? band_of_block(blockIdx.x, ntiles) : blockIdx.x;
  const int j = tile / tiles_x;
  step_tile<T, ODD, POW, LOGDA, SR, NEAR>(p, p, (tile - j * tiles_x) * (int)blockDim.x, j, threadIdx.x);
}

// The same step, read from state src and written to state dst (another
// buffer of the same layout).
template <typename T, bool ODD, bool POW, bool LOGDA, bool SR, bool NEAR>
__global__ __launch_bounds__(TILE) void k_step_oop(KParams<T> src, KParams<T> dst, int tiles_x, int ntiles) {
  const int tile = NEAR ? band_of_block(blockIdx.x, ntiles) : blockIdx.x;
  const int j = tile / tiles_x;
  step_tile<T, ODD, POW, LOGDA, SR, NEAR>(src, dst, (tile - j * tiles_x) * (int)blockDim.x, j, threadIdx.x);
}

// ---- batched parameter sweep: one launch steps every live case ----
// Workgroup b takes the (case, tile) pair of entry b of the schedule; cases
// that have met their stopping test are skipped.  A tile is tw columns by th
// rows (tw a multiple of 64, tw * th threads): thread t works on column
// t % tw, row t / tw of the tile, so every wave lies within one grid row.
// Each case runs the same per-node body as the single-case kernel, so a case
// advanced here is bitwise identical to the same case advanced alone,
// whatever the tile shape.  SR_ANY: some case rounds stochastically (FP32
// only); without it the kernel carries no stochastic-rounding branch, which
// would cost round-to-nearest sweeps registers and occupancy.  NEAR (as in
// k_step): the states of the cases in this launch fit the last-level cache
// together.  27 FP32 cases (185 MB): 56.5 us per step near, 62.2 streaming; in
// FP64 (370 MB in one launch) near would be 141 against 130.
template <typename T, bool ODD, bool SR_ANY, bool NEAR>
__global__ __launch_bounds__(TILE) void k_step_multi(const SweepCase<T>* __restrict__ cases,
                                                     const int2* __restrict__ sched,
                                                     const int* __restrict__ live, int tw, int th) {
  const int2 e = sched[NEAR ? band_of_block(blockIdx.x, gridDim.x) : blockIdx.x];  // (case, tile within the case)
  if (!live[e.x]) return;
  const SweepCase<T>& c = cases[e.x];
  const int ty = e.y / c.tiles_x;
  const int lx = (int)threadIdx.x % tw, j = ty * th + (int)threadIdx.x / tw;
  if (j >= c.p.ny) return;  // whole waves
  const int i0 = (e.y - ty * c.tiles_x) * tw;
  if constexpr (SR_ANY && std::is_same<T, float>::value) {
    if (c.p.sr) {
      if (c.pow) step_tile<T, ODD, true, false, true, NEAR>(c.p, c.p, i0, j, lx);
      else step_tile<T, ODD, false, false, true, NEAR>(c.p, c.p, i0, j, lx);
      return;
    }
  }
  if (c.pow) step_tile<T, ODD, true, false, false, NEAR>(c.p, c.p, i0, j, lx);
  else step_tile<T, ODD, false, false, false, NEAR>(c.p, c.p, i0, j, lx);
}

// Rest state: df = 0, dg_q = w_q (T_init - T_ref).  (The padding of the
// population region is cleared by the launcher.)
template <typename T, typename S>
__global__ void k_init(KParams<T, S> p, T dg_init) {
  const int64_t n = (int64_t)p.nx * p.ny;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(k / p.nx), i = (int)(k - (int64_t)j * p.nx);
    const int64_t o = pop_off(p, i, j);
#pragma unroll
    for (int q = 0; q < 9; ++q) p.f[q * p.qs + o] = S(0);
    p.g[o] = (S)(dg_init * T(2));  // w_0 = 1/3 = 2 w_1
#pragma unroll
    for (int q = 1; q < 5; ++q) p.g[q * p.qs + o] = (S)dg_init;
  }
}

// Eq. (24): one wave per 64 rows (and per further 64 NU_BLOCKS), its sum into
// its slot of partial; the host adds the slots in order, so the order of
// summation is fixed.  Every value read is in a cache line of its own, so that
// the rows are spread over the CUs: 2048 rows took 35 us by one workgroup of 256,
// pm_nu 59 us; like this pm_nu takes 18 us at any size up to 4096^2.
template <typename T, typename S>
__global__ __launch_bounds__(64) void k_nu(KParams<T, S> p, int parity, double* __restrict__ partial) {
  double acc = 0.0;
  for (int64_t j0 = (int64_t)blockIdx.x * 64 + threadIdx.x; j0 < p.ny; j0 += (int64_t)gridDim.x * 64) {
    const int j = (int)j0;
    T g0[5], g1[5];
    if (parity) {
      load_g<T, true>(p, 0, j, g0);
      load_g<T, true>(p, 1, j, g1);
    } else {
      load_g<T, false>(p, 0, j, g0);
      load_g<T, false>(p, 1, j, g1);
    }
    const double t0 = (double)p.T_ref + (double)(g0[0] + ((g0[1] + g0[2]) + (g0[3] + g0[4])));
    const double t1 = (double)p.T_ref + (double)(g1[0] + ((g1[1] + g1[2]) + (g1[3] + g1[4])));
    acc += (double)p.nx * (8.0 - 9.0 * t0 + t1) / 3.0;
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off);
  if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// max over the workgroup's threads, in thread 0 (values >= 0).
__device__ __forceinline__ double block_max(double mx) {
  __shared__ double red[TILE / 64];
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_down(mx, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < ((int)blockDim.x + 63) / 64; ++w) mx = fmax(mx, red[w]);
  return mx;
}

// Residual: per-workgroup max |theta - snapshot|, snapshot := theta.  Each wave
// takes RESID_SEGS segments of 64 nodes of a row at a time, so that their loads
// are in flight together: it is bound by those, 5 + 1 values read and one
// written per node.  us per call, 1 / 2 / 4 segments: 2048^2 FP32 30.6 / 31.0 /
// 30.5, 4096^2 FP32 odd step count 111 / 108 / 100, 3000^2 FP64 102 / 104 / 106
// (one thread per node with 64-bit divisions, and the maximum by a second
// kernel and a copy: 41, 121 and 117).
constexpr int RESID_SEGS = 2;
template <typename T, typename S>
__global__ __launch_bounds__(256) void k_resid(KParams<T, S> p, int parity, T* __restrict__ snap,
                                               double* __restrict__ partial, int snapshot_only) {
  double mx = 0.0;
  const int segs = (p.nx + 63) / 64, lane = threadIdx.x & 63;
  const int n = segs * p.ny;  // at most the number of nodes, below 2^30
  const int s0 = ((int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) * RESID_SEGS;
  for (int s = s0; s < n; s += (int)gridDim.x * 4 * RESID_SEGS) {
    T g[RESID_SEGS][5], old[RESID_SEGS];
    int64_t k[RESID_SEGS];
    bool in[RESID_SEGS];
#pragma unroll
    for (int t = 0; t < RESID_SEGS; ++t) {  // no branches: a lane past the end repeats the last node
      const int st = min(s + t, n - 1), j = st / segs, i = (st - j * segs) * 64 + lane, ic = min(i, p.nx - 1);
      in[t] = s + t < n && i < p.nx;
      k[t] = (int64_t)j * p.nx + ic;
      if (parity) load_g<T, true>(p, ic, j, g[t]); else load_g<T, false>(p, ic, j, g[t]);
      old[t] = snap[k[t]];
    }
#pragma unroll
    for (int t = 0; t < RESID_SEGS; ++t) {
      const T dT = g[t][0] + ((g[t][1] + g[t][2]) + (g[t][3] + g[t][4]));
      double d = fabs((double)dT - (double)old[t]);
      if (!(d <= 1.7976931348623157e308)) d = INFINITY;  // NaN / Inf -> +Inf
      mx = in[t] && d > mx ? d : mx;
      if (in[t]) snap[k[t]] = dT;
    }
  }
  mx = block_max(mx);
  if (threadIdx.x == 0 && !snapshot_only) partial[blockIdx.x] = mx;
}

// Sweep residual: one workgroup per schedule entry (a tile of a live case,
// laid out as in k_step_multi) -> max |theta - snapshot| over the tile into
// the tile's slot of the case-major partial array, snapshot := theta.
template <typename T>
__global__ __launch_bounds__(TILE) void k_resid_multi(const SweepCase<T>* __restrict__ cases,
                                                      const int2* __restrict__ sched,
                                                      const int* __restrict__ live, int parity,
                                                      double* __restrict__ partial, int tw, int th) {
  const int2 e = sched[blockIdx.x];
  if (!live[e.x]) return;  // uniform over the workgroup
  const SweepCase<T>& c = cases[e.x];
  const int ty = e.y / c.tiles_x;
  const int j = ty * th + (int)threadIdx.x / tw;
  const int i = (e.y - ty * c.tiles_x) * tw + (int)threadIdx.x % tw;
  double mx = 0.0;
  if (i < c.p.nx && j < c.p.ny) {
    T g[5];
    if (parity) load_g<T, true>(c.p, i, j, g); else load_g<T, false>(c.p, i, j, g);
    const T dT = g[0] + ((g[1] + g[2]) + (g[3] + g[4]));
    const int64_t k = (int64_t)j * c.p.nx + i;
    double d = fabs((double)dT - (double)c.snap[k]);
    if (!(d <= 1.7976931348623157e308)) d = INFINITY;  // NaN / Inf -> +Inf
    mx = d;
    c.snap[k] = dT;
  }
  mx = block_max(mx);
  if (threadIdx.x == 0) partial[c.tile_base + e.y] = mx;
}

// Stopping test of every live case after a chunk of steps: r = max over the
// case's tiles; the case stops when r < tol, when r is not finite, or when
// it has reached max_steps.  One workgroup per case (a thread per case took
// 104 us for the 27-case sweep, a chain of up to 2048 loads).
template <typename T>
__global__ __launch_bounds__(TILE) void k_retire(const SweepCase<T>* __restrict__ cases,
                                                 const double* __restrict__ partial, int* __restrict__ live,
                                                 SweepStatus* __restrict__ st, int64_t chunk, double tol,
                                                 int64_t max_steps) {
  const int c = blockIdx.x;
  if (!live[c]) return;  // uniform over the workgroup
  const SweepCase<T>& cs = cases[c];
  double r = 0.0;
  for (int b = threadIdx.x; b < cs.ntiles; b += TILE) r = fmax(r, partial[cs.tile_base + b]);
  r = block_max(r);
  if (threadIdx.x) return;
  st[c].steps += chunk;
  st[c].residual = r;
  const bool finite = r <= 1.7976931348623157e308;
  if (r < tol || !finite || st[c].steps >= max_steps) live[c] = 0;
}

template <typename T, bool ODD, bool POW, bool LOGDA, typename O, typename S>
__global__ __launch_bounds__(TILE) void k_fields(KParams<T, S> p, O* U, O* V, O* th, O* nuo) {
  const int i = blockIdx.x * TILE + threadIdx.x;
  if (i >= p.nx) return;
  for (int j = blockIdx.y; j < p.ny; j += gridDim.y) {
    T df[9], dg[5];
    const int k = j * p.nx + i;
    const T ldk = load_logda<LOGDA>(p, k);
    load_node<T, ODD>(p, i, j, df, dg);
    T drho, rho, jx, jy, dT, Gx, Gy, nu, ux, uy, invK, invsK, m1, m7, m8;
    node_macros<T, POW, LOGDA>(p, ldk, df, dg, drho, rho, jx, jy, dT, Gx, Gy, nu, ux, uy, invK,
                               invsK, m1, m7, m8);
    // Streaming stores leave the state in the caches (4096^2 FP32, three fields:
    // 207 -> 193 us); U alone is for the stream function, whose scan reads it next.
    if (U && V) __builtin_nontemporal_store((O)(ux * p.inv_U), &U[k]);
    else if (U) U[k] = (O)(ux * p.inv_U);
    if (V) __builtin_nontemporal_store((O)(uy * p.inv_U), &V[k]);
    if (th) __builtin_nontemporal_store((O)(p.T_ref + dT), &th[k]);
    if (nuo) __builtin_nontemporal_store((O)nu, &nuo[k]);
  }
}

// D2Q9 / D2Q5 rest weights for the absolute <-> shifted conversions.
template <typename T>
__device__ __forceinline__ T w9(int q) {
  return q == 0 ? T(4.0 / 9.0) : (q < 5 ? T(1.0 / 9.0) : T(1.0 / 36.0));
}
template <typename T>
__device__ __forceinline__ T w5(int q) {
  return q == 0 ? T(1.0 / 3.0) : T(1.0 / 6.0);
}

// Bound by its traffic, one read and one write of the state.  STREAM (each
// wave's piece of a row is whole lines): streaming stores, which leave the state
// in the caches (2048^2 FP32 at an odd step count 82 -> 72 us, 4096^2 332 -> 317);
// a line that two waves write parts of would go to memory twice (2049 x 2047
// 79 -> 136, 1500 x 1031 34 -> 42, 100 x 40000 88 -> 119).
template <typename T, bool ODD, typename O, bool STREAM, typename S>
__global__ __launch_bounds__(TILE) void k_get_pop(KParams<T, S> p, O* f, O* g) {
  const int i = blockIdx.x * TILE + threadIdx.x;
  if (i >= p.nx) return;
  const int64_t n = (int64_t)p.nx * p.ny;
  auto put = [](O* a, double v) {
    if constexpr (STREAM) __builtin_nontemporal_store((O)v, a);
    else *a = (O)v;
  };
  for (int j = blockIdx.y; j < p.ny; j += gridDim.y) {
    T df[9], dg[5];
    load_node<T, ODD>(p, i, j, df, dg);
    const int64_t k = (int64_t)j * p.nx + i;
#pragma unroll
    for (int q = 0; q < 9; ++q) put(&f[q * n + k], (double)df[q] + (double)w9<T>(q));
#pragma unroll
    for (int q = 0; q < 5; ++q) put(&g[q * n + k], (double)dg[q] + (double)w5<T>(q) * (double)p.T_ref);
  }
}

template <typename T, typename I, typename S>
__global__ __launch_bounds__(TILE) void k_set_pop(KParams<T, S> p, const I* f, const I* g) {
  const int i = blockIdx.x * TILE + threadIdx.x;
  if (i >= p.nx) return;
  const int64_t n = (int64_t)p.nx * p.ny;
  for (int j = blockIdx.y; j < p.ny; j += gridDim.y) {
    const int64_t k = (int64_t)j * p.nx + i, o = pop_off(p, i, j);
#pragma unroll
    for (int q = 0; q < 9; ++q) p.f[q * p.qs + o] = (S)((double)f[q * n + k] - (double)w9<T>(q));
#pragma unroll
    for (int q = 0; q < 5; ++q)
      p.g[q * p.qs + o] = (S)((double)g[q * n + k] - (double)w5<T>(q) * (double)p.T_ref);
  }
}

template <typename T, typename I>
__global__ void k_convert(T* dst, const I* src, int64_t n) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.x * blockDim.x)
    dst[k] = (T)src[k];
}

__global__ void k_header(int64_t* dst, int64_t steps, uint64_t tag, uint64_t phys) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    dst[0] = (int64_t)tag;
    dst[1] = steps;
    dst[2] = (int64_t)phys;
  }
}

// Stream function from the U field, in place: on entry psi holds U at the
// nodes, on exit psi(j) = (sum_{j' < j} U(j') + U(j) / 2) / L up each column
// (the integral of U dy from the bottom wall to the node by the midpoint
// rule), as a blocked scan with FP64 sums: (1) every thread sums one
// column over one block of R rows; (2) one thread per column turns the
// block sums into exclusive block offsets; (3) every (column, block) thread
// walks its rows from its block's offset.  A wave reads 64 adjacent columns
// of a row at a time, so every access is contiguous.
// Rows per block: 64, doubled until the block count fits a launch's y extent.
inline int psi_rows(int ny) {
  int r = 64;
  while ((ny + r - 1) / r > GRID_Y_MAX) r *= 2;
  return r;
}

// Rows whose loads are in flight together: a column's block is a chain of memory
// round trips otherwise, and there are few waves (2048^2: one per SIMD).  Stream
// function of a 1024^2 FP32 state with groups of 8 / 16 / 32: 38.0 / 36.3 / 35.7
// us, 501^2 31.4 / 29.8 / 32.8 (stores between the loads: 43.2 and 35.6).
constexpr int PSI_GROUP = 16;

template <typename O>
__global__ __launch_bounds__(256) void k_psi_blocks(const O* __restrict__ u, double* __restrict__ blk, int nx,
                                                    int ny, int R) {
  const int i = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (i >= nx) return;
  const int j1 = (int)min((int64_t)ny, (int64_t)(b + 1) * R);
  double s = 0.0;
#pragma unroll PSI_GROUP
  for (int j = b * R; j < j1; ++j) s += (double)u[(int64_t)j * nx + i];
  blk[(int64_t)b * nx + i] = s;
}

// Exclusive prefix over the block sums of each column, in order.  The sums
// are loaded 16 at a time before any is overwritten, so the loads of a
// group are in flight together.
__global__ __launch_bounds__(256) void k_psi_offsets(double* __restrict__ blk, int nx, int nblk) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= nx) return;
  constexpr int G = 16;
  double acc = 0.0;
  for (int b0 = 0; b0 < nblk; b0 += G) {
    double s[G];
#pragma unroll
    for (int t = 0; t < G; ++t) s[t] = b0 + t < nblk ? blk[(int64_t)(b0 + t) * nx + i] : 0.0;
#pragma unroll
    for (int t = 0; t < G; ++t) {
      if (b0 + t < nblk) blk[(int64_t)(b0 + t) * nx + i] = acc;
      acc += s[t];
    }
  }
}

template <typename O>
__global__ __launch_bounds__(256) void k_psi_apply(O* __restrict__ psi, const double* __restrict__ blk, int nx,
                                                   int ny, int R, double inv_L) {
  const int i = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
  if (i >= nx) return;
  const int j1 = (int)min((int64_t)ny, (int64_t)(b + 1) * R);
  double acc = blk[(int64_t)b * nx + i];
  for (int j = b * R; j < j1; j += PSI_GROUP) {
    O u[PSI_GROUP];  // all loads of a group before its first store (the field is overwritten in place)
#pragma unroll
    for (int t = 0; t < PSI_GROUP; ++t) u[t] = psi[(int64_t)min(j + t, j1 - 1) * nx + i];
#pragma unroll
    for (int t = 0; t < PSI_GROUP; ++t) {
      if (j + t < j1) psi[(int64_t)(j + t) * nx + i] = (O)((acc + 0.5 * (double)u[t]) * inv_L);
      acc += (double)u[t];
    }
  }
}

typedef float v4f __attribute__((ext_vector_type(4)));

// One 16-byte vector per thread, streaming (non-temporal) load and store.
__global__ __launch_bounds__(256) void k_copy(const v4f* __restrict__ src, v4f* __restrict__ dst,
                                              int64_t n) {
  const int64_t k = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (k < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + k), dst + k);
}

inline int grid_for(int64_t n, int per = 256, int cap = 65536) {
  int64_t b = (n + per - 1) / per;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (int)b;
}

}  // namespace

template <typename T, typename S>
hipError_t launch_step(const KParams<T, S>& p, const Launch& L, int parity, bool pow, bool logda) {
  if (!(L.step_w == 64 || L.step_w == 128 || L.step_w == 256) || L.step_w > TILE) return hipErrorInvalidValue;
  dim3 grid(L.step_ntiles), block(L.step_w);
#define PM_STEP(ODD, POW, LOG, SR)                                                                              \
  do {                                                                                                         \
    if (L.near)                                                                                                \
      hipLaunchKernelGGL((k_step<T, ODD, POW, LOG, SR, true, S>), grid, block, 0, L.stream, p, L.step_tiles_x,  \
                         L.step_ntiles);                                                                       \
    else                                                                                                       \
      hipLaunchKernelGGL((k_step<T, ODD, POW, LOG, SR, false, S>), grid, block, 0, L.stream, p, L.step_tiles_x, \
                         L.step_ntiles);                                                                       \
  } while (0)
#define PM_STEP_ALL(SR)                                                                             \
  if (parity) {                                                                                     \
    if (pow) { if (logda) PM_STEP(true, true, true, SR); else PM_STEP(true, true, false, SR); }       \
    else { if (logda) PM_STEP(true, false, true, SR); else PM_STEP(true, false, false, SR); }        \
  } else {                                                                                          \
    if (pow) { if (logda) PM_STEP(false, true, true, SR); else PM_STEP(false, true, false, SR); }    \
    else { if (logda) PM_STEP(false, false, true, SR); else PM_STEP(false, false, false, SR); }     \
  }
  bool done = false;
  if constexpr (std::is_same<T, float>::value) {
    if (p.sr) {
      PM_STEP_ALL(true)
      done = true;
    }
  }
  if (!done) { PM_STEP_ALL(false) }
#undef PM_STEP_ALL
#undef PM_STEP
  return hipGetLastError();
}

template <typename T>
hipError_t launch_step_oop(const KParams<T>& src, const KParams<T>& dst, const Launch& L, int parity,
                           bool pow, bool logda) {
  if (!(L.step_w == 64 || L.step_w == 128 || L.step_w == 256) || L.step_w > TILE) return hipErrorInvalidValue;
  dim3 grid(L.step_ntiles), block(L.step_w);
#define PM_OOP(ODD, POW, LOG, SR)                                                                           \
  do {                                                                                                     \
    if (L.near)                                                                                            \
      hipLaunchKernelGGL((k_step_oop<T, ODD, POW, LOG, SR, true>), grid, block, 0, L.stream, src, dst,      \
                         L.step_tiles_x, L.step_ntiles);                                                   \
    else                                                                                                   \
      hipLaunchKernelGGL((k_step_oop<T, ODD, POW, LOG, SR, false>), grid, block, 0, L.stream, src, dst,     \
                         L.step_tiles_x, L.step_ntiles);                                                   \
  } while (0)
#define PM_OOP_ALL(SR)                                                                              \
  if (parity) {                                                                                     \
    if (pow) { if (logda) PM_OOP(true, true, true, SR); else PM_OOP(true, true, false, SR); }         \
    else { if (logda) PM_OOP(true, false, true, SR); else PM_OOP(true, false, false, SR); }          \
  } else {                                                                                          \
    if (pow) { if (logda) PM_OOP(false, true, true, SR); else PM_OOP(false, true, false, SR); }      \
    else { if (logda) PM_OOP(false, false, true, SR); else PM_OOP(false, false, false, SR); }       \
  }
  bool done = false;
  if constexpr (std::is_same<T, float>::value) {
    if (src.sr) {
      PM_OOP_ALL(true)
      done = true;
    }
  }
  if (!done) { PM_OOP_ALL(false) }
#undef PM_OOP_ALL
#undef PM_OOP
  return hipGetLastError();
}

template <typename T>
hipError_t launch_step_multi(const SweepCase<T>* cases, const int2* sched, const int* live,
                             int nsched, int parity, int tw, int th, bool any_sr, bool near, hipStream_t s) {
  if (!sweep_tile_ok(tw, th)) return hipErrorInvalidValue;
  if (nsched <= 0) return hipSuccess;  // no live case scheduled
#define PM_MULTI(ODD, SR)                                                                                            \
  do {                                                                                                              \
    if (near)                                                                                                       \
      hipLaunchKernelGGL((k_step_multi<T, ODD, SR, true>), dim3(nsched), dim3(tw * th), 0, s, cases, sched, live, tw, \
                         th);                                                                                       \
    else                                                                                                            \
      hipLaunchKernelGGL((k_step_multi<T, ODD, SR, false>), dim3(nsched), dim3(tw * th), 0, s, cases, sched, live,   \
                         tw, th);                                                                                   \
  } while (0)
  bool sr = false;
  if constexpr (std::is_same<T, float>::value) {
    sr = any_sr;
    if (sr) {
      if (parity) PM_MULTI(true, true); else PM_MULTI(false, true);
    }
  }
  if (!sr) {
    if (parity) PM_MULTI(true, false); else PM_MULTI(false, false);
  }
#undef PM_MULTI
  return hipGetLastError();
}

template <typename T>
hipError_t launch_resid_multi(const SweepCase<T>* cases, int ncases, const int2* sched, int* live,
                              int nsched, int parity, int tw, int th, double* partial, SweepStatus* st,
                              int64_t chunk, double tol, int64_t max_steps, hipStream_t s) {
  if (!sweep_tile_ok(tw, th)) return hipErrorInvalidValue;
  if (nsched <= 0) return hipSuccess;  // no live case scheduled
  hipLaunchKernelGGL((k_resid_multi<T>), dim3(nsched), dim3(tw * th), 0, s, cases, sched,
                     (const int*)live, parity, partial, tw, th);
  hipLaunchKernelGGL((k_retire<T>), dim3(ncases), dim3(TILE), 0, s, cases, (const double*)partial, live, st,
                     chunk, tol, max_steps);
  return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_init(const KParams<T, S>& p, const Launch& L, T dg_init, size_t pop_bytes) {
  // whole population region first (row padding included), then the nodes
  hipError_t e = hipMemsetAsync(p.f, 0, pop_bytes, L.stream);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_init<T, S>), dim3(grid_for((int64_t)p.nx * p.ny)), dim3(256), 0, L.stream,
                     p, dg_init);
  return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_nu(const KParams<T, S>& p, const Launch& L, int parity, double* partial, int* n) {
  *n = std::min((p.ny + 63) / 64, RED_BLOCKS);
  hipLaunchKernelGGL((k_nu<T, S>), dim3(*n), dim3(64), 0, L.stream, p, parity, partial);
  return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_residual(const KParams<T, S>& p, const Launch& L, int parity, T* snap, double* partial, int* n,
                           int snapshot_only) {
  *n = grid_for((int64_t)((p.nx + 63) / 64) * p.ny, 4 * RESID_SEGS, RED_BLOCKS);
  hipLaunchKernelGGL((k_resid<T, S>), dim3(*n), dim3(256), 0, L.stream, p, parity, snap, partial, snapshot_only);
  return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_fields(const KParams<T, S>& p, const Launch& L, int parity, bool pow, bool logda,
                         void* U, void* V, void* th, void* nu, int out_fp64) {
  dim3 grid(L.tiles_x, std::min(p.ny, GRID_Y_MAX)), block(TILE);
#define PM_F(ODD, POW, LOG, O)                                                              \
  hipLaunchKernelGGL((k_fields<T, ODD, POW, LOG, O, S>), grid, block, 0, L.stream, p, (O*)U, \
                     (O*)V, (O*)th, (O*)nu)
#define PM_F2(ODD, POW, LOG) \
  do { if (out_fp64) PM_F(ODD, POW, LOG, double); else PM_F(ODD, POW, LOG, float); } while (0)
#define PM_F3(ODD, POW) \
  do { if (logda) PM_F2(ODD, POW, true); else PM_F2(ODD, POW, false); } while (0)
#define PM_F4(ODD) do { if (pow) PM_F3(ODD, true); else PM_F3(ODD, false); } while (0)
  if (parity) PM_F4(true); else PM_F4(false);
#undef PM_F4
#undef PM_F3
#undef PM_F2
#undef PM_F
  return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_get_pop(const KParams<T, S>& p, const Launch& L, int parity, void* f, void* g,
                          int out_fp64) {
  dim3 grid(L.tiles_x, std::min(p.ny, GRID_Y_MAX)), block(TILE);
  const size_t line = 128;
  const bool stream = (size_t)p.nx * (out_fp64 ? 8 : 4) % line == 0 && ((uintptr_t)f | (uintptr_t)g) % line == 0;
#define PM_G(ODD, O, STREAM) \
  hipLaunchKernelGGL((k_get_pop<T, ODD, O, STREAM, S>), grid, block, 0, L.stream, p, (O*)f, (O*)g)
#define PM_G1(ODD, O) do { if (stream) PM_G(ODD, O, true); else PM_G(ODD, O, false); } while (0)
#define PM_G2(ODD) do { if (out_fp64) PM_G1(ODD, double); else PM_G1(ODD, float); } while (0)
  if (parity) PM_G2(true); else PM_G2(false);
#undef PM_G2
#undef PM_G1
#undef PM_G
  return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_set_pop(const KParams<T, S>& p, const Launch& L, const void* f, const void* g,
                          int in_fp64) {
  dim3 grid(L.tiles_x, std::min(p.ny, GRID_Y_MAX)), block(TILE);
  if (in_fp64)
    hipLaunchKernelGGL((k_set_pop<T, double, S>), grid, block, 0, L.stream, p, (const double*)f, (const double*)g);
  else
    hipLaunchKernelGGL((k_set_pop<T, float, S>), grid, block, 0, L.stream, p, (const float*)f, (const float*)g);
  return hipGetLastError();
}

template <typename T, typename S>
hipError_t launch_set_logda(const KParams<T, S>& p, const Launch& L, T* dst, const void* src,
                            int in_fp64) {
  const int64_t n = (int64_t)p.nx * p.ny;
  if (in_fp64)
    hipLaunchKernelGGL((k_convert<T, double>), dim3(grid_for(n)), dim3(256), 0, L.stream, dst, (const double*)src, n);
  else
    hipLaunchKernelGGL((k_convert<T, float>), dim3(grid_for(n)), dim3(256), 0, L.stream, dst, (const float*)src, n);
  return hipGetLastError();
}

hipError_t launch_write_header(void* dst, int64_t steps, uint64_t tag, uint64_t phys, hipStream_t s) {
  hipLaunchKernelGGL(k_header, dim3(1), dim3(64), 0, s, (int64_t*)dst, steps, tag, phys);
  return hipGetLastError();
}

size_t stream_scratch_bytes(int nx, int ny) {
  const int R = psi_rows(ny);
  return (size_t)nx * (size_t)((ny + R - 1) / R) * sizeof(double);
}

hipError_t launch_stream_y(void* psi, int nx, int ny, double inv_L, int out_fp64, double* scratch,
                           hipStream_t s) {
  const int R = psi_rows(ny), nblk = (ny + R - 1) / R;
  const dim3 grid((unsigned)((nx + 255) / 256), (unsigned)nblk);
  if (out_fp64)
    hipLaunchKernelGGL((k_psi_blocks<double>), grid, dim3(256), 0, s, (const double*)psi, scratch, nx, ny, R);
  else
    hipLaunchKernelGGL((k_psi_blocks<float>), grid, dim3(256), 0, s, (const float*)psi, scratch, nx, ny, R);
  hipLaunchKernelGGL(k_psi_offsets, dim3(grid.x), dim3(256), 0, s, scratch, nx, nblk);
  if (out_fp64)
    hipLaunchKernelGGL((k_psi_apply<double>), grid, dim3(256), 0, s, (double*)psi, (const double*)scratch, nx,
                       ny, R, inv_L);
  else
    hipLaunchKernelGGL((k_psi_apply<float>), grid, dim3(256), 0, s, (float*)psi, (const double*)scratch, nx, ny,
                       R, inv_L);
  return hipGetLastError();
}

hipError_t launch_copy_probe(const void* src, void* dst, size_t bytes, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 16);
  const int64_t blocks = (n + 255) / 256;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)blocks), dim3(256), 0, s, (const v4f*)src, (v4f*)dst, n);
  return hipGetLastError();
}

#define PM_INST_S(T, S)                                                                          \
  template hipError_t launch_step<T, S>(const KParams<T, S>&, const Launch&, int, bool, bool);    \
  template hipError_t launch_init<T, S>(const KParams<T, S>&, const Launch&, T, size_t);          \
  template hipError_t launch_nu<T, S>(const KParams<T, S>&, const Launch&, int, double*, int*);   \
  template hipError_t launch_residual<T, S>(const KParams<T, S>&, const Launch&, int, T*, double*, \
                                            int*, int);                                            \
  template hipError_t launch_fields<T, S>(const KParams<T, S>&, const Launch&, int, bool, bool,   \
                                          void*, void*, void*, void*, int);                        \
  template hipError_t launch_get_pop<T, S>(const KParams<T, S>&, const Launch&, int, void*, void*, \
                                           int);                                                   \
  template hipError_t launch_set_pop<T, S>(const KParams<T, S>&, const Launch&, const void*,      \
                                           const void*, int);                                      \
  template hipError_t launch_set_logda<T, S>(const KParams<T, S>&, const Launch&, T*, const void*, int);
#define PM_INST(T)                                                                              \
  PM_INST_S(T, T)                                                                               \
  template hipError_t launch_step_oop<T>(const KParams<T>&, const KParams<T>&, const Launch&, int, \
                                         bool, bool);                                           \
  template hipError_t launch_step_multi<T>(const SweepCase<T>*, const int2*, const int*, int, int, \
                                           int, int, bool, bool, hipStream_t);                    \
  template hipError_t launch_resid_multi<T>(const SweepCase<T>*, int, const int2*, int*, int, int, \
                                            int, int, double*, SweepStatus*, int64_t, double,     \
                                            int64_t, hipStream_t);
PM_INST(float)
PM_INST(double)
PM_INST_S(float, _Float16)
#undef PM_INST
#undef PM_INST_S

}  // namespace pm
