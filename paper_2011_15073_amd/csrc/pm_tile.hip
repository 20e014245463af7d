// pm_tile.hip -- small cavities: several time steps of a tile in one launch
// (gfx950).
//
// A small cavity leaves a step launch of one time step with little to do: at
// 64^2 a step takes 3.3 us, of which 1.6 are the launch itself (an empty kernel
// in a graph), about one the way from and to the last-level cache, and the
// rest one wave's chain of ~350 instructions on 64 of the 1024 SIMDs.  This
// kernel takes ts steps per launch instead.  Each workgroup reads a region of
// w x h nodes, one node per thread, keeps it in registers, and after each step
// outputs what is still exact: all but the ts rows and columns next to a side
// that is no cavity wall.  Neighbouring regions overlap by 2 ts nodes, so the
// overlap is computed twice and no workgroup waits for another.
//
// Per step a thread collides its node, writes the 12 populations that move to
// their planes in LDS (two buffers in turn, so one barrier per step is enough)
// and reads the 12 that arrive; the addresses, walls included, are worked out
// once per launch.  The rest populations f0 and g0 stay in registers.  The
// per-node arithmetic is the step kernels' (collide), so the populations are
// theirs bit for bit.
//
// Regions are dealt to the XCDs in bands (band_of_block): the lines that the
// regions' edges split and the overlaps then stay within one XCD's L2.  That
// is worth more than anything else here: 256^2 FP32 2.7 us per step in bands,
// 4.1 in launch order.
//
// us per step at n = 0.8, one step per launch / this kernel: FP32 64^2 3.25 / 1.59,
// 128^2 3.35 / 1.80, 256^2 3.80 / 2.69, 384^2 5.31 / 3.72, 512^2 7.12 / 6.46 (640^2
// 9.7 / 9.5: the overlap's share grows; tile_plan ends at 520^2); FP64 64^2 4.29 /
// 2.58, 160^2 4.72 / 3.26, 256^2 5.33 / 4.86 (320^2 7.2 / 7.1: there n != 1 takes one
// step per launch, n = 1 this kernel up to 360^2).
// The time is launch + memory latency (about 2.5 us) and the steps' own chains
// (1.1 us each with one wave per SIMD, 2.6 with four; FP64 2.3 with one).
#include "pm_device.h"

#include <algorithm>
#include <type_traits>

namespace pm {
namespace {

using namespace pm::dev;

// LDS plane of population q (f0..f8, g0..g4 as 0..13; f0 and g0 have none).
constexpr int plane_of(int q) { return q < 9 ? q - 1 : q - 2; }

// NMAX: the largest region (threads per workgroup) of this instance.
template <typename T, bool POW, bool LOGDA, bool SR, int NMAX>
__global__ __launch_bounds__(NMAX) void k_tile(KParams<T> src, T* __restrict__ dst_f, T* __restrict__ dst_g, int tiles_x,
                                               int w, int h, int ts) {
  __shared__ T buf[2][12][NMAX];
  const int tid = threadIdx.x;
  const int tile = band_of_block(blockIdx.x, gridDim.x);
  const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
  const int nx = src.nx, ny = src.ny;
  const int c0 = tx * (w - 2 * ts), r0 = ty * (h - 2 * ts);
  const int cw = min(w, nx - c0), rh = min(h, ny - r0);
  const int row = tid / w, col = tid - row * w;
  const int i = c0 + col, j = r0 + row, k = j * nx + i;
  // Steps after which this node is still exact, at most ts: its distance to the
  // nearest side of the region that is no wall (-1: not in the region).  Step
  // t collides the nodes of depth >= t; those of depth > t then have all
  // their neighbours' results.
  int depth = -1;
  if (col < cw && row < rh) {
    depth = ts;
    if (c0 > 0) depth = min(depth, col);
    if (c0 + cw < nx) depth = min(depth, cw - 1 - col);
    if (r0 > 0) depth = min(depth, row);
    if (r0 + rh < ny) depth = min(depth, rh - 1 - row);
  }
  T f[9] = {}, g[5] = {}, ldk = T(0);
  int from[14] = {};  // where population q is pulled from: plane and thread
  bool hot = false, cold = false;
  if (depth >= 0) {
    const int64_t o = pop_off(src, i, j);
    ldk = load_logda<LOGDA>(src, k);
#pragma unroll
    for (int q = 0; q < 9; ++q) f[q] = src.f[q * src.qs + o];
#pragma unroll
    for (int q = 0; q < 5; ++q) g[q] = src.g[q * src.qs + o];
    // as load_node_raw and pull_walls: from node (i, j) - e_q, or the node's own
    // population in the opposite direction where that crosses a wall
    const bool in_im = i >= 1, in_ip = i + 1 < nx, in_jm = j >= 1, in_jp = j + 1 < ny;
    hot = !in_im;
    cold = !in_ip;
#pragma unroll
    for (int q = 1; q < 14; ++q) {
      if (q == 9) continue;
      const int d = q < 9 ? q : q - 9;  // direction within D2Q9 / D2Q5
      const bool in = (EXv[d] > 0 ? in_im : (EXv[d] < 0 ? in_ip : true)) &
                      (EYv[d] > 0 ? in_jm : (EYv[d] < 0 ? in_jp : true));
      // (depth 0: a neighbour outside the region; the value is not used)
      const int nb = min(max(tid - EXv[d] - EYv[d] * w, 0), NMAX - 1);
      from[q] = in ? plane_of(q) * NMAX + nb : plane_of(q < 9 ? OPP[d] : 9 + OPP[d]) * NMAX + tid;
    }
  }
  auto step = [&](int t, auto B) __attribute__((always_inline)) {
    T* const L = &buf[decltype(B)::value][0][0];
    if (depth >= t) {
      collide<T, POW, LOGDA, SR, true>(src, k, ldk, f, g);
#pragma unroll
      for (int q = 1; q < 9; ++q) L[plane_of(q) * NMAX + tid] = f[q];
#pragma unroll
      for (int q = 1; q < 5; ++q) L[plane_of(9 + q) * NMAX + tid] = g[q];
    }
    __syncthreads();
    if (depth > t) {
#pragma unroll
      for (int q = 1; q < 9; ++q) f[q] = L[from[q]];
#pragma unroll
      for (int q = 1; q < 5; ++q) g[q] = L[from[9 + q]];
      g[1] = hot ? src.hotc - g[1] : g[1];
      g[3] = cold ? src.coldc - g[3] : g[3];
    }
  };
  int t = 0;
  for (; t + 1 < ts; t += 2) {
    step(t, std::integral_constant<int, 0>{});
    step(t + 1, std::integral_constant<int, 1>{});
  }
  if (t < ts) step(t, std::integral_constant<int, 0>{});
  if (depth >= ts) {
    const int64_t o = pop_off(src, i, j);
#pragma unroll
    for (int q = 0; q < 9; ++q) stg<T, true>(dst_f + q * src.qs + o, f[q]);
#pragma unroll
    for (int q = 0; q < 5; ++q) stg<T, true>(dst_g + q * src.qs + o, g[q]);
  }
}

// Regions along an axis of n nodes: w wide, w - 2 ts apart.
int64_t tiles_along(int n, int w, int ts) { return n <= w ? 1 : (n - w + (w - 2 * ts) - 1) / (w - 2 * ts) + 1; }

constexpr int TILE_TOP_F32 = 1024, TILE_TOP_F64 = 768;  // largest regions (registers, LDS)

}  // namespace

// The region and step count with the shortest modelled time per step, for the
// grids on which this kernel is the faster one.  With W waves of 64 threads on
// each SIMD of the fullest CU a launch takes F + b W + ts (c + d W) us; the
// constants are fitted, at n = 0.8, to 48^2 .. 512^2 in FP32 (F 1.8, b 0.55, c 0.55, d
// 0.53; within 10%) and 48^2 .. 256^2 in FP64 (2.0, 0.6, 0.85, 1.4).  n = 1 uses the
// same plan, though its chain c + d W is shorter (FP64 64^2 1.3 us, modelled 2.7):
// nothing is fitted there but the limits below.  A workgroup of
// more than 512 threads (FP64: 256) has a CU to itself, and each further round of
// them starts with its loads exposed.  Near the FP32 limit the plan is compared
// with one step per launch, 2.9 us + 16.2 ps per node.  n = 0.8, us per step, one
// step / this kernel: 460^2 6.7 / 6.1, 500^2 7.0 / 6.7, 510^2 7.0 / 7.2, 520^2
// 7.9 / 7.4, 400 x 650 7.4 / 6.1, 650 x 400 7.5 / 7.5, 130 x 2000 8.1 / 7.4 (without
// the rounds in the model the regions chosen took 6.4, 6.6, 7.6, 8.0, 6.2, 8.7, 9.0).
// In FP64 the viscosity solve leaves room for two waves per SIMD: 280^2 6.6 /
// 5.6, 255 x 333 6.8 / 5.7, 100 x 900 7.0 / 5.7, but with three 300^2 6.8 / 7.7;
// n = 1: 264^2 4.5 / 3.3, 300^2 4.8 / 3.2, 340^2 5.4 / 4.0, 360^2 6.0 / 5.4, 400^2 6.6 / 7.8.
TilePlan tile_plan(int nx, int ny, bool fp64, bool pow, int cus) {
  TilePlan best{0, 0, 0};
  if ((int64_t)nx * ny > (fp64 ? TILE_NODES_F64 : TILE_NODES_F32)) return best;
  const double F = fp64 ? 2.0 : 1.8, b = fp64 ? 0.6 : 0.55, c = fp64 ? 0.85 : 0.55, d = fp64 ? 1.4 : 0.53;
  double best_us = 1e300;
  for (int n : {256, 512, 768, 1024}) {
    if (n > (fp64 ? TILE_TOP_F64 : TILE_TOP_F32)) break;
    for (int w : {16, 24, 32}) {
      const int h = n / w;
      for (int ts = 2; ts <= 8 && 2 * ts < w && 2 * ts < h; ++ts) {
        const int64_t tiles = tiles_along(nx, w, ts) * tiles_along(ny, h, ts);
        const double waves = (double)((tiles + cus - 1) / cus) * (n / 64) / 4.0;
        if (fp64 && pow && waves > 2.0) continue;
        const int fit = fp64 ? (n <= 256 ? 2 : 1) : (n <= 256 ? 5 : n <= 512 ? 3 : 1);  // workgroups on a CU at a time
        const int64_t rounds = (tiles + (int64_t)cus * fit - 1) / ((int64_t)cus * fit);
        const double us = (F + (double)(rounds - 1) * (F + 1.2) + b * waves) / ts + c + d * waves;
        if (us < best_us) {
          best_us = us;
          best = TilePlan{w, h, ts};
        }
      }
    }
  }
  if (!fp64 && best_us > 6.0 && best_us > 1.02 * (2.9 + 16.2e-6 * (double)nx * ny)) return TilePlan{0, 0, 0};
  return best;
}

template <typename T>
hipError_t launch_tile(const KParams<T>& src, const KParams<T>& dst, const TilePlan& plan, int ts, hipStream_t s, bool pow,
                       bool logda) {
  constexpr int TOP = sizeof(T) == 8 ? TILE_TOP_F64 : TILE_TOP_F32;
  const int n = plan.w * plan.h, nt = (n + 63) / 64 * 64;
  if (src.px || src.py || ts < 1 || plan.w <= 2 * ts || plan.h <= 2 * ts || n > TOP) return hipErrorInvalidValue;
  const int64_t tx = tiles_along(src.nx, plan.w, ts), tiles = tx * tiles_along(src.ny, plan.h, ts);
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
#define PM_T(POW, LOG, SR, NMAX)                                                                                      \
  hipLaunchKernelGGL((k_tile<T, POW, LOG, SR, NMAX>), dim3((unsigned)tiles), dim3(nt), 0, s, src, dst.f, dst.g, (int)tx, \
                     plan.w, plan.h, ts)
#define PM_T_N(POW, LOG, SR)                    \
  do {                                          \
    if (nt <= 256) PM_T(POW, LOG, SR, 256);     \
    else if (nt <= 512) PM_T(POW, LOG, SR, 512); \
    else PM_T(POW, LOG, SR, TOP);               \
  } while (0)
#define PM_T_ALL(SR)                                                               \
  if (pow) { if (logda) PM_T_N(true, true, SR); else PM_T_N(true, false, SR); }     \
  else { if (logda) PM_T_N(false, true, SR); else PM_T_N(false, false, SR); }
  bool done = false;
  if constexpr (std::is_same<T, float>::value) {
    if (src.sr) {
      PM_T_ALL(true)
      done = true;
    }
  }
  if (!done) { PM_T_ALL(false) }
#undef PM_T_ALL
#undef PM_T_N
#undef PM_T
  return hipGetLastError();
}

template hipError_t launch_tile<float>(const KParams<float>&, const KParams<float>&, const TilePlan&, int, hipStream_t,
                                       bool, bool);
template hipError_t launch_tile<double>(const KParams<double>&, const KParams<double>&, const TilePlan&, int, hipStream_t,
                                        bool, bool);

}  // namespace pm
