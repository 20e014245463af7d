// pm_march.hip -- large cavities: several time steps in one pass (gfx950).
//
// A one-step pass reads and writes every population once, 112 B per node
// update in FP32, and at the copy rate of 6.5 TB/s that alone takes 290 us at
// 4096^2.  This kernel takes TS steps per pass.  A wave owns a strip of 64
// columns, one per lane, and marches up its rows: row a of the state is
// collided (step k), row a - 1 takes step k + 1 from the post-collision rows
// a - 2 .. a, and so on; row a - TS of step k + TS is stored.  What a stage
// needs of the two rows below it stays in the lane's registers (16 values), the
// populations that move along x come from the neighbouring lane by a whole-wave
// DPP shift, so there is no LDS and no dependence between waves; the strips
// overlap by 2 TS columns and the row groups by 2 TS rows instead.  The
// per-node arithmetic is the single-step kernel's (collide): the populations
// are the same bit for bit.
//
// Measured (n = 0.8, stochastic rounding, us per step; one step per pass / an
// earlier two-step kernel with LDS row rings / this one with TS = 3):
// 2048^2 66 / 73 / 58, 3000^2 166 / 167 / 110, 4096^2 299 / 230 / 183 .. 199,
// 8192^2 1243 / 855 / 628.  FP64 with TS = 2: 3000^2 345 / - / 321, 4096^2 608 /
// - / 551.  At TS = 3 FP32 the VALU issues all the time (SQ_INSTS_VALU, 410
// instructions per node update with the overlaps, of which 350 per row and
// stage; 333 and 285 with round-to-nearest), at TS = 2 the pass moves 2.3 GB at
// 4 TB/s (4096^2 221 us), at TS = 4 the registers no longer hold (240).
//
// What the details are worth at 4096^2:
//   * the four waves of a workgroup hold adjacent strips and meet at a barrier
//     every row, so that they read and write 1 KB pieces together: 193 us, 204
//     without it (TS = 2: 221 and 283);
//   * cached loads and stores: lines are shared with the neighbouring strip;
//     streaming loads 218, streaming stores 235;
//   * row r + 1 is loaded once row r has been collided, all of it: otherwise the
//     two rows' registers overlap and each value is copied (pin);
//   * two columns per lane (fewer overlaps, half the shifts) need 230 registers:
//     with two waves per SIMD 243 us at best.
#include "pm_device.h"

#include <algorithm>
#include <type_traits>

namespace pm {
namespace {

using namespace pm::dev;

// Whole-wave lane shifts (DPP): the value of lane l - 1 (from_left) or l + 1
// (from_right); the lane without a neighbour (0 or 63) gets `old`.  All 64
// lanes must be active.
template <int CTRL>
__device__ __forceinline__ float lane_shift(float old, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v),
                                                               CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double old, double v) {
  const uint64_t o = __builtin_bit_cast(uint64_t, old), w = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)o, (int)(unsigned)w, CTRL, 0xf, 0xf, false);
  const unsigned hi =
      (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(o >> 32), (int)(unsigned)(w >> 32), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
constexpr int DPP_WAVE_SHL1 = 0x130, DPP_WAVE_SHR1 = 0x138;
template <typename T>
__device__ __forceinline__ T from_left(T old, T v) { return lane_shift<DPP_WAVE_SHR1>(old, v); }
template <typename T>
__device__ __forceinline__ T from_right(T old, T v) { return lane_shift<DPP_WAVE_SHL1>(old, v); }

// f(0), f(1), .. f(N - 1) with compile-time arguments: what they index is then
// in registers from the start, whatever the unroller decides.
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (N > 0) {
    unrolled<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// a or b by value (a conditional expression on two array elements would select
// between their addresses and keep the arrays out of registers).
template <typename T>
__device__ __forceinline__ T sel(bool c, T a, T b) { return c ? a : b; }

template <typename T>
struct Node {
  T f[9], g[5];
};

// Every value of a is computed here and no later (no instruction).
template <typename T>
__device__ __forceinline__ void pin(Node<T>& a) {
  unrolled<14>([&](auto Q) {
    constexpr int q = decltype(Q)::value;
    T t;
    if constexpr (q < 9) t = a.f[q];
    else t = a.g[q - 9];
    asm volatile("" : "+v"(t));
    if constexpr (q < 9) a.f[q] = t;
    else a.g[q - 9] = t;
  });
}

// What a stage keeps of the post-collision rows b and b - 1 of the step
// before it, for this lane's column.
template <typename T>
struct Rows {
  T h0, h1, h3, k0, k1, k3;  // row b: f0 f1 f3 g0 g1 g3
  T u2, u5, u6, v2;          // row b: f2 f5 f6 g2 (moving up)
  T d7, d8;                  // row b: f7 f8 (needed at walls only)
  T w2, w5, w6, x2;          // row b - 1: f2 f5 f6 g2; on the bottom row f4 and g4 of the row itself in w2, x2
};

// The next post-collision row (`row`) enters; INNER: it is not the bottom row.
template <bool INNER, typename T>
__device__ __forceinline__ void push(Rows<T>& c, int row, const Node<T>& a) {
  c.w2 = sel(!INNER && row == 0, a.f[4], c.u2);
  c.x2 = sel(!INNER && row == 0, a.g[4], c.v2);
  c.w5 = c.u5;
  c.w6 = c.u6;
  c.h0 = a.f[0]; c.h1 = a.f[1]; c.h3 = a.f[3];
  c.k0 = a.g[0]; c.k1 = a.g[1]; c.k3 = a.g[3];
  c.u2 = a.f[2]; c.u5 = a.f[5]; c.u6 = a.f[6]; c.v2 = a.g[2];
  c.d7 = a.f[7]; c.d8 = a.f[8];
}

// Pre-collision populations at row b from rows b and b - 1 (cp) and b + 1 (ap):
// direction q from the node at -e_q, or the own population in the opposite
// direction where that crosses a wall (bounce-back; thermal anti-bounce-back at
// the hot and cold walls).  INNER: b is not the bottom or top row.  Lane 0 of
// the leftmost strip is the hot wall's column: its values from the left are the
// shifts' `old`.  right: the strip holds the cold wall's column, the lanes
// `wall`.
template <bool INNER, typename T>
__device__ __forceinline__ void pull(const KParams<T>& p, const Rows<T>& cp, int b, bool right, bool wall,
                                     const Node<T>& ap, Node<T>& d) {
  // by value first: loads sunk into the branches below would keep them in memory
  const Rows<T> c = cp;
  const Node<T> a = ap;
  T* f = d.f;
  T* g = d.g;
  f[0] = c.h0;
  f[1] = from_left(c.h3, c.h1);
  f[3] = from_right(c.h1, c.h3);
  g[0] = c.k0;
  g[1] = from_left(p.hotc - c.k3, c.k1);
  g[3] = from_right(p.coldc - c.k1, c.k3);
  f[2] = c.w2;
  g[2] = c.x2;
  if (!INNER && b == 0) {
    f[5] = c.d7;
    f[6] = c.d8;
  } else {
    f[5] = from_left(c.d7, c.w5);
    f[6] = from_right(c.d8, c.w6);
  }
  if (!INNER && b == p.ny - 1) {
    f[4] = c.u2;
    f[7] = c.u5;
    f[8] = c.u6;
    g[4] = c.v2;
  } else {
    f[4] = a.f[4];
    f[7] = from_right(c.u5, a.f[7]);
    f[8] = from_left(c.u6, a.f[8]);
    g[4] = a.g[4];
  }
  if (right) {
    f[3] = sel(wall, c.h1, f[3]);
    f[6] = sel(wall, c.d8, f[6]);
    f[7] = sel(wall, c.u5, f[7]);
    g[3] = sel(wall, p.coldc - c.k1, g[3]);
  }
}

// One workgroup: a wave for each of up to MARCH_WAVES adjacent strips, by `rows`
// output rows.
template <typename T, bool POW, bool LOGDA, bool SR, int TS>
__global__ __launch_bounds__(64 * MARCH_WAVES, sizeof(T) == 8 ? 2 : (TS == 2 ? 4 : 3)) void k_march(
    KParams<T> src, T* __restrict__ dst_f, T* __restrict__ dst_g, int strips, int waves, int rows) {
  // Workgroups (row group major, strips minor) are dealt to the 8 XCDs in blocks
  // of 8 adjacent ones, so that the columns two of them share are mostly fetched
  // into one L2, while all XCDs advance through the same rows.  The last
  // gridDim mod 64 keep their own place (a bijection).
  constexpr int XCD_BLOCK = 8;
  int blk = blockIdx.x;
  if (blk < (int)gridDim.x / (8 * XCD_BLOCK) * (8 * XCD_BLOCK)) {
    const int xcd = blk & 7, q = blk >> 3;
    blk = ((q / XCD_BLOCK) * 8 + xcd) * XCD_BLOCK + q % XCD_BLOCK;
  }
  const int across = (strips + waves - 1) / waves;
  const int sy = blk / across;
  // a wave past the last strip repeats it and stores nothing: all waves of the
  // workgroup run the same rows and reach every barrier
  const int s0 = __builtin_amdgcn_readfirstlane((blk - sy * across) * waves + ((int)threadIdx.x >> 6));
  const int sx = min(s0, strips - 1);
  const int lane = threadIdx.x & 63;
  const int nx = src.nx, ny = src.ny;
  const int c0 = sx * (64 - 2 * TS), cl = c0 + lane;
  const bool right = c0 + 64 >= nx;   // the strip holds the last column
  const int c = min(cl, nx - 1);      // lanes past it repeat it
  const bool wall = cl >= nx - 1;
  const bool out = s0 < strips && cl >= (sx == 0 ? 0 : c0 + TS) && cl < (right ? nx : c0 + 64 - TS);
  const int y0 = sy * rows, y1 = min(y0 + rows, ny) - 1;  // output rows [y0, y1]
  const int last = min(y1 + TS, ny - 1);                  // last row read
  // This lane's element of a row given by a wave-uniform pointer, o the column's
  // byte offset.  The empty asm statements keep the pointer in scalar registers
  // and the offset a 32-bit one (otherwise the compiler forms each address with
  // a 64-bit vector add).
  auto at = [](const T* base, unsigned o) {
    auto g = (__attribute__((address_space(1))) char*)base;
    asm("" : "+s"(g));
    return (__attribute__((address_space(1))) T*)(g + o);
  };
  auto offset = [&] {
    unsigned o = (unsigned)c * (unsigned)sizeof(T);
    asm volatile("" : "+v"(o));
    return o;
  };
  Node<T> n;  // the row that enters next
  T ldn = T(0), ld[TS] = {};
  auto load_row = [&](int a) {
    const unsigned o = offset();
    unrolled<14>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      if constexpr (q < 9) n.f[q] = *at(src.f + (int64_t)a * src.rs + q * src.qs, o);
      else n.g[q - 9] = *at(src.g + (int64_t)a * src.rs + (q - 9) * src.qs, o);
    });
    if (LOGDA) ldn = *at(src.logda + (int64_t)a * nx, o);
  };
  Rows<T> C[TS] = {};
  // Row a enters: step k there, then step k + t at row a - t, and the output.
  // INNER: every stage has a row, and none at the bottom or top wall.
  auto row = [&](int a, auto inner) __attribute__((always_inline)) {
    constexpr bool INNER = decltype(inner)::value;
    Node<T> v = n;
    if (LOGDA) {
      unrolled<TS - 1>([&](auto I) {
        constexpr int t = TS - 1 - decltype(I)::value;
        ld[t] = ld[t - 1];
      });
      ld[0] = ldn;
    }
    if (INNER || a <= last) collide<T, POW, LOGDA, SR>(src, a * nx + c, ld[0], v.f, v.g);
    pin(v);
    if (INNER || a + 1 <= last) load_row(a + 1);
    bool live = true;
    unrolled<TS>([&](auto I) {
      constexpr int t = decltype(I)::value + 1;
      const int b = a - t;
      if (!live) return;
      if (!INNER && b < max(0, y0 - TS + t)) {  // this stage has not begun, nor have the later ones
        push<INNER>(C[t - 1], b + 1, v);
        live = false;
      } else if (INNER || b <= min(ny - 1, y1 + TS - t)) {
        Node<T> d;
        pull<INNER>(src, C[t - 1], b, right, wall, v, d);
        push<INNER>(C[t - 1], b + 1, v);
        v = d;
        if constexpr (t < TS) {
          collide<T, POW, LOGDA, SR>(src, b * nx + c, ld[t], v.f, v.g);
        } else if (out) {
          const unsigned o = offset();
          unrolled<14>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            if constexpr (q < 9) *at(dst_f + (int64_t)b * src.rs + q * src.qs, o) = v.f[q];
            else *at(dst_g + (int64_t)b * src.rs + (q - 9) * src.qs, o) = v.g[q - 9];
          });
        }
      }
    });
  };
  int a = max(0, y0 - TS);
  load_row(a);
  const int inner0 = max(y0, 1) + TS, inner1 = last - 1;
  for (; a < inner0 && a <= y1 + TS; ++a) row(a, std::false_type{});
  for (; a <= inner1; ++a) {
    __builtin_amdgcn_s_barrier();  // orders no data: keeps the strips on the same rows
    row(a, std::true_type{});
  }
  for (; a <= y1 + TS; ++a) row(a, std::false_type{});
}

// Strips across nx columns: 64 wide, 64 - 2 ts apart.
int march_strips(int nx, int ts) { return nx <= 64 ? 1 : (nx - 64 + (64 - 2 * ts) - 1) / (64 - 2 * ts) + 1; }

}  // namespace

// Steps per pass and output rows per workgroup (ts = 0: take one step per pass).
// The pass pays off where the grid gives the waves enough rows, and it is bound
// by vector issue where one step per pass is bound by memory: so it depends on
// the viscosity.  us per step, one step per pass / this pass (FP32
// stochastically rounded; a range where the state of the flow decides how long
// the Newton iterations are):
//   n = 1:   FP32 900^2 15.8 / 14.2, 1100^2 20.4 / 19.8, 2048^2 65 / 38,
//            4000 x 250 17.4 / 19.1, 700 x 8000 97 / 54;
//            FP64 1100^2 36.7 .. 40 / 38.3, 1300^2 50 .. 55 / 46.6, 2400^2 215 / 135
//   n = 0.8: FP32 1760^2 45 .. 50 / 47 .. 55, 2200^2 79 .. 84 / 67 .. 88,
//            2400^2 100 / 79 .. 102, 2600^2 112 .. 118 / 92 .. 119, 4096^2 293 / 195 .. 205;
//            FP64 2600^2 246 .. 260 / 209 .. 249, 3000^2 342 .. 357 / 291 .. 350,
//            4096^2 607 .. 623 / 551 .. 578, 6000^2 1440 .. 1462 / 915 .. 1324
// A flow that sets in from rest is no exception (FP64 4096^2 n = 0.6, 4800 steps 619 /
// 562, no window of 240 steps slower; 2900^2 315 / 296).
// FP64 takes it from 12 strips (128 x 64062, n = 0.8: 326 / 363; 250 x 32800 330 / 329).
//
// Waves: four adjacent strips to a workgroup, unless more than an eighth of the
// waves had none then; apart from each other they take longer by `apart`.  FP32
// 250 x 58000, 5 strips, us per step with 1 / 2 / 3 / 4 waves: n = 0.8 204 / 250 / 269
// / 308, n = 1 177 / 182 / 193 / 215, one step per pass 304 and 310, the earlier
// two-step kernel 220 and 211; 420 x 34523, 8 strips: 196 / 204 / 234 / 192 and 193 /
// 175 / 172 / 148; FP64 1000 x 8200, 17 strips, n = 0.8: 293 / 334 / 379 / 339, one
// step per pass 320.  (Wide grids: FP32 2700^2 n = 0.8 with 1 / 4 waves 103 / 90, FP64
// 4096^2 n = 0.6 from rest 530 / 484.)
//
// Rows: a workgroup of R output rows collides ts R + ts (ts + 1) rows, and 12
// waves (141 registers; FP64 8 of 250) fit a CU.  With r rounds of workgroups the
// time goes as the rows times f(r), measured at 4096^2, 3000^2 and 2048^2: one or
// two rounds end as whole ones, later ones overlap.  (4096^2, R = 24 / 36 / 44 / 48
// / 56 / 72: 202 / 200 / 204 / 193 / 219 / 221 us.)
MarchPlan march_plan(int nx, int ny, bool fp64, bool pow, int cus, bool force) {
  MarchPlan best{0, 0, 0};
  const int ts = fp64 ? 2 : 3;
  const int64_t strips = march_strips(nx, ts);
  const int64_t least = pow ? (fp64 ? 8000000 : 5500000) : (fp64 ? 1600000 : 1200000);
  if (!force && ((int64_t)nx * ny < least || (fp64 && strips < 12))) return best;
  int waves = MARCH_WAVES;
  const int64_t dealt = (strips + 3) / 4 * 4;
  double least_cost = (double)dealt;
  for (int w : {2, 3, 1}) {
    const double apart = w == 3 ? (pow ? 1.08 : 1.3) : w == 2 ? (pow ? 1.06 : 1.15) : (pow ? 1.02 : 1.28);
    const double cost = (double)((strips + w - 1) / w * w) * apart;
    if ((dealt - strips) * 8 > dealt && cost < least_cost) {
      least_cost = cost;
      waves = w;
    }
  }
  const int64_t across = (strips + waves - 1) / waves;
  const double slots = (double)((fp64 ? 8 : 12) / waves) * cus;
  double best_cost = 1e300;
  for (int R = 16; R <= 56; ++R) {
    const double r = (double)(across * std::max(1, ny / R)) / slots;
    const double f = r <= 2 ? std::ceil(r) + 0.05 : std::max(r + 0.1, std::floor(r) + 0.35);
    const double cost = (double)(ts * R + ts * (ts + 1)) * f;
    if (cost < best_cost) {
      best_cost = cost;
      best = MarchPlan{ts, R, waves};
    }
  }
  return best;
}

template <typename T>
hipError_t launch_march(const KParams<T>& src, const KParams<T>& dst, const MarchPlan& plan, int ts, hipStream_t s,
                        bool pow, bool logda) {
  if (src.px || src.py || plan.rows < 1 || plan.waves < 1 || plan.waves > MARCH_WAVES) return hipErrorInvalidValue;
  const int strips = march_strips(src.nx, ts);
  const int64_t groups = (int64_t)((strips + plan.waves - 1) / plan.waves) * ((src.ny + plan.rows - 1) / plan.rows);
  if (groups > 0x7fffffff) return hipErrorInvalidValue;
#define PM_M(POW, LOG, SR, TS)                                                                                     \
  hipLaunchKernelGGL((k_march<T, POW, LOG, SR, TS>), dim3((unsigned)groups), dim3(64 * plan.waves), 0, s, src, dst.f,  \
                     dst.g, strips, plan.waves, plan.rows)
#define PM_M_TS(POW, LOG, SR)                                   \
  do {                                                          \
    if (ts == 2) PM_M(POW, LOG, SR, 2);                         \
    else if (ts == 3 && sizeof(T) == 4) PM_M(POW, LOG, SR, (sizeof(T) == 4 ? 3 : 2)); \
    else return hipErrorInvalidValue;                           \
  } while (0)
#define PM_M_ALL(SR)                                                                 \
  if (pow) { if (logda) PM_M_TS(true, true, SR); else PM_M_TS(true, false, SR); }     \
  else { if (logda) PM_M_TS(false, true, SR); else PM_M_TS(false, false, SR); }
  bool done = false;
  if constexpr (std::is_same<T, float>::value) {
    if (src.sr) {
      PM_M_ALL(true)
      done = true;
    }
  }
  if (!done) { PM_M_ALL(false) }
#undef PM_M_ALL
#undef PM_M_TS
#undef PM_M
  return hipGetLastError();
}

template hipError_t launch_march<float>(const KParams<float>&, const KParams<float>&, const MarchPlan&, int, hipStream_t,
                                        bool, bool);
template hipError_t launch_march<double>(const KParams<double>&, const KParams<double>&, const MarchPlan&, int,
                                         hipStream_t, bool, bool);

}  // namespace pm
