// Device code: many SSP Runge-Kutta steps of a 1D problem in one launch (the
// scalar fluxes and the Euler system, the second-, third- and fourth-order
// methods).
//
// One thread holds one cell in registers from the first step of the launch to
// the last; a stage publishes the cells' states in LDS, passes one barrier
// and evaluates every cell from its registers and its two neighbours' slots
// (two LDS buffers in turn, so one barrier per operator evaluation is
// enough).  A mesh of at most kLineThreads cells is one workgroup, periodic
// wrap and walls included, and its steps run without leaving it.  A larger
// mesh is cut into windows of kLineThreads cells: a window loads `halo` cells
// on each side of the `own` cells it stores, and every operator evaluation
// makes one more cell at each end of it stale, so halo = evaluations per step
// x steps.  Stale cells are computed like the others and never stored.  The
// cell arithmetic and the RK combinations are those of the per-stage kernels
// in the same order: the results are the same bit for bit.
//
// What bounds it: a small mesh is one chain of dependent FP64 operations, LDS
// round trips and barriers per evaluation on a few waves, and a launch per
// step (or per stage) spends more time between the launches than in them; a
// large one is bound by its arithmetic, where the threads of a launch per
// step idle at the tile's ends (five waves for 262 of 320 cells) and the
// per-stage Euler kernel moves the state seven times a step.  Per step, one
// launch per step or stage -> this kernel: 64 cells P2 advection 4.4 -> 1.5
// us, 1024 cells P3 fourth order 17.4 -> 3.5, Sod 128 cells P2 8.0 -> 3.7,
// Sod 2^20 cells P2 121 -> 67.
#pragma once

#include "dg_euler.hpp"

namespace dgk {

constexpr int kLineThreads = 256;
// The Euler system on few windows: kLineSplitCells cells on three times as
// many threads, a cell's work on three of them (line_kernel's SPLIT)
constexpr int kLineSplitCells = 128;
constexpr int kLineSplitThreads = 3 * kLineSplitCells;

// Coefficients of the SSP methods in the form out = a un + b (u + dt' L(u)).
// The five-stage fourth-order method of Spiteri and Ruuth (Shu-Osher form
// U_k = sum_j alpha_kj U_j + beta_kj dt L(U_j)); dt' = dt beta / alpha.
constexpr double kA10 = 1.0, kB10 = 0.391752226571890;
constexpr double kA20 = 0.444370493651235, kA21 = 0.555629506348765, kB21 = 0.368410593050371;
constexpr double kA30 = 0.620101851488403, kA32 = 0.379898148511597, kB32 = 0.251891774271694;
constexpr double kA40 = 0.178079954393132, kA43 = 0.821920045606868, kB43 = 0.544974750228521;
constexpr double kA52 = 0.517231671970585, kA53 = 0.096059710526147, kB53 = 0.063692468666290;
constexpr double kA54 = 0.386708617503269, kB54 = 0.226007483236906;

// operator evaluations of one step of the method of this order (the
// fourth-order method uses L(U3) in two combinations)
__host__ __device__ constexpr int rk_evals(int order) { return order == 4 ? 5 : order; }

struct LineArgs {
  StageArgs s;   // uin, out (the same array only for a mesh of one workgroup), mesh and parameters
  int steps;     // steps of this launch
  int own;       // cells a workgroup stores (the whole mesh: nx)
  int halo;      // cells it loads on each side of them (the whole mesh: 0)
  double dts[6]; // dt' of the combinations, in order (fourth order: U1 U2 U3 U4 W U^{n+1})
};

// Thread t of the workgroup of window `tile`: its cell's mesh index before
// wrapping (gx), whether it holds a cell of the window (else it only joins
// the barriers), and whether it stores it.  own + 2 halo <= the workgroup's
// threads.
__host__ __device__ inline bool line_cell(const LineArgs& B, int tile, int t, int& gx, bool& stores) {
  gx = tile * B.own - B.halo + t;
  stores = t >= B.halo && t < B.halo + B.own && gx < B.s.nx;
  return t < B.own + 2 * B.halo;
}

// Whether this kernel takes a mesh of nx cells: every index a thread forms
// (line_cell) stays below 2^31.  (Meshes beyond run their stages one by one.)
inline bool line_takes(int nx) { return nx <= 2147483647 - 2 * kLineThreads; }

// Launch shape for a mesh of nx cells and a run of nsteps steps (every count of
// the type).
// Up to kLineThreads cells: one workgroup, any number of steps.  Beyond:
// windows of kLineThreads threads, and as many steps per launch as pay.  A
// longer launch hides more of a launch's fixed time (kLineFixed: the gap to
// the next launch, the loads and the stores) and recomputes more halo cells.
// While every window has a compute unit of its own the halo costs nothing, so
// the longest launch wins (halo <= 48 of 256 threads); past that the sum of
// the two costs is minimised, with kLineEval us of a compute unit's time per
// operator evaluation of a window and stored value of a cell.  (Fixed costs of
// 3 to 6 and 0.10 instead of 0.14 stay within 1 % of it in the mean of 432
// runs, advection, Burgers and Sod at 30000 to 2^20 cells, every degree and
// order, and lose up to 50 % in single ones.)
constexpr int kLineMaxHalo = 48;
constexpr int kLineChunk = 128;  // steps per launch of a mesh of one workgroup
constexpr double kLineFixed = 4.0, kLineEval = 0.14;
//   The Euler system takes split windows while each has a compute unit of its
// own (128 cells, halo <= 24).  Sod P2, per step, whole cells -> split: 128
// cells 4.39 -> 3.75 us, 256 cells (one workgroup -> windows relaunched every
// eight steps) 4.61 -> 4.16, 1000 cells 4.87 -> 4.21, 15000 cells 4.91 -> 4.25
// (P1 3.42 -> 2.90 at 128, P4 6.51 -> 5.91); past that, windows share compute
// units and whole cells are cheaper.  Over 64 to 19000 cells, every degree,
// order and mode, the split takes .84 to 1.02 of the whole cells' time (up to
// 1.05 between 129 and 256 cells, where windows stand against one workgroup), but
// 1.02 to 1.11 with the fourth order at P4 without a sensor, where it spills:
// that one takes whole cells.
constexpr int kLineSplitMaxHalo = 24;
struct LinePlan {
  int threads, own, halo, steps;
  bool split;
};
inline LinePlan line_plan(int nx, int nv, int order, int cus, int nsteps, bool euler, bool sensor) {
  const int ev = rk_evals(order);
  const int steps = nsteps / 2 + nsteps % 2;  // windows alternate between two arrays: two launches at least
  if (euler && (sensor || nv < 15 || order < 4)) {
    if (nx <= kLineSplitCells) return {kLineSplitThreads, nx, 0, kLineChunk, true};
    const int s = steps < kLineSplitMaxHalo / ev ? steps : kLineSplitMaxHalo / ev;
    const int own = kLineSplitCells - 2 * ev * s;
    if ((nx + own - 1) / own <= cus) return {kLineSplitThreads, own, ev * s, s, true};
  }
  if (nx <= kLineThreads) return {(nx + 63) / 64 * 64, nx, 0, kLineChunk, false};
  LinePlan best{};
  double cost = 0.0;
  for (int s = 1; s <= kLineMaxHalo / ev && s <= steps; ++s) {
    const int own = kLineThreads - 2 * ev * s;
    const double load = (double)((nx + own - 1) / own) / cus;
    const double c = ev * kLineEval * nv * (load > 1.0 ? load : 1.0) + kLineFixed / s;
    if (s == 1 || c < cost) {
      cost = c;
      best = {kLineThreads, own, ev * s, s, false};
    }
  }
  return best;
}

// Launches of a run of nsteps steps and the steps of launch k: spread evenly,
// one at least.  Where they alternate between two arrays their number is even,
// so that the last one writes the caller's, unless there is no step left for
// another launch (one step each, an odd count: a copy follows the last).
inline long long line_launches(const LinePlan& p, int nsteps) {
  long long n = nsteps / p.steps + (nsteps % p.steps != 0);
  if (p.halo > 0 && n % 2 == 1 && n < nsteps) ++n;
  return n;
}
inline int line_launch_steps(int nsteps, long long launches, long long k) {
  return (int)(nsteps * (k + 1) / launches - nsteps * k / launches);
}

// dU/dt of one cell of a scalar flux, from its coefficients and the slots of
// its neighbours
template <int P, int FLUX, int MODE, int CELLS = kLineThreads>
struct LineCell {
  using G = TileGeom<1, CELLS, 1>;
  using C = Cell<1, P, FLUX, MODE, G::S, G::W>;
  static constexpr int NV = P + 1, S = G::S;
  __device__ static inline void rhs(const StageArgs& A, const double* b, const double (&c)[NV], int ix,
                                    double (&L)[NV]) {
    C::template rhs<true>(A, b, c, ix, 0, L);
  }
};

template <int P, int MODE, int CELLS>
struct LineCell<P, FLUX_EULER, MODE, CELLS> {
  using E = EulerCell<P, MODE, CELLS>;
  using C = typename E::C;
  static constexpr int N = P + 1, NV = 3 * N, S = E::S;
  __device__ static inline void rhs(const StageArgs& A, const double* b, const double (&c)[NV], int ix,
                                    double (&L)[NV]) {
    double u[3][N], R[3][N], lam;
#pragma unroll
    for (int j = 0; j < NV; ++j) u[j / N][j % N] = c[j];
    const double gam = C::template gamma_of<true>(A, b, u[0], ix, 0);
    E::residual(A, b, u, ix, R, lam);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double Lk[N];
      C::finish(A, u[k], gam, lam, R[k], Lk);
#pragma unroll
      for (int a = 0; a < N; ++a) L[k * N + a] = Lk[a];
    }
  }
};

// (two state buffers; split: and the exchange of nv + 2 planes)
__host__ __device__ constexpr int line_lds_doubles(int nv, bool split) {
  return split ? (2 * nv + nv + 2) * TileGeom<1, kLineSplitCells, 1>::S : 2 * nv * TileGeom<1, kLineThreads, 1>::S;
}

// Grid: ceil(nx / own) workgroups of at most kLineThreads threads (a multiple
// of 64), LDS line_lds_doubles.
// SPLIT (the Euler system): workgroups of kLineSplitThreads, three threads per
// cell on different waves.  One holds the cell (its state, the faces, the
// combination), one evaluates the volume terms and lambda_e, one gamma_e; the
// last two read the cell from LDS and hand their results over in LDS, behind a
// second barrier.  On a wave alone on its SIMD an FP64 instruction takes about
// 2.5 ns however independent it is of its neighbours, so an evaluation takes
// what its longest wave has, instead of what a cell has (641 instructions at
// P2), and one more barrier.
// The Euler system's whole cells at P4 are held to two waves per SIMD: left to
// itself the compiler takes 1 to 8 registers more than that with the sensor of
// the paper's exponents, and a compute unit then holds one workgroup (Sod P4
// per step, one -> two: 65536 cells 17.3 -> 14.6 us, 2^20 cells 192 -> 125).
template <int P, int FLUX, int MODE, int RK, bool SPLIT = false>
__global__ void __launch_bounds__(SPLIT ? kLineSplitThreads : kLineThreads,
                                  FLUX == FLUX_EULER && P == 4 && !SPLIT ? 2 : 1) line_kernel(const LineArgs B) {
  static_assert(!SPLIT || FLUX == FLUX_EULER, "the scalar fluxes' cells are too short to split");
  using LC = LineCell<P, FLUX, MODE, SPLIT ? kLineSplitCells : kLineThreads>;
  constexpr int NV = LC::NV, S = LC::S;
  extern __shared__ double lds[];
  const StageArgs& A = B.s;
  const int t = SPLIT ? threadIdx.x % kLineSplitCells : threadIdx.x;
  // 0: volume, 1: the cell's owner, 2: sensor (waves go to SIMDs in turn: the
  // sensor's two share one with the volume's)
  const int role = SPLIT ? threadIdx.x / kLineSplitCells : 1;
  const bool owner = role == 1;
  int gx, wx = 0, wy;
  bool stores;
  const bool held = line_cell(B, xcd_tile(blockIdx.x, gridDim.x), t, gx, stores);
  // cells beyond a non-periodic end hold the exterior state in every stage
  const bool active = held && step_cell<1>(A, gx, 0, wx, wy);
  double c[NV], u0[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) c[j] = active ? A.uin[(size_t)wx * NV + j] : (j == 0 ? A.bc : 0.0);
  // cell t at slot t + 1; on a periodic mesh of one workgroup each end cell
  // also fills the slot beyond the other end
  const bool ring = B.halo == 0 && A.per_x;
  // otherwise the slots beyond the workgroup's cells, which only stale cells
  // and the ends of a non-periodic mesh read, hold the exterior state; in the
  // windows of an Euler mesh the end cells' first, so that stale cells are
  // states of a gas (off the middle range their evaluations would be repeated,
  // euler_flux)
  const int last = B.own + 2 * B.halo - 1;
  const bool echo = FLUX == FLUX_EULER && B.halo > 0;
#pragma unroll
  for (int e = 0; e < 2; ++e)
    if (owner && !ring && t == (e ? last : 0)) {
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const double v = echo ? c[j] : (j == 0 ? A.bc : 0.0);
        lds[j * S + (e ? last + 2 : 0)] = v;
        lds[(NV + j) * S + (e ? last + 2 : 0)] = v;
      }
    }
  int par = 0;
  // L := L(c); the state is published in this evaluation's buffer first
  auto eval = [&](double (&L)[NV]) {
    double* const buf = lds + par * (NV * S);
    par ^= 1;
    if (held && owner) {
#pragma unroll
      for (int j = 0; j < NV; ++j) buf[j * S + t + 1] = c[j];
      if (ring && t == 0) {
#pragma unroll
        for (int j = 0; j < NV; ++j) buf[j * S + last + 2] = c[j];
      }
      if (ring && t == last) {
#pragma unroll
        for (int j = 0; j < NV; ++j) buf[j * S] = c[j];
      }
    }
    tile_barrier();
    if constexpr (SPLIT) {
      using E = typename LC::E;
      constexpr int N = P + 1;
      double* const ex = lds + 2 * NV * S + t;  // volume terms (planes 0 .. NV-1), lambda_e, gamma_e
      double u[3][N], H[2][3];
      if (active) {
#pragma unroll
        for (int j = 0; j < NV; ++j) u[j / N][j % N] = owner ? c[j] : buf[j * S + t + 1];
        if (role == 0) {
          double R[3][N], lam;
          uint32_t off = 0;
          E::template volume<false>(u, R, lam, off);
          if (__builtin_expect(off >= kRangeWidth, 0)) {
            E::again(buf, u);
            E::template volume<true>(u, R, lam, off);
          }
#pragma unroll
          for (int j = 0; j < NV; ++j)
            if (j % N) ex[j * S] = R[j / N][j % N];
          ex[NV * S] = lam;
        } else if (role == 2) {
          ex[(NV + 1) * S] = LC::C::template gamma_of<true>(A, buf + t + 1, u[0], wx, 0);
        } else {
          uint32_t off = 0;
#pragma unroll
          for (int f = 0; f < 2; ++f) E::template face_flux<false>(A, buf + t + 1, u, wx, f, H[f], off);
          if (__builtin_expect(off >= kRangeWidth, 0)) {
            const double* const bx = E::again(buf + t + 1, u);
#pragma unroll
            for (int f = 0; f < 2; ++f) E::template face_flux<true>(A, bx, u, wx, f, H[f], off);
          }
        }
      }
      tile_barrier();
      if (active && owner) {
        double R[3][N];
#pragma unroll
        for (int j = 0; j < NV; ++j) R[j / N][j % N] = j % N ? ex[j * S] : 0.0;
        const double lam = ex[NV * S], gam = ex[(NV + 1) * S];
#pragma unroll
        for (int f = 0; f < 2; ++f) E::add_face(f, H[f], R);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          double Lk[N];
          LC::C::finish(A, u[k], gam, lam, R[k], Lk);
#pragma unroll
          for (int a = 0; a < N; ++a) L[k * N + a] = Lk[a];
        }
      }
    } else {
      if (active) LC::rhs(A, buf + t + 1, c, wx, L);
    }
  };
  // v = a un + b (c + dt L), rounded as in the per-stage kernels (contraction
  // off: with a = 1 the compiler would fuse b (..) + un, which they do not)
  auto comb = [&](double a, double b, double dt, const double (&L)[NV], const double (&un)[NV], double (&v)[NV]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const double w = b * fma(dt, L[j], c[j]);
      v[j] = a != 0.0 ? fma(a, un[j], w) : w;
    }
  };
  const bool mine = active && owner;
#pragma unroll 1
  for (int s = 0; s < B.steps; ++s) {
    double L[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) u0[j] = c[j];
    eval(L);
    if (mine) comb(0.0, 1.0, B.dts[0], L, u0, c);
    if constexpr (RK == 2) {
      eval(L);
      if (mine) comb(0.5, 0.5, B.dts[1], L, u0, c);
    } else if constexpr (RK == 3) {
      eval(L);
      if (mine) comb(0.75, 0.25, B.dts[1], L, u0, c);
      eval(L);
      if (mine) comb(1.0 / 3.0, 2.0 / 3.0, B.dts[2], L, u0, c);
    } else {
      double u2[NV], w[NV];
      eval(L);
      if (mine) comb(kA20, kA21, B.dts[1], L, u0, c);
#pragma unroll
      for (int j = 0; j < NV; ++j) u2[j] = c[j];
      eval(L);
      if (mine) comb(kA30, kA32, B.dts[2], L, u0, c);
      eval(L);
      if (mine) {
        comb(kA52, kA53, B.dts[4], L, u2, w);  // W = a52 U2 + a53 U3 + b53 dt L(U3)
        comb(kA40, kA43, B.dts[3], L, u0, c);
      }
      eval(L);
      if (mine) comb(1.0, kA54, B.dts[5], L, w, c);
    }
  }
  if (mine && stores) {
    double* const dst = A.out + (size_t)gx * NV;
#pragma unroll
    for (int j = 0; j < NV; ++j) dst[j] = c[j];
  }
}

}  // namespace dgk
