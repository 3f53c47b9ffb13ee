// Host-only check of line_kernel's windows: every mesh cell is stored by
// exactly one thread, the loads and LDS slots stay inside their buffers, and
// a stored cell is further from the window's ends than the launch has
// operator evaluations; and the steps of a run's launches add up to the run,
// for step counts up to the type's largest.
#include <cstdio>
#include <vector>

#include "../../paper_2309_12019_amd/csrc/dg_line.hpp"

using namespace dgk;

int main() {
  int bad = 0, launches = 0;
  for (int nx : {1, 2, 63, 64, 65, 128, 255, 256, 257, 300, 511, 512, 1000, 4099, 65536, 70001, 1 << 20})
    for (int order : {2, 3, 4})
      for (int nv : {2, 5, 6, 15})
        for (int nsteps : {2, 3, 4, 9, 10, 128})
          for (int pers : {0, 1, 2, 3}) {
            const int per = pers & 1;
            const bool euler = nv > 5, sensor = pers < 2;
            const LinePlan p = line_plan(nx, nv, order, 256, nsteps, euler, sensor);
            // cells a workgroup holds, its threads, its LDS slots
            const int cells = p.split ? kLineSplitCells : kLineThreads;
            const int slots = p.split ? TileGeom<1, kLineSplitCells, 1>::S : TileGeom<1, kLineThreads, 1>::S;
            LineArgs B{};
            B.s.nx = nx;
            B.s.ny = 1;
            B.s.per_x = per;
            B.own = p.own;
            B.halo = p.halo;
            const bool one = p.halo == 0;
            const int ev = rk_evals(order);
            bad += p.threads % 64 != 0 || p.threads != (p.split ? kLineSplitThreads : (one ? (nx + 63) / 64 * 64 : kLineThreads)) || (p.split && !euler) || p.own < 1 || p.steps < 1 || (p.halo > 0 && p.steps > (nsteps + 1) / 2);
            bad += p.own + 2 * p.halo > cells || (one ? p.halo != 0 || p.own != nx : p.halo != ev * p.steps);
            std::vector<int> written(nx, 0);
            const int grid = (nx + p.own - 1) / p.own;
            for (int tile = 0; tile < grid; ++tile)
              for (int t = 0; t < (p.split ? cells : p.threads); ++t) {
                int gx, wx, wy;
                bool stores;
                const bool held = line_cell(B, tile, t, gx, stores);
                if (!held) {
                  bad += stores;
                  continue;
                }
                bad += t + 1 >= slots - 1 || p.own + 2 * p.halo + 1 >= slots;
                if (step_cell<1>(B.s, gx, 0, wx, wy)) {
                  bad += wx < 0 || wx >= nx;
                  if (stores) {
                    bad += wx != gx;
                    if (wx == gx) ++written[gx];
                    // beyond the window's ends lies another window's cell, or the mesh's end
                    if (!one) bad += t < ev * p.steps || p.own + 2 * p.halo - 1 - t < ev * p.steps;
                  }
                }
              }
            for (int e = 0; e < nx; ++e) bad += written[e] != 1;
            ++launches;
          }
  // launches of a run: one step at least and the plan's steps at most in each
  // (so that halo == 0 means the whole mesh and no cell that a window stores
  // goes stale), all the steps in total, an even number where they alternate
  // between two arrays, unless each has a single step
  for (int nx : {1, 64, 256, 1000, 70001, 1 << 20, 1 << 22})
    for (int order : {2, 3, 4})
      for (int nv : {2, 5, 6, 15})
        for (int nsteps : {2, 3, 5, 15, 16, 17, 127, 128, 129, 1000, 65537, 1 << 30, 2147483519, 2147483520, 2147483600,
                           2147483646, 2147483647}) {
          const LinePlan p = line_plan(nx, nv, order, 256, nsteps, nv > 5, nsteps % 2);
          const long long n = line_launches(p, nsteps);
          const bool bounds = p.own >= 1 && p.steps >= 1 && n >= 1 && (p.halo == 0 || n % 2 == 0 || n == nsteps) &&
                              (p.halo == 0 || p.halo == rk_evals(order) * p.steps);
          bad += !bounds;
          if (!bounds) {
            std::printf("nx %d order %d nv %d: %d steps in %lld launches of %d (own %d)\n", nx, order, nv, nsteps, n,
                        p.steps, p.own);
            continue;
          }
          long long sum = 0;
          const long long stride = n < 100000 ? 1 : n / 50000;  // (of very many launches, groups spread over the run)
          for (long long k = 0; k < n; k += stride) {
            const int s = line_launch_steps(nsteps, n, k);
            bad += s < 1 || s > p.steps;
            if (stride == 1) sum += s;
          }
          if (stride == 1) bad += sum != nsteps;
          bad += line_launch_steps(nsteps, n, n - 1) > p.steps || line_launch_steps(nsteps, n, 0) > p.steps;
          ++launches;
        }
  // the largest meshes: no index of the last window's threads beyond int
  for (int nx : {(1 << 30) + 1, 2147483647 - 600, 2147483647 - 512, 2147483647 - 300, 2147483647 - 200, 2147483647 - 150,
                 2147483647})
    for (int nv : {2, 15})
      for (int order : {2, 3, 4}) {
        if (!line_takes(nx)) continue;
        const LinePlan p = line_plan(nx, nv, order, 256, 10, nv > 5, true);
        const long long grid = ((long long)nx + p.own - 1) / p.own;
        const bool over = (long long)nx + p.own - 1 > 2147483647ll ||
                          (grid - 1) * p.own - p.halo + p.threads - 1 > 2147483647ll;
        if (over) std::printf("nx %d nv %d order %d: an index past int\n", nx, nv, order);
        bad += over;
      }
  for (int nx : {1, 64, 1 << 30, 2147483647 - 600}) bad += !line_takes(nx);
  // (the Euler system at P4 on large meshes takes one step per launch: the
  // odd counts there end in a copy)
  for (int order : {3, 4}) {
    const LinePlan p = line_plan(900001, 15, order, 256, 3, true, true);
    bad += p.steps != 1 || line_launches(p, 3) != 3;
  }
  std::printf("%d launches, %d failures\n", launches, bad);
  return bad ? 1 : 0;
}
