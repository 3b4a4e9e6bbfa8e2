// The walks of the neighbour search, run on the host: for boxes of few and of
// more cells, the partners of every particle in the order of the one-thread
// walk and in that of several lanes per particle.  Prints one line per box:
//   short-axis rule, particles whose order differs with pruned rows
//   throughout, the same with the exact rows of short axes, and particles
//   whose order differs between the whole rows and the ordered pruned ones
//   (the reaction's walks of the rigid grid; no outer walls)
#include <hip/hip_runtime.h>
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#define __builtin_amdgcn_sqrtf sqrtf
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "sdpdem_device.h"
using namespace sdpdem;

struct Box {
  Geo B;
  Grid G;
  std::vector<D4> x;
  std::vector<int> start, item;  // cells, then the cells of the outer walls
  int woff;
};

template <class Fn>
static void take(const Box& b, int i, double R, int c0, int c1, Fn&& fn) {
  for (int q = b.start[c0]; q < b.start[c1]; ++q) {
    const int j = b.item[q];
    double ex = b.x[i].x - b.x[j].x, ey = b.x[i].y - b.x[j].y, ez = b.x[i].z - b.x[j].z;
    min_img_box(b.B, ex, ey, ez);
    if (j != i && r2_exact(ex, ey, ez) < R * R) fn(j);
  }
}

template <bool FP32, bool EXACT>
static int differing(const Box& b, double R) {
  int bad = 0;
  const int kr = reach_cells(b.G, R), cells = b.G.nc[0] * b.G.nc[1] * b.G.nc[2];
  for (int i = 0; i < (int)b.x.size(); ++i) {
    const D4 p = b.x[i];
    int oob = 0;
    const int cc[3] = {cell_coord(p.x, b.G, 0, &oob), cell_coord(p.y, b.G, 1, &oob),
                       cell_coord(p.z, b.G, 2, &oob)};
    std::vector<int> one, many;
    const auto into = [&](std::vector<int>& v, int c0, int c1) {
      take(b, i, R, c0, c1, [&](int j) { v.push_back(j); });
      if (b.woff) take(b, i, R, c0 + b.woff, c1 + b.woff, [&](int j) { v.push_back(j); });
    };
    for_search(b.B, b.G, 0, p.x, p.y, p.z, R, cc, kr,
               [&](int c0, int c1) { into(one, c0, c1); });
    const StencilShape sh = stencil_shape(b.G, cc, kr);
    PlainRows rows = {};
    if (FP32 || EXACT) rows = plain_rows(b.B, b.G, p.x, p.y, p.z, R, cc, kr);
    for (int zi = 0; zi < sh.zn; ++zi)
      for (int yi = 0; yi < sh.yn; ++yi) {
        int a0, a1, b0, b1;
        bool all;
        search_row<FP32, EXACT>(b.B, b.G, 0, p.x, p.y, p.z, R, cc, kr, sh, rows, zi, yi, a0, a1,
                                b0, b1, all);
        if (all) {  // both runs, then the walls of both
          const auto found = [&](int j) { many.push_back(j); };
          for (int w = 0; w <= b.woff; w += cells) {
            take(b, i, R, a0 + w, a1 + w, found);
            take(b, i, R, b0 + w, b1 + w, found);
          }
        } else {
          if (a1 > a0) into(many, a0, a1);
          if (b1 > b0) into(many, b0, b1);
        }
      }
    bad += one != many;
  }
  return bad;
}

static int differing_ordered(const Box& b, double R) {
  int bad = 0;
  const int kr = reach_cells(b.G, R);
  for (int i = 0; i < (int)b.x.size() && !b.woff; ++i) {
    const D4 p = b.x[i];
    int oob = 0;
    const int cc[3] = {cell_coord(p.x, b.G, 0, &oob), cell_coord(p.y, b.G, 1, &oob),
                       cell_coord(p.z, b.G, 2, &oob)};
    std::vector<int> one, many;
    for_stencil<false>(b.B, b.G, 0, p.x, p.y, p.z, R, cc, kr, [&](int c0, int c1) {
      take(b, i, R, c0, c1, [&](int j) { one.push_back(j); });
    });
    const StencilShape sh = stencil_shape(b.G, cc, kr);
    for (int r = 0; r < sh.zn * sh.yn; ++r) {
      int a0, a1, b0, b1;
      stencil_row<true, true>(b.B, b.G, 0, p.x, p.y, p.z, R, cc, kr, sh, r, a0, a1, b0, b1);
      take(b, i, R, a0, a1, [&](int j) { many.push_back(j); });
      take(b, i, R, b0, b1, [&](int j) { many.push_back(j); });
    }
    bad += one != many;
  }
  return bad;
}

int main() {
  std::mt19937_64 gen(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  for (int kr = 1; kr <= 3; ++kr)
    for (int nx = 3; nx <= 11; ++nx)
      for (int other : {3, 7})
        for (int per = 0; per < 4; ++per) {  // walls in x; in z; none; none, sheared
          Box b = {};
          const double R = 1.0;
          b.B.le = per == 3;
          int cells = 1;
          for (int a = 0; a < 3; ++a) {
            b.G.per[a] = b.B.per[a] = !(per == 0 && a == 0) && !(per == 1 && a == 2);
            b.G.nc[a] = a == 0 ? nx : other;
            // from just above R / kr up to R / (kr - 1/2)
            const double cs = R / (kr - 0.5 * u(gen)) * (1.0 + 1e-6);
            b.G.cs[a] = cs;
            b.G.inv_cs[a] = 1.0 / cs;
            b.G.lo[a] = -0.3;
            b.B.L[a] = cs * b.G.nc[a];
            b.B.halfL[a] = 0.5 * b.B.L[a];
            b.B.lim[a] = b.G.per[a] ? b.B.halfL[a] : 1e300;
            cells *= b.G.nc[a];
          }
          if (reach_cells(b.G, R) != kr) return 1;
          b.B.inv_Lx = 1.0 / b.B.L[0];
          b.B.le_shift = b.B.le ? u(gen) * b.B.L[0] : 0.0;
          b.woff = per < 2 ? cells : 0;
          const int n = std::min(4 * cells, 600);
          std::vector<std::vector<int>> in((size_t)2 * cells);
          for (int i = 0; i < n; ++i) {
            D4 p = {b.G.lo[0] + u(gen) * b.B.L[0], b.G.lo[1] + u(gen) * b.B.L[1],
                    b.G.lo[2] + u(gen) * b.B.L[2], 0.0};
            if (i % 5 == 0)  // on a cell's face
              p.x = b.G.lo[0] + b.G.cs[0] * (double)(int)(u(gen) * nx);
            b.x.push_back(p);
            int oob = 0;
            const int c = cell_index(b.G, cell_coord(p.x, b.G, 0, &oob),
                                     cell_coord(p.y, b.G, 1, &oob), cell_coord(p.z, b.G, 2, &oob));
            in[(size_t)c + (b.woff && i % 7 == 0 ? cells : 0)].push_back(i);
          }
          for (const auto& c : in) {
            b.start.push_back((int)b.item.size());
            b.item.insert(b.item.end(), c.begin(), c.end());
          }
          b.start.push_back((int)b.item.size());
          std::printf("%d %d %d %d %d %d %d %d %d %d\n", kr, nx, other, per,
                      search_axis_short(b.G, b.B.le, kr) ? 1 : 0, differing<true, false>(b, R),
                      differing<false, false>(b, R), differing<true, true>(b, R),
                      differing<false, true>(b, R), differing_ordered(b, R));
        }
}
