// sdpdem_neighbors.hip -- neighbour build with density, pressure filter and
// SDPD pair forces: one thread per particle in cell-sorted order (several
// lanes per particle where a system is too small to fill the chip), blocks
// mapped to XCDs in contiguous chunks, neighbour data gathered through L1/L2
// (the sorted order keeps a wave's neighbourhood compact).
#include <hip/hip_ext.h>

#include "sdpdem_device.h"

namespace sdpdem {

// ---------------------------------------------------------------------------
// (a2)+(a3) neighbour sets {j : r_ij^2 < h^2} (double precision, no
// contraction) fused with the density summation (Eq. compdens), the
// equation of state (Eq. prtcpres) and the free-surface clamp.  The
// stencil is walked row by row; the cells of a row are one contiguous slice
// of the sorted arrays unless the row wraps.  With CAND (candidate reuse)
// the walk reaches h + skin and also keeps every partner within it, with
// the positions it saw, for the list builds until the next search.

// density and pressure of particle i from its kernel sum, and its
// (position, pressure) record for the filter
__device__ __forceinline__ void finish_density(const Dev& d, int i, const D4& pi, double acc) {
  const double rho = d.cw_m * acc;
  double p = d.p0 * pow(rho / d.rho0, d.alpha) - d.beta;
  if (d.clamp && p < 0.0) p = 0.0;  // free-surface correction (Sec. 2.5)
  d.rho[i] = rho;
  d.p[i] = p;
  d.xp[i] = D4{pi.x, pi.y, pi.z, p};
}

// Lucy kernel of a pair, W = x * y (the sum takes the product fused, in the
// same form everywhere, so that every kernel that sums a row in slot order
// gives the same bits)
__device__ __forceinline__ double2 lucy_parts(const Dev& d, double r2) {
  const double q = sqrt_nr(r2) * d.inv_h;
  const double om = 1.0 - q;
  return make_double2(d.w_norm * (1.0 + 3.0 * q) * om * om, om);
}

// Wide kernels: G consecutive lanes per particle, each evaluating one slot
// (or candidate) of a round, for systems whose particles alone would leave
// most of the chip's 1024 SIMDs idle; there the time is the length of the
// chain of dependent loads of one particle, which G lanes walk G times
// shorter.  The contributions pass through LDS and are added in slot order,
// exactly the sums of the one-lane kernels bit for bit: a box gives the same
// bits whichever kernels its batch is large enough for.  A lane without a
// slot contributes an exact zero.
//
// How many lanes, from the particles a launch covers: measured on periodic
// boxes, us per launch with 1 / 4 / 16 lanes (h = 1.5 dx):
//
//   particles               4,096           32,768         110,592         373,248
//   search, cells of h   100/32/16       96/35/31       112/58/72      153/136/190
//   candidate filter   14.5/10.6/8.5  14.7/11.1/13.9  16.7/16.0/28.6  29.5/37.4/74.9
//   pressure filter    15.3/9.7/8.3   15.4/11.1/13.4  20.6/15.9/27.9  32.2/34.4/69.9
//   pair forces, kT = 0 12.9/9.5/7.5  14.1/10.4/11.3  15.9/18.2/25.8  38.0/43.3/72.3
//   pair forces, kT > 0 22.3/12.3/9.0 23.0/13.7/16.8  30.1/25.9/37.6  64.2/64.9/111
//
// Sixteen lanes win up to about 2^14 particles; four up to 2.6e5 in the
// pressure filter, 2e5 in the thermal and 1e5 in the plain pair forces and
// the candidate filter.  In the search, whose walk is the longest, four lanes
// win up to 6e5 particles (512,000: 178/175 us, 729,000: 230/236), 8.5e5 in
// sheared boxes (766,801: 310/280, in cells of 0.67 h 248/243; 924,604:
// 286/291) and 2e5 active ones between walls, whose blocks are unevenly full
// (56^3 of water, 307,208 in all: 74/74).
static constexpr int LANES16_MAX = 1 << 14;
static constexpr int SEARCH4_MAX = 600000, SEARCH4_SHEARED = 850000, SEARCH4_WALLED = 200000;
static constexpr int SMOOTH4_MAX = 1 << 18, THERMAL4_MAX = 200000, ROWS4_MAX = 100000;
static int lanes_per_particle(int particles, int max4) {
  return particles <= LANES16_MAX ? 16 : particles <= max4 ? 4 : 1;
}

// acc + x0 y0 + x1 y1 + ... over the group's lanes in order, every lane
// getting the result; sh: the wave's 64 entries
template <int G>
__device__ __forceinline__ double ordered_fma(double acc, double x, double y, double2* sh) {
  const int lane = (int)threadIdx.x & 63;
  wave_lds_sync();
  sh[lane] = make_double2(x, y);
  wave_lds_sync();
  const double2* g = sh + (lane & ~(G - 1));
#pragma unroll
  for (int l = 0; l < G; ++l) {
    const double2 v = g[l];
    acc = __builtin_fma(v.x, v.y, acc);
  }
  wave_lds_sync();
  return acc;
}

// the lanes of this group for which p holds, as bits 0 .. G-1
template <int G>
__device__ __forceinline__ unsigned group_ballot(bool p) {
  const int gbase = (int)(threadIdx.x & 63) & ~(G - 1);
  return (unsigned)(__ballot(p) >> gbase) & ((1u << G) - 1u);
}

__device__ __forceinline__ void outer_wall_fields(const Dev& d, int i, const D4& pi) {
  d.nbr_cnt[i] = 0;
  d.rho[i] = d.rho0;
  d.p[i] = d.p_ref;
  d.xp[i] = D4{pi.x, pi.y, pi.z, d.p_ref};
}

// after_drift: the build between the two passes of a step, at the
// positions the step's drift made; otherwise a build ahead of the first
// pass, at the positions the previous step's drift made
template <bool CAND>
__device__ __forceinline__ void build_density(const Dev& d, int after_drift) {
  // a search resets the moved flag: positions are measured from here on
  if (CAND && blockIdx.x == 0 && threadIdx.x == 0) {
    d.moved[0] = 0;
    d.sstep[0] = d.dstep[0] - (after_drift ? 0 : 1);
  }
  int i;
  const int b = blk_box(d, i);
  if (b < 0) return;
  const BoxD& B = d.boxes[b];
  if (i >= B.first + B.count) return;
  uint8_t ti = d.type[i];
  const D4 pi = d.pos[i];
  if (CAND) d.xref[i] = pi;
  if (ti == T_OUTER) {
    outer_wall_fields(d, i, pi);
    if (CAND) d.cand_cnt[i] = 0;
    return;
  }
  const Geo G = geo_of(B);
  const Grid gr = B.g;
  const int coff = B.cell_off;
  int oob = 0;
  const int cc[3] = {cell_coord(pi.x, gr, 0, &oob), cell_coord(pi.y, gr, 1, &oob),
                     cell_coord(pi.z, gr, 2, &oob)};
  const double h2 = d.h2;
  const double R = CAND ? d.hc : d.h;
  const double R2 = CAND ? d.hc2 : h2;
  double acc = d.W0;
  int cnt = 0, ccnt = 0;
  const size_t npad = (size_t)d.npad;
  int* const nb = d.nbr + i;
  int* const cb = CAND ? d.cand + i : nullptr;
  auto cells = [&](int k0, int k1) {
    const int jb = d.cstart[k0];
    const int je = d.cstart[k1];
    for (int j = jb; j < je; ++j) {
      const D4 pj = d.pos[j];
      double ex = pi.x - pj.x, ey = pi.y - pj.y, ez = pi.z - pj.z;
      min_img_fast(G, ex, ey, ez);
      const double r2 = r2_exact(ex, ey, ez);
      if (r2 < R2 && j != i) {
        if (CAND) {
          if (ccnt < d.maxcand) cb[(size_t)ccnt * npad] = j;
          ++ccnt;
        }
        if (!CAND || r2 < h2) {
          const double2 w = lucy_parts(d, r2);
          if (cnt < d.maxn) nb[(size_t)cnt * npad] = j;
          ++cnt;
          acc = __builtin_fma(w.x, w.y, acc);
        }
      }
    }
  };
  // a run of cells, then the outer walls binned in the same cells
  const int woff = B.wall_off;
  auto run = [&](int k0, int k1) {
    cells(k0, k1);
    if (woff) cells(k0 + woff, k1 + woff);
  };
  for_search(G, gr, coff, pi.x, pi.y, pi.z, R, cc, reach_cells(gr, R), run);
  if (cnt > d.maxn || (CAND && ccnt > d.maxcand)) {
    atomicOr(d.status, ST_NBR_OVERFLOW);
    cnt = min(cnt, d.maxn);
    ccnt = min(ccnt, d.maxcand);
  }
  d.nbr_cnt[i] = cnt;
  if (CAND) d.cand_cnt[i] = ccnt;
  finish_density(d, i, pi, acc);
}

// eight waves per SIMD for the plain search; the candidate search holds
// more state and spills below 96 registers, so it takes five
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(8))) void k_build_density(Dev d) {
  build_density<false>(d, 0);
}
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(5))) void k_build_candidates(Dev d, int after_drift) {
  build_density<true>(d, after_drift);
}

// The search with G lanes per particle (bound by the chain cell starts ->
// position -> next run of the one-lane walk: 105 us for a lattice of 8,000
// particles in cells of h, 15 us with sixteen lanes; 187 and 60 us with four
// lanes for 75,000 particles at h = 2 dx).  Lane g of a group takes every G-th
// row of the stencil (its geometry and cell starts, which the one-lane walk
// loads one after the other), then the lanes take the candidates of the
// concatenated rows G at a time; ballots give the slots in candidate order.
template <int G, bool CAND, bool EXACT>
__device__ __forceinline__ void build_density_wide(const Dev& d, int after_drift) {
  __shared__ double sums[BS / G];
  __shared__ double2 xch[BS];
  if (CAND && blockIdx.x == 0 && threadIdx.x == 0) {
    d.moved[0] = 0;
    d.sstep[0] = d.dstep[0] - (after_drift ? 0 : 1);
  }
  int i0;
  const int b = blk_box_split<G>(d, i0);
  if (b < 0) return;  // uniform over the block
  const BoxD& B = d.boxes[b];
  const int last = B.first + B.count;
  const int g = (int)threadIdx.x % G;
  const int i = i0 + (int)threadIdx.x / G;
  double2* const sh = xch + (threadIdx.x & ~63);
  if (i < last && d.type[i] != T_OUTER) {
    const D4 pi = d.pos[i];
    const Geo geo = geo_of(B);
    const Grid gr = B.g;
    const int coff = B.cell_off, woff = B.wall_off;
    int oob = 0;
    const int cc[3] = {cell_coord(pi.x, gr, 0, &oob), cell_coord(pi.y, gr, 1, &oob),
                       cell_coord(pi.z, gr, 2, &oob)};
    const double h2 = d.h2;
    const double R = CAND ? d.hc : d.h;
    const double R2 = CAND ? d.hc2 : h2;
    const int kr = reach_cells(gr, R);
    const StencilShape sh_ = stencil_shape(gr, cc, kr);
    const int nrows = sh_.zn * sh_.yn;
    PlainRows rows = {};
    if (!CAND || EXACT) rows = plain_rows(geo, gr, pi.x, pi.y, pi.z, R, cc, kr);
    const float inv_yn = 1.0f / (float)sh_.yn;
    double acc = d.W0;
    int cnt = 0, ccnt = 0;
    const size_t npad = (size_t)d.npad;
    int* const nb = d.nbr + i;
    int* const cb = CAND ? d.cand + i : nullptr;
    const unsigned below = (1u << g) - 1u;
    for (int rb = 0; rb < nrows; rb += G) {
      // row rb + g: up to two runs of consecutive cells, each followed by
      // the outer walls binned in the same cells (both first where they make
      // one run of the one-lane walk); s: first particle of a run, e: the
      // run's end in the row
      int s0 = 0, e0 = 0, s1 = 0, e1 = 0, s2 = 0, e2 = 0, s3 = 0, e3 = 0;
      if (rb + g < nrows) {
        int a0, a1, b0, b1;
        bool all;
        // row / yn without an integer division: (row + 1/2) / yn stays at
        // least 1 / (2 yn) away from every integer
        const int zi = (int)(((float)(rb + g) + 0.5f) * inv_yn), yi = rb + g - zi * sh_.yn;
        search_row<!CAND, EXACT>(geo, gr, coff, pi.x, pi.y, pi.z, R, cc, kr, sh_, rows, zi, yi, a0,
                                 a1, b0, b1, all);
        if (a1 > a0) {
          s0 = d.cstart[a0];
          e0 = d.cstart[a1] - s0;
          if (woff) {
            s1 = d.cstart[a0 + woff];
            e1 = d.cstart[a1 + woff] - s1;
          }
        }
        if (b1 > b0) {
          s2 = d.cstart[b0];
          e2 = d.cstart[b1] - s2;
          if (woff) {
            s3 = d.cstart[b0 + woff];
            e3 = d.cstart[b1 + woff] - s3;
          }
        }
        if (EXACT && all && woff) {
          const int s = s1, e = e1;
          s1 = s2;
          e1 = e2;
          s2 = s;
          e2 = e;
        }
      }
      e1 += e0;
      e2 += e1;
      e3 += e2;
      int inc = e3;
#pragma unroll
      for (int o = 1; o < G; o <<= 1) {
        const int t = __shfl_up(inc, o, G);
        if (g >= o) inc += t;
      }
      const int total = __shfl(inc, G - 1, G);
      const int off = inc - e3;
      // candidate t of the concatenated rows (i itself past their end)
      auto candidate = [&](int t) {
        int r = 0;  // last row whose offset is <= t
#pragma unroll
        for (int stp = G / 2; stp > 0; stp >>= 1)
          if (__shfl(off, r + stp, G) <= t) r += stp;
        const int q = t - __shfl(off, r, G);
        const int q0 = __shfl(e0, r, G), f0 = __shfl(s0, r, G), f2 = __shfl(s2, r, G);
        int j;
        if (woff) {
          const int q1 = __shfl(e1, r, G), q2 = __shfl(e2, r, G);
          const int f1 = __shfl(s1, r, G), f3 = __shfl(s3, r, G);
          j = q < q0 ? f0 + q : q < q1 ? f1 + (q - q0) : q < q2 ? f2 + (q - q1) : f3 + (q - q2);
        } else {
          j = q < q0 ? f0 + q : f2 + (q - q0);
        }
        return t < total ? j : i;
      };
      for (int t = g; t - g < total; t += G) {
        const int j = candidate(t);
        bool in = false, near = false;
        double2 w = make_double2(0.0, 0.0);
        if (j != i) {
          const D4 pj = d.pos[j];
          double ex = pi.x - pj.x, ey = pi.y - pj.y, ez = pi.z - pj.z;
          min_img_fast(geo, ex, ey, ez);
          const double r2 = r2_exact(ex, ey, ez);
          near = CAND && r2 < R2;
          in = r2 < h2;
          if (in) w = lucy_parts(d, r2);
        }
        const unsigned m = group_ballot<G>(in);
        const int slot = cnt + __popc(m & below);
        if (in && slot < d.maxn) nb[(size_t)slot * npad] = j;
        cnt += __popc(m);
        if (CAND) {
          const unsigned mc = group_ballot<G>(near);
          const int cs = ccnt + __popc(mc & below);
          if (near && cs < d.maxcand) cb[(size_t)cs * npad] = j;
          ccnt += __popc(mc);
        }
        acc = ordered_fma<G>(acc, w.x, w.y, sh);
      }
    }
    if (g == 0) {
      if (cnt > d.maxn || (CAND && ccnt > d.maxcand)) {
        atomicOr(d.status, ST_NBR_OVERFLOW);
        cnt = min(cnt, d.maxn);
        ccnt = min(ccnt, d.maxcand);
      }
      d.nbr_cnt[i] = cnt;
      if (CAND) d.cand_cnt[i] = ccnt;
      sums[threadIdx.x / G] = acc;
    }
  }
  __syncthreads();
  // the equation of state (an FP64 power) on full lanes
  const int k = i0 + (int)threadIdx.x;
  if ((int)threadIdx.x < BS / G && k < last) {
    const D4 pk = d.pos[k];
    if (CAND) d.xref[k] = pk;
    if (d.type[k] == T_OUTER) {
      outer_wall_fields(d, k, pk);
      if (CAND) d.cand_cnt[k] = 0;
    } else {
      finish_density(d, k, pk, sums[threadIdx.x]);
    }
  }
}

// (seven waves per SIMD pay in the larger systems that take four lanes)
template <int G, bool EXACT>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(G == 4 ? 7 : 5))) void
k_build_density_wide(Dev d) {
  build_density_wide<G, false, EXACT>(d, 0);
}
template <int G, bool EXACT>
__global__ __launch_bounds__(BS) void k_build_candidates_wide(Dev d, int after_drift) {
  build_density_wide<G, true, EXACT>(d, after_drift);
}

template <int G>
static void build_density_lanes(const Dev& d, bool cand, int after_drift, hipStream_t st) {
  const int nb = d.nblk * G;
  if (cand && d.short_x)
    k_build_candidates_wide<G, true><<<nb, BS, 0, st>>>(d, after_drift);
  else if (cand)
    k_build_candidates_wide<G, false><<<nb, BS, 0, st>>>(d, after_drift);
  else if (d.short_x)
    k_build_density_wide<G, true><<<nb, BS, 0, st>>>(d);
  else
    k_build_density_wide<G, false><<<nb, BS, 0, st>>>(d);
}

void launch_build_density(const Dev& d, bool cand, bool after_drift, hipStream_t st) {
  const int ad = after_drift ? 1 : 0;
  const int lanes = lanes_per_particle(d.nactive, d.any_le          ? SEARCH4_SHEARED
                                                  : d.nactive < d.n ? SEARCH4_WALLED
                                                                    : SEARCH4_MAX);
  if (lanes == 16)
    build_density_lanes<16>(d, cand, ad, st);
  else if (lanes == 4)
    build_density_lanes<4>(d, cand, ad, st);
  else if (cand)
    k_build_candidates<<<d.nblk, BS, 0, st>>>(d, ad);
  else
    k_build_density<<<d.nblk, BS, 0, st>>>(d);
}

// The lists of a drift that kept every particle within skin/2 of where the
// last search saw it: a partner within h now was within h + skin then, so
// the exact test over the candidates (in the same FP64 arithmetic) gives
// the same set as a search.  Density, pressure and the filter's record as
// in the search.
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(8))) void k_filter_density(Dev d) {
  int i;
  const int b = blk_box<true>(d, i);
  if (b < 0) return;
  const BoxD& B = d.boxes[b];
  if (i >= B.first + B.count) return;
  const uint8_t ti = d.type[i];
  const D4 pi = d.pos[i];
  if (ti == T_OUTER) {
    outer_wall_fields(d, i, pi);
    return;
  }
  const Geo G = geo_of(B);
  const double h2 = d.h2;
  double acc = d.W0;
  int cnt = 0;
  const size_t npad = (size_t)d.npad;
  int* const nb = d.nbr + i;
  const int* const cb = d.cand + i;
  const int cc = d.cand_cnt[i];
  // software pipeline: the position of candidate k+1 and the index of
  // candidate k+2 are in flight while candidate k is tested (past the end
  // the loads fetch the particle's own, unused, entries)
  int jn = cc > 0 ? cb[0] : i;
  D4 pn = d.pos[jn];
  int jnn = cc > 1 ? cb[npad] : i;
  for (int k = 0; k < cc; ++k) {
    const int j = jn;
    const D4 pj = pn;
    jn = jnn;
    pn = d.pos[jn];
    jnn = k + 2 < cc ? cb[(size_t)(k + 2) * npad] : i;
    double ex = pi.x - pj.x, ey = pi.y - pj.y, ez = pi.z - pj.z;
    min_img_fast(G, ex, ey, ez);
    const double r2 = r2_exact(ex, ey, ez);
    if (r2 < h2) {
      const double2 w = lucy_parts(d, r2);
      if (cnt < d.maxn) nb[(size_t)cnt * npad] = j;
      ++cnt;
      acc = __builtin_fma(w.x, w.y, acc);
    }
  }
  if (cnt > d.maxn) {
    atomicOr(d.status, ST_NBR_OVERFLOW);
    cnt = d.maxn;
  }
  d.nbr_cnt[i] = cnt;
  finish_density(d, i, pi, acc);
}

// the same with G lanes per particle
template <int G>
__global__ __launch_bounds__(BS) void k_filter_density_wide(Dev d) {
  __shared__ double sums[BS / G];
  __shared__ double2 xch[BS];
  int i0;
  const int b = blk_box_split<G, true>(d, i0);
  if (b < 0) return;  // uniform over the block
  const BoxD& B = d.boxes[b];
  const int last = B.first + B.count;
  const int g = (int)threadIdx.x % G;
  const int i = i0 + (int)threadIdx.x / G;
  double2* const sh = xch + (threadIdx.x & ~63);
  if (i < last && d.type[i] != T_OUTER) {
    const D4 pi = d.pos[i];
    const Geo geo = geo_of(B);
    const double h2 = d.h2;
    const size_t npad = (size_t)d.npad;
    int* const nb = d.nbr + i;
    const int* const cb = d.cand + i;
    const int cc = d.cand_cnt[i];
    const unsigned below = (1u << g) - 1u;
    double acc = d.W0;
    int cnt = 0;
    for (int k = g; k - g < cc; k += G) {
      bool in = false;
      double2 w = make_double2(0.0, 0.0);
      int j = i;
      if (k < cc) {
        j = cb[(size_t)k * npad];
        const D4 pj = d.pos[j];
        double ex = pi.x - pj.x, ey = pi.y - pj.y, ez = pi.z - pj.z;
        min_img_fast(geo, ex, ey, ez);
        const double r2 = r2_exact(ex, ey, ez);
        in = r2 < h2;
        if (in) w = lucy_parts(d, r2);
      }
      const unsigned m = group_ballot<G>(in);
      const int slot = cnt + __popc(m & below);
      if (in && slot < d.maxn) nb[(size_t)slot * npad] = j;
      cnt += __popc(m);
      acc = ordered_fma<G>(acc, w.x, w.y, sh);
    }
    if (g == 0) {
      if (cnt > d.maxn) {
        atomicOr(d.status, ST_NBR_OVERFLOW);
        cnt = d.maxn;
      }
      d.nbr_cnt[i] = cnt;
      sums[threadIdx.x / G] = acc;
    }
  }
  __syncthreads();
  const int k = i0 + (int)threadIdx.x;
  if ((int)threadIdx.x < BS / G && k < last) {
    const D4 pk = d.pos[k];
    if (d.type[k] == T_OUTER)
      outer_wall_fields(d, k, pk);
    else
      finish_density(d, k, pk, sums[threadIdx.x]);
  }
}

void launch_filter_density(const Dev& d, hipStream_t st) {
  const int lanes = lanes_per_particle(d.nactive, ROWS4_MAX);
  if (lanes == 16)
    k_filter_density_wide<16><<<d.nablk * 16, BS, 0, st>>>(d);
  else if (lanes == 4)
    k_filter_density_wide<4><<<d.nablk * 4, BS, 0, st>>>(d);
  else
    k_filter_density<<<d.nablk, BS, 0, st>>>(d);
}

// ---------------------------------------------------------------------------
// (a4) Shepard filter of the pressure (weights recomputed from the FP64
// positions) and the pair records of the force pass.

// the filtered pressure and the pair record of particle i
__device__ __forceinline__ void finish_smooth(const Dev& d, int i, uint8_t ti, const D4& x,
                                              double ps) {
  d.ps[i] = (float)ps;
  const double di = d.rho[i] / d.m_f;
  const D4 v = d.vel[i], w = d.om[i];
  PR r;
  r.x = x.x;
  r.y = x.y;
  r.z = x.z;
  r.vx = (float)v.x;
  r.vy = (float)v.y;
  r.vz = (float)v.z;
  r.pc = (float)(d.coef_c * ps / (di * di));
  r.wx = (float)w.x;
  r.wy = (float)w.y;
  r.wz = (float)w.z;
  r.invd = (float)(1.0 / di);
  r.gid = d.gid[i];
  r.type = ti;
  d.prec[i] = r;
}

template <bool ACT>
__global__ __launch_bounds__(BS) void k_smooth(Dev d) {
  int i;
  const int b = blk_box<ACT>(d, i);
  if (b < 0) return;
  const BoxD& B = d.boxes[b];
  if (i >= B.first + B.count) return;
  const uint8_t ti = d.type[i];
  const D4 x = d.xp[i];  // position and pressure
  const double pi = x.w;
  const Geo G = geo_of(B);
  double ps = pi;
  if (d.smooth && ti != T_OUTER) {
    double num = pi * d.W0, den = d.W0;
    const int cnt = d.nbr_cnt[i];
    const size_t npad = (size_t)d.npad;
    const int* nb = d.nbr + i;
    const double inv_h = d.inv_h;
    for (int k = 0; k < cnt; ++k) {
      const int j = nb[(size_t)k * npad];
      const D4 xj = d.xp[j];  // one 32-byte record: position and pressure
      double ex = x.x - xj.x, ey = x.y - xj.y, ez = x.z - xj.z;
      min_img_fast(G, ex, ey, ez);
      const double q = sqrt_nr(r2_exact(ex, ey, ez)) * inv_h;
      const double om = fmax(1.0 - q, 0.0);
      const double wx = d.w_norm * (1.0 + 3.0 * q) * om * om;  // W = wx om
      num = __builtin_fma(xj.w, wx * om, num);
      den = __builtin_fma(wx, om, den);
    }
    ps = num / den;
  }
  finish_smooth(d, i, ti, x, ps);
}

// the same with G lanes per particle
template <int G, bool ACT>
__global__ __launch_bounds__(BS) void k_smooth_wide(Dev d) {
  __shared__ double2 sums[BS / G];
  __shared__ double2 xch[BS];
  __shared__ double xchp[BS];
  int i0;
  const int b = blk_box_split<G, ACT>(d, i0);
  if (b < 0) return;  // uniform over the block
  const BoxD& B = d.boxes[b];
  const int last = B.first + B.count;
  const int g = (int)threadIdx.x % G;
  const int i = i0 + (int)threadIdx.x / G;
  const int lane = (int)threadIdx.x & 63;
  double2* const sh = xch + (threadIdx.x & ~63);
  if (d.smooth && i < last && d.type[i] != T_OUTER) {
    const D4 x = d.xp[i];
    const Geo geo = geo_of(B);
    double num = x.w * d.W0, den = d.W0;
    const int cnt = d.nbr_cnt[i];
    const size_t npad = (size_t)d.npad;
    const int* nb = d.nbr + i;
    for (int k = g; k - g < cnt; k += G) {
      double2 w = make_double2(0.0, 0.0);
      double pj = 0.0;
      if (k < cnt) {
        const D4 xj = d.xp[nb[(size_t)k * npad]];
        double ex = x.x - xj.x, ey = x.y - xj.y, ez = x.z - xj.z;
        min_img_fast(geo, ex, ey, ez);
        const double q = sqrt_nr(r2_exact(ex, ey, ez)) * d.inv_h;
        const double om = fmax(1.0 - q, 0.0);
        w = make_double2(d.w_norm * (1.0 + 3.0 * q) * om * om, om);
        pj = xj.w;
      }
      wave_lds_sync();
      sh[lane] = w;
      xchp[threadIdx.x] = pj;
      wave_lds_sync();
#pragma unroll
      for (int l = 0; l < G; ++l) {
        const double2 v = sh[(lane & ~(G - 1)) + l];
        num = __builtin_fma(xchp[(threadIdx.x & ~(G - 1)) + l], v.x * v.y, num);
        den = __builtin_fma(v.x, v.y, den);
      }
      wave_lds_sync();
    }
    if (g == 0) sums[threadIdx.x / G] = make_double2(num, den);
  }
  __syncthreads();
  const int k = i0 + (int)threadIdx.x;
  if ((int)threadIdx.x < BS / G && k < last) {
    const uint8_t tk = d.type[k];
    const D4 x = d.xp[k];
    double ps = x.w;
    if (d.smooth && tk != T_OUTER) ps = sums[threadIdx.x].x / sums[threadIdx.x].y;
    finish_smooth(d, k, tk, x, ps);
  }
}

template <int G>
static void smooth_lanes(const Dev& d, bool all, hipStream_t st) {
  if (all)
    k_smooth_wide<G, false><<<d.nblk * G, BS, 0, st>>>(d);
  else
    k_smooth_wide<G, true><<<d.nablk * G, BS, 0, st>>>(d);
}

// after a search over every particle (the outer walls' records too: the
// sort may have moved them), after a candidate filter over the active parts
void launch_smooth(const Dev& d, bool all, hipStream_t st) {
  const int lanes = lanes_per_particle(all ? d.n : d.nactive, SMOOTH4_MAX);
  if (lanes == 16)
    smooth_lanes<16>(d, all, st);
  else if (lanes == 4)
    smooth_lanes<4>(d, all, st);
  else if (all)
    k_smooth<false><<<d.nblk, BS, 0, st>>>(d);
  else
    k_smooth<true><<<d.nablk, BS, 0, st>>>(d);
}

// ---------------------------------------------------------------------------
// (a5) SDPD+a pair forces, Eqs. FijC, FijD, FijR, FijT, for fluid and
// inner-wall particles: FP32 math on FP64-differenced separations, FP32
// per-particle sums; outputs F^SDPD, its torque and the F^C + F^D sum.

// what the pair loop needs of particle i besides its record
struct PairCtx {
  Geo G;
  uint32_t ib, gi;  // box's first id, box-local noise index of i
  float jump;
  float across, along, nl_hi, nl_lo;  // thermal amplitudes (BoxD)
  bool le, noise;
  uint32_t key0, key1, step;
};

template <bool NOISE>
__device__ __forceinline__ PairCtx pair_ctx(const Dev& d, const BoxD& B, const PR& ri) {
#pragma clang fp contract(off)
  PairCtx c;
  c.ib = B.id_base;
  c.gi = (uint32_t)ri.gid - c.ib;
  c.G = geo_of(B);
  c.le = c.G.le;
  c.jump = (float)c.G.le_jump;
  c.noise = NOISE && B.noise;
  c.across = NOISE ? B.across : 0.0f;
  c.along = NOISE ? B.along : 0.0f;
  c.nl_hi = NOISE ? B.nl_hi : 0.0f;
  c.nl_lo = NOISE ? B.nl_lo : 0.0f;
  c.key0 = B.key0;
  c.key1 = B.key1;
  c.step = NOISE ? (uint32_t)d.dstep[0] : 0u;  // noise counter
  return c;
}

// the pair force of partner j on i: [0..2] F, [3..5] torque without its
// lever, [6..8] F^C + F^D, [9] virial share.  Fused operations are written
// out, so that every kernel that calls this rounds alike.
enum { PT_N = 10 };

template <bool NOISE, bool STRESS>
__device__ __forceinline__ void pair_terms(const Dev& d, const PairCtx& c, const PR& ri,
                                           const PR& rj, float out[PT_N]) {
#pragma clang fp contract(off)
  const auto fma = [](float x, float y, float z) { return __builtin_fmaf(x, y, z); };
  double dx_ = ri.x - rj.x, dy_ = ri.y - rj.y, dz_ = ri.z - rj.z;
  const int kz = NOISE ? min_img_fast(c.G, dx_, dy_, dz_) : min_img_box(c.G, dx_, dy_, dz_);
  const double r2d = __builtin_fma(dz_, dz_, __builtin_fma(dx_, dx_, dy_ * dy_));
  const float rx = (float)dx_, ry = (float)dy_, rz = (float)dz_;
  const float r2f = (float)r2d, inv_r = __builtin_amdgcn_rsqf(r2f);
  const float ex = rx * inv_r, ey = ry * inv_r, ez = rz * inv_r;
  // 1 - r/h = (h^2 - r^2) / (h (h + r)), the difference taken in FP64 so
  // that pairs close to the cut-off keep full FP32 relative precision
  const float omq = fmaxf(
      (float)(d.h2 - r2d) * d.inv_hf * __builtin_amdgcn_rcpf(fma(r2f, inv_r, d.hf)), 0.0f);
  const float Fk = d.cFf * omq * omq;  // F(r) = -W'(r)/r, Eq. F
  // Pair force = along-e part + transverse part.  The torque takes the
  // transverse part only (e x e = 0), which keeps the FP32 cross product
  // free of the cancellation of the dominant pressure term.
  // conservative force, Eq. FijC: (p_i/d_i^2 + p_j/d_j^2) F r_ij
  const float pc = (ri.pc + rj.pc) * Fk;
  // F / (d_i d_j): the two inverse densities multiply symmetrically so
  // that F_ji = -F_ij holds bit for bit
  const float fdd = Fk * (ri.invd * rj.invd);
  // dissipative force, Eq. FijD: -ga v_ij - (ga + 2 gb)/3 (e.v_ij) e; a
  // partner seen through a sheared z face moves with its image velocity
  float vx = ri.vx - rj.vx;
  if (c.le) vx = fma(-(float)kz, c.jump, vx);
  const float vy = ri.vy - rj.vy, vz = ri.vz - rj.vz;
  const float ev = fma(ez, vz, fma(ex, vx, ey * vy));
  const float cde = d.kBf * fdd * ev;
  const float cdv = d.kAf * fdd;
  const float cx_ = fma(cdv, vx, fma(pc, rx, cde * ex));
  const float cy_ = fma(cdv, vy, fma(pc, ry, cde * ey));
  const float cz_ = fma(cdv, vz, fma(pc, rz, cde * ez));
  // rotational force, Eq. FijR: -gamma^a (r_ij / 2) x (w_i + w_j)
  const float sx = ri.wx + rj.wx, sy = ri.wy + rj.wy, sz = ri.wz + rj.wz;
  const float gr = d.kRf * fdd;
  const float qx = fma(ry, sz, -(rz * sy)), qy = fma(rz, sx, -(rx * sz)),
              qz = fma(rx, sy, -(ry * sx));
  float fx = fma(gr, qx, cx_), fy = fma(gr, qy, cy_), fz = fma(gr, qz, cz_);
  float tx = fma(cdv, vx, gr * qx), ty = fma(cdv, vy, gr * qy), tz = fma(cdv, vz, gr * qz);
  if (c.noise) {
    // thermal force, Eq. FijT: (sa dW^S + sb tr(dW)/3 1) e for a matrix
    // of independent increments is Gaussian with variance 1/2 across e
    // and sa^2 2/3 + sb^2 1/3 along it (in units of sa^2 and dt), the
    // two parts independent: s_ij P_perp z / sqrt 2 with z = (z0, z1,
    // z2) plus z3 along e, s_ij = +1 for gid_i < gid_j (F_ji = -F_ij)
    float z[4];
    const uint32_t gi = c.gi, gj = (uint32_t)rj.gid - c.ib;
    pair_normals(gi, gj, c.step, c.key0, c.key1, c.nl_hi, c.nl_lo, z);
    const float ze = fma(z[2], ez, fma(z[0], ex, z[1] * ey));
    const float px = fma(-ze, ex, z[0]), py = fma(-ze, ey, z[1]), pz = fma(-ze, ez, z[2]);
    const float sf = sqrtf_nr(fdd);
    const float cp = sf * (gi < gj ? c.across : -c.across);
    const float cq = sf * c.along * z[3];
    fx = fma(cq, ex, fma(cp, px, fx));
    fy = fma(cq, ey, fma(cp, py, fy));
    fz = fma(cq, ez, fma(cp, pz, fz));
    // the torque takes the part across e (e x e = 0)
    tx = fma(cp, px, tx);
    ty = fma(cp, py, ty);
    tz = fma(cp, pz, tz);
  }
  out[0] = fx;
  out[1] = fy;
  out[2] = fz;
  // torque: lever dx/2 along -e_ij (Sec. 2.6), lever applied to the sum
  out[3] = fma(ey, tz, -(ez * ty));
  out[4] = fma(ez, tx, -(ex * tz));
  out[5] = fma(ex, ty, -(ey * tx));
  out[6] = cx_;
  out[7] = cy_;
  out[8] = cz_;
  // virial r_z F_x: half of a pair that j evaluates too, all of a pair with
  // a rigid or outer-wall partner (it does not)
  out[9] = STRESS ? ((rj.type == T_FLUID || rj.type == T_INNER) ? 0.5f : 1.0f) * rz * fx : 0.0f;
}

// one addition, rounded
__device__ __forceinline__ float add_rounded(float a, float b) {
#pragma clang fp contract(off)
  return a + b;
}

template <bool STRESS>
__global__ __launch_bounds__(BS) void k_fluid_forces(Dev d, int) {
  int i;
  const int b = blk_box<true>(d, i);
  if (b < 0) return;
  const BoxD& B = d.boxes[b];
  if (i >= B.first + B.count) return;
  const uint8_t ti = d.type[i];
  float acc[PT_N];
#pragma unroll
  for (int q = 0; q < PT_N; ++q) acc[q] = 0.0f;
  if (ti == T_FLUID || ti == T_INNER) {
    const PR ri = load_pr(d.prec, i);
    const PairCtx c = pair_ctx<false>(d, B, ri);
    const int cnt = d.nbr_cnt[i];
    const int* nb = d.nbr + i;
    const size_t npad = (size_t)d.npad;
    // the index of slot k+1 is in flight while slot k is evaluated (holding
    // the next record too costs 19 registers: 7 waves per SIMD instead of 8,
    // and the kernel is 4 % slower)
    int jn = cnt > 0 ? nb[0] : i;
    for (int k = 0; k < cnt; ++k) {
      const PR rj = load_pr(d.prec, jn);
      jn = k + 1 < cnt ? nb[(size_t)(k + 1) * npad] : i;
      float t[PT_N];
      pair_terms<false, STRESS>(d, c, ri, rj, t);
#pragma unroll
      for (int q = 0; q < (STRESS ? 10 : 9); ++q) acc[q] = add_rounded(acc[q], t[q]);
    }
    acc[3] *= -d.leverf;
    acc[4] *= -d.leverf;
    acc[5] *= -d.leverf;
  }
  const size_t np = (size_t)d.npad;
  float* o = d.fout;
#pragma unroll
  for (int q = 0; q < 9; ++q) o[q * np + i] = acc[q];
  if (STRESS) o[12 * np + i] = acc[9];
}

// The thermal pair kernel of large systems.  Its arithmetic (the Philox
// block and the normals of a pair) leaves little of the texture-address unit
// to spare, and a lane loading its partner's 64-byte record takes that unit
// one cycle per lane and 16 bytes: 95 % of the time.  Here the four lanes of
// a quad load one record together, so a cycle fetches 64 bytes, straight into
// LDS (no registers for loads in flight), and every lane then reads its own
// partner from there; the next slot's records are on their way while a slot
// is evaluated.  Periodic box of 4.2 M particles: 620 us per launch with
// per-lane loads, 512 us so; 256 sheared cells' worth of spheres and fluid
// 290 to 255 us.  (The plain pair kernel has a third of the arithmetic and
// waits on the caches: 136 us per-lane, 143 us so on the dam break, so it
// keeps the loads per lane.)
//
// A quad's record lies in LDS in the quarters' order q ^ t (t: which of its
// lanes wants it), which spreads the lanes' reads over the banks.  WIDE_OFS:
// byte offsets into the records need more than 32 bits.
template <bool STRESS, bool WIDE_OFS, bool UPDATE>
__global__ __launch_bounds__(BS) void k_fluid_forces_thermal(Dev d, int track) {
  __shared__ __attribute__((aligned(64))) char stage[BS * sizeof(PR)];
  int i;
  const int b = blk_box<true>(d, i);
  if (b < 0) return;  // uniform over the block
  const BoxD& B = d.boxes[b];
  // every lane stays to load for its quad; one past the box's end as its
  // first particle, with no slots of its own
  const bool live = i < B.first + B.count;
  if (!live) i = B.first;
  const uint8_t ti = d.type[i];
  const PR ri = load_pr(d.prec, i);
  const PairCtx c = pair_ctx<true>(d, B, ri);
  const int cnt = live && (ti == T_FLUID || ti == T_INNER) ? d.nbr_cnt[i] : 0;
  const int* const nb = d.nbr + i;
  const size_t npad = (size_t)d.npad;
  const uint32_t lane = threadIdx.x & 63u, t = lane & 3u;
  char* const st = stage + __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u)) * sizeof(PR);
  const char* const base = reinterpret_cast<const char*>(d.prec);
  // the records of the wave's 64 partners, 16 by 16: lane q of a quad takes
  // quarter q ^ t of the record its lane t wants
  auto fetch = [&](int j) {
#define SDPDEM_FETCH(T)                                                                        \
  {                                                                                            \
    const uint32_t jt =                                                                        \
        (uint32_t)__builtin_amdgcn_mov_dpp(j, (T) * 0x55, 0xF, 0xF, true);                     \
    const uint32_t quarter = (t ^ (T)) * 16u;                                                  \
    const char* const src = WIDE_OFS ? base + ((size_t)jt * sizeof(PR) + quarter)              \
                                     : base + (jt * (uint32_t)sizeof(PR) + quarter);           \
    load_to_lds16(src, st + (T) * 1024);                                                       \
  }
    SDPDEM_FETCH(0)
    SDPDEM_FETCH(1)
    SDPDEM_FETCH(2)
    SDPDEM_FETCH(3)
#undef SDPDEM_FETCH
  };
  const uint32_t mine = t * 1024u + (lane >> 2) * 64u + t * 16u;
  int kmax = cnt;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, 64));
  kmax = __builtin_amdgcn_readfirstlane(kmax);
  // a lane past its row's end asks for its own record
  int jn = cnt > 0 ? nb[0] : i;
  int jnn = cnt > 1 ? nb[npad] : i;
  if (kmax > 0) fetch(jn);
  jn = jnn;
  float acc[PT_N];
#pragma unroll
  for (int q = 0; q < PT_N; ++q) acc[q] = 0.0f;
  for (int k = 0; k < kmax; ++k) {
    wait_loads();
    union {
      PR r;
      float4 q[4];
    } rj;
#pragma unroll
    for (int m = 0; m < 4; ++m)
      rj.q[m] = *reinterpret_cast<const float4*>(st + (mine ^ (uint32_t)(m * 16)));
    wait_lds();  // read before the next records land there
    jnn = k + 2 < cnt ? nb[(size_t)(k + 2) * npad] : i;
    fetch(jn);
    jn = jnn;
    if (k < cnt) {
      float tt[PT_N];
      pair_terms<true, STRESS>(d, c, ri, rj.r, tt);
#pragma unroll
      for (int q = 0; q < (STRESS ? 10 : 9); ++q) acc[q] = add_rounded(acc[q], tt[q]);
    }
  }
  wait_loads();  // no load into LDS outlives its wave
  if (!live) return;
  acc[3] *= -d.leverf;
  acc[4] *= -d.leverf;
  acc[5] *= -d.leverf;
  if (UPDATE) {
    first_update(d, track, B, i, ti, acc);
    return;
  }
  const size_t np = (size_t)d.npad;
  float* const o = d.fout;
#pragma unroll
  for (int q = 0; q < 9; ++q) o[q * np + i] = acc[q];
  if (STRESS) o[12 * np + i] = acc[9];
}

// the same with G lanes per particle: the lanes' pair terms pass through
// LDS and lane q of the group adds component q over the slots in order
template <int G, bool NOISE, bool STRESS, bool UPDATE>
__global__ __launch_bounds__(BS) void k_fluid_forces_wide(Dev d, int track) {
  constexpr int NT = STRESS ? 10 : 9, PER = (NT + G - 1) / G;
  constexpr int ST = 12;                  // floats of a lane's row (16-byte stores)
  __shared__ __align__(16) float xch[BS * ST];
  int i0;
  const int b = blk_box_split<G, true>(d, i0);
  if (b < 0) return;  // uniform over the block
  const BoxD& B = d.boxes[b];
  const int g = (int)threadIdx.x % G;
  const int i = i0 + (int)threadIdx.x / G;
  const int last = B.first + B.count;
  if (!UPDATE && i >= last) return;
  const uint8_t ti = i < last ? d.type[i] : (uint8_t)T_OUTER;
  float acc[PER];
#pragma unroll
  for (int m = 0; m < PER; ++m) acc[m] = 0.0f;
  if (ti == T_FLUID || ti == T_INNER) {
    const PR ri = load_pr(d.prec, i);
    const PairCtx c = pair_ctx<NOISE>(d, B, ri);
    const int cnt = d.nbr_cnt[i];
    const int* nb = d.nbr + i;
    const size_t npad = (size_t)d.npad;
    float* const row = xch + (size_t)threadIdx.x * ST;
    const float* const grp = xch + (size_t)(threadIdx.x & ~(G - 1)) * ST;
    for (int k = g; k - g < cnt; k += G) {
      float t[ST];
#pragma unroll
      for (int q = 0; q < ST; ++q) t[q] = 0.0f;
      if (k < cnt) pair_terms<NOISE, STRESS>(d, c, ri, load_pr(d.prec, nb[(size_t)k * npad]), t);
      wave_lds_sync();
#pragma unroll
      for (int q = 0; q < ST; q += 4)
        *reinterpret_cast<float4*>(row + q) = make_float4(t[q], t[q + 1], t[q + 2], t[q + 3]);
      wave_lds_sync();
      // adding an exact zero past the row's end would turn a sum of -0
      // into +0: stop at the last slot
      const int m = min(G, cnt - (k - g));
      for (int l = 0; l < m; ++l)
#pragma unroll
        for (int p = 0; p < PER; ++p)
          if (p * G + g < NT) acc[p] = add_rounded(acc[p], grp[l * ST + p * G + g]);
      wave_lds_sync();
    }
  }
  const size_t np = (size_t)d.npad;
  if (UPDATE) __syncthreads();  // the exchange rows are free
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int q = p * G + g;
    if (q >= NT) continue;
    if (q >= 3 && q < 6) acc[p] *= -d.leverf;
    if (UPDATE)
      xch[((int)threadIdx.x / G) * ST + q] = acc[p];
    else
      d.fout[(q < 9 ? q : 12) * np + i] = acc[p];
  }
  if (UPDATE) {
    // on full lanes
    __syncthreads();
    const int k = i0 + (int)threadIdx.x;
    if ((int)threadIdx.x < BS / G && k < last)
      first_update(d, track, B, k, d.type[k], xch + threadIdx.x * ST);
  }
}

// Where the kernel of a step's first pass also updates its particles (without
// active spheres nothing else comes between, so the sums need not pass through
// memory): the thermal kernel, whose arithmetic covers the update's memory
// traffic (periodic box of 4.2 M particles, 514 + 210 us in two launches, 647
// in one), and the several-lane kernels, where a launch less counts (8,000
// particles 7.8 + 4.7 us, 8.9 in one).  Not the plain one-lane kernel (117 +
// 55, 192 us: it waits on memory itself), and not a second pass, whose update
// rewrites the pair records that the launch still reads (with a second array
// of records 514 + 237, 776 us).
static int forces_lanes_count(const Dev& d, bool noise) {
  return lanes_per_particle(d.nactive, noise ? THERMAL4_MAX : ROWS4_MAX);
}
bool forces_can_update(const Dev& d, bool noise) {
  return noise || forces_lanes_count(d, noise) > 1;
}

template <int G, bool NOISE>
static auto forces_lanes(const Dev& d, bool update) {
  return d.stress ? k_fluid_forces_wide<G, NOISE, true, false>
         : update ? k_fluid_forces_wide<G, NOISE, false, true>
                  : k_fluid_forces_wide<G, NOISE, false, false>;
}
template <bool WIDE_OFS>
static auto forces_thermal(const Dev& d, bool update) {
  return d.stress ? k_fluid_forces_thermal<true, WIDE_OFS, false>
         : update ? k_fluid_forces_thermal<false, WIDE_OFS, true>
                  : k_fluid_forces_thermal<false, WIDE_OFS, false>;
}

void launch_fluid_forces(const Dev& d, bool noise, bool update, bool track, hipStream_t st,
                         hipEvent_t t0, hipEvent_t t1) {
  auto k = d.stress ? k_fluid_forces<true> : k_fluid_forces<false>;
  const int lanes = forces_lanes_count(d, noise);
  if (lanes == 16)
    k = noise ? forces_lanes<16, true>(d, update) : forces_lanes<16, false>(d, update);
  else if (lanes == 4)
    k = noise ? forces_lanes<4, true>(d, update) : forces_lanes<4, false>(d, update);
  else if (noise)
    k = (size_t)d.npad * sizeof(PR) > (size_t)UINT32_MAX ? forces_thermal<true>(d, update)
                                                         : forces_thermal<false>(d, update);
  int moved = track ? 1 : 0;
  const unsigned nb = (unsigned)(d.nablk * lanes);
  if (t0 && t1) {
    // the dispatch itself stamps the two events (no marker packets around
    // the kernel, which would stall the stream)
    Dev arg = d;
    void* args[] = {&arg, &moved};
    if (hipExtLaunchKernel(reinterpret_cast<const void*>(k), dim3(nb), dim3(BS), args, 0, st,
                           t0, t1, 0) == hipSuccess)
      return;
  }
  k<<<nb, BS, 0, st>>>(d, moved);
}

// neighbour columns k0..k0+kn-1 as ids (-1 past a row's end), for export
__global__ __launch_bounds__(BS) void k_nbr_cols(Dev d, int k0, int kn, int* out) {
  const int i = xcd_tid();
  if (i >= d.n) return;
  const int cnt = d.nbr_cnt[i];
  const size_t np = (size_t)d.npad;
  for (int k = 0; k < kn; ++k) {
    const int kk = k0 + k;
    out[(size_t)k * np + i] = kk < cnt ? d.gid[d.nbr[(size_t)kk * np + i]] : -1;
  }
}

void launch_nbr_cols(const Dev& d, int k0, int kn, int* out, hipStream_t st) {
  k_nbr_cols<<<nblocks(d.n), BS, 0, st>>>(d, k0, kn, out);
}

}  // namespace sdpdem
