// The coarse part of a V-cycle (Alg. 2, nu1 = nu2 = 1, zero initial guess)
// for levels lp .. L-1 in one launch, one workgroup per right-hand side, or in
// two where the coarsest product is the long part (second half of this file).
// The right-hand sides are independent, so every sweep of a level only
// needs a workgroup barrier; the level buffers of one right-hand side stay
// in LDS or L2.  Per level l (h_l^2-scaled operators, W = omega / diag(K_l)):
//   down: e = W r;  t = r - K e = (1 - w) r + sum of neighbours of e;  r_{l+1} = 4 R t
//   coarsest: e = K^-1 r (explicit inverse)
//   up:   t = e + P e_{l+1};  e = (1 - w) t + W (r + sum of neighbours of t)
#include <algorithm>

#include "dev_common.h"
#include "kernels.h"

namespace {

constexpr int CC_NT = 1024;

// The three stencils below read their neighbours without branches, from the nearest point of
// the grid, and select: a read under `inside` is a branch and a wait of its own for each
// neighbour, and a stage of these kernels is little else.

// sum of the in-grid neighbours of point p (the order of neighbour_sum)
template <int DIM>
__device__ __forceinline__ c32 neighbours(const c32* v, int p, const Coord& c, int n) {
  const int st[3] = {1, n, n * n}, x[3] = {c.x, c.y, c.z};
  c32 q[2 * DIM];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    q[2 * d] = v[x[d] > 0 ? p - st[d] : p];
    q[2 * d + 1] = v[x[d] < n - 1 ? p + st[d] : p];
  }
  c32 s = make_float2(0.f, 0.f);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const bool lo = x[d] > 0, hi = x[d] < n - 1;
    s.x += lo ? q[2 * d].x : 0.f;
    s.y += lo ? q[2 * d].y : 0.f;
    s.x += hi ? q[2 * d + 1].x : 0.f;
    s.y += hi ? q[2 * d + 1].y : 0.f;
  }
  return s;
}

// 4 * full weighting of s at coarse point C (neighbours outside the fine grid count as 0)
template <int DIM>
__device__ __forceinline__ c32 fw4(const c32* s, const Coord& C, int nf) {
  const float w1[3] = {0.25f, 0.5f, 0.25f};
  int ix[3], iy[3], iz[3];
  bool bx[3], by[3], bz[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int fx = 2 * C.x + d - 1, fy = 2 * C.y + d - 1, fz = 2 * C.z + d - 1;
    bx[d] = fx >= 0 && fx < nf;
    by[d] = fy >= 0 && fy < nf;
    bz[d] = fz >= 0 && fz < nf;
    ix[d] = min(max(fx, 0), nf - 1);
    iy[d] = min(max(fy, 0), nf - 1) * nf;
    iz[d] = min(max(fz, 0), nf - 1) * nf * nf;
  }
  c32 acc = make_float2(0.f, 0.f);
#pragma unroll
  for (int dz = DIM == 3 ? 0 : 1; dz <= (DIM == 3 ? 2 : 1); ++dz) {
    c32 v[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = s[(DIM == 3 ? iz[dz] : 0) + iy[k / 3] + ix[k % 3]];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const bool in = bx[k % 3] && by[k / 3] && (DIM == 2 || bz[dz]);
      const float wgt = w1[k % 3] * w1[k / 3] * (DIM == 3 ? w1[dz] : 1.0f);
      acc.x = fmaf(in ? v[k].x : 0.f, wgt, acc.x);
      acc.y = fmaf(in ? v[k].y : 0.f, wgt, acc.y);
    }
  }
  return cscale(acc, 4.0f);
}

// (P e)(f): bilinear / trilinear prolongation from the coarse grid (nc points per side)
template <int DIM>
__device__ __forceinline__ c32 prolong_at(const c32* e, const Coord& f, int nc) {
  const int ox = f.x & 1, oy = f.y & 1, oz = DIM == 3 ? f.z & 1 : 0;
  const float wx = ox ? 0.5f : 1.f, wy = oy ? 0.5f : 1.f, wz = oz ? 0.5f : 1.f, w = wx * wy * wz;
  const int base = ((DIM == 3 ? (f.z >> 1) * nc : 0) + (f.y >> 1)) * nc + (f.x >> 1);
  c32 v[1 << DIM];
#pragma unroll
  for (int k = 0; k < (1 << DIM); ++k)
    v[k] = e[base + (k & 1) * ox + (k >> 1 & 1) * oy * nc + (DIM == 3 ? (k >> 2) * oz * nc * nc : 0)];
  c32 acc = make_float2(0.f, 0.f);
#pragma unroll
  for (int k = 0; k < (1 << DIM); ++k) {  // a second point along an even axis counts 0
    const bool in = (!(k & 1) || ox) && (!(k >> 1 & 1) || oy) && (!(k >> 2) || oz);
    acc.x = fmaf(in ? v[k].x : 0.f, w, acc.x);
    acc.y = fmaf(in ? v[k].y : 0.f, w, acc.y);
  }
  return acc;
}

template <int DIM>
__global__ __launch_bounds__(CC_NT) void k_coarse_cycle(CoarseCycleArgs a) {
  __shared__ c32 red[CC_NT];
  const int b = blockIdx.x;
  if (a.active && !a.active[b]) return;
  const float om = a.omega;
  // ---- down ----
  for (int l = a.lp; l < a.L - 1; ++l) {
    const CoarseLevel& F = a.lv[l];
    const CoarseLevel& C = a.lv[l + 1];
    const c32* r = F.rc + (long long)b * F.N;
    c32* e = F.e + (long long)b * F.N;
    c32* t = F.t + (long long)b * F.N;
    for (int p = threadIdx.x; p < F.N; p += CC_NT) e[p] = cmul(F.wd[p], r[p]);
    __syncthreads();
    for (int p = threadIdx.x; p < F.N; p += CC_NT) {
      const Coord c = coord_of32((unsigned)p, (unsigned)F.n, DIM);
      t[p] = cadd(cscale(r[p], 1.0f - om), neighbours<DIM>(e, p, c, F.n));
    }
    __syncthreads();
    c32* rcn = C.rc + (long long)b * C.N;
    for (int q = threadIdx.x; q < C.N; q += CC_NT) {
      const Coord cq = coord_of32((unsigned)q, (unsigned)C.n, DIM);
      rcn[q] = fw4<DIM>(t, cq, F.n);
    }
    __syncthreads();
  }
  // ---- coarsest: e = M r, rows split over thread groups, partial sums reduced in LDS ----
  {
    const CoarseLevel& Q = a.lv[a.L - 1];
    const int Nc = (int)Q.N;
    const c32* r = Q.rc + (long long)b * Nc;
    c32* e = Q.e + (long long)b * Nc;
    const int groups = max(1, CC_NT / max(Nc, 1));  // k-split factor when Nc < CC_NT
    for (int row0 = 0; row0 < Nc; row0 += CC_NT / groups) {
      const int rows = min(CC_NT / groups, Nc - row0);
      const int g = threadIdx.x / (CC_NT / groups), rr = threadIdx.x % (CC_NT / groups);
      c32 acc = make_float2(0.f, 0.f);
      if (g < groups && rr < rows) {
        for (int k = g; k < Nc; k += groups) acc = cfma(a.minvT[(long long)k * Nc + row0 + rr], r[k], acc);
      }
      red[threadIdx.x] = acc;
      __syncthreads();
      if (threadIdx.x < rows) {
        c32 s2 = make_float2(0.f, 0.f);
        for (int q = 0; q < groups; ++q) s2 = cadd(s2, red[q * (CC_NT / groups) + threadIdx.x]);
        e[row0 + threadIdx.x] = s2;
      }
      __syncthreads();
    }
  }
  // ---- up ----
  for (int l = a.L - 2; l >= a.lp; --l) {
    const CoarseLevel& F = a.lv[l];
    const CoarseLevel& C = a.lv[l + 1];
    const c32* r = F.rc + (long long)b * F.N;
    c32* e = F.e + (long long)b * F.N;
    c32* t = F.t + (long long)b * F.N;
    const c32* ec = C.e + (long long)b * C.N;
    for (int p = threadIdx.x; p < F.N; p += CC_NT) {
      const Coord c = coord_of32((unsigned)p, (unsigned)F.n, DIM);
      t[p] = cadd(e[p], prolong_at<DIM>(ec, c, C.n));
    }
    __syncthreads();
    for (int p = threadIdx.x; p < F.N; p += CC_NT) {
      const Coord c = coord_of32((unsigned)p, (unsigned)F.n, DIM);
      e[p] = cadd(cscale(t[p], 1.0f - om), cmul(F.wd[p], cadd(r[p], neighbours<DIM>(t, p, c, F.n))));
    }
    __syncthreads();
  }
}

// The same cycle with every level's right-hand side, solution and scratch in
// LDS (dynamic shared memory, laid out level after level, then CC_NT
// reduction slots): the input right-hand side is read once and the solution
// written once; every other access of the cycle stays on the CU.  Used when
// the levels fit (see coarse_cycle_lds_bytes).
// Offset in the LDS layout of level l's block (r, e, t; r, e on the coarsest;
// the reduction slots after the coarsest).  Uniform scalar arithmetic: the
// per-level pointers are formed where used instead of living in a
// dynamically indexed (scratch) array.
__device__ __forceinline__ int lds_base(const CoarseCycleArgs& a, int l) {
  int o = 0;
  for (int q = a.lp; q < l; ++q) o += (q < a.L - 1 ? 3 : 2) * (int)a.lv[q].N;
  return o;
}

template <int DIM>
__global__ __launch_bounds__(CC_NT) void k_coarse_cycle_lds(CoarseCycleArgs a) {
  extern __shared__ c32 lds[];
  const int b = blockIdx.x;
  if (a.active && !a.active[b]) return;
  const float om = a.omega;
  auto R = [&](int l) { return lds + lds_base(a, l); };
  auto E = [&](int l) { return lds + lds_base(a, l) + (int)a.lv[l].N; };
  auto T = [&](int l) { return l < a.L - 1 ? lds + lds_base(a, l) + 2 * (int)a.lv[l].N : lds + lds_base(a, a.L); };
  // The coarsest solve's entries of this thread, loaded now when they fit in
  // registers (one pass of rows, at most MK per thread), so that the solve
  // waits on no global load.
  constexpr int MK = 10;
  const int Ncst = (int)a.lv[a.L - 1].N;
  const int groups = max(1, CC_NT / max(Ncst, 1));
  const bool pre = Ncst <= CC_NT && (Ncst + groups - 1) / groups <= MK;
  c32 mk[MK];
  if (pre) {
    const int g = threadIdx.x / (CC_NT / groups), rr = threadIdx.x % (CC_NT / groups);
    const bool mine = g < groups && rr < Ncst;
#pragma unroll
    for (int u = 0; u < MK; ++u) {
      const int k = g + u * groups;
      mk[u] = mine && k < Ncst ? a.minvT[(long long)k * Ncst + rr] : make_float2(0.f, 0.f);
    }
  }
  {
    const CoarseLevel& F = a.lv[a.lp];
    const c32* rg = F.rc + (long long)b * F.N;
    for (int p = threadIdx.x; p < F.N; p += CC_NT) R(a.lp)[p] = rg[p];
  }
  __syncthreads();
  // ---- down ----
  for (int l = a.lp; l < a.L - 1; ++l) {
    const CoarseLevel& F = a.lv[l];
    const CoarseLevel& C = a.lv[l + 1];
    const int Nf = (int)F.N, Ncl = (int)C.N;
    c32 *r = R(l), *e = E(l), *t = T(l);
    for (int p = threadIdx.x; p < Nf; p += CC_NT) e[p] = cmul(F.wd[p], r[p]);
    __syncthreads();
    for (int p = threadIdx.x; p < Nf; p += CC_NT) {
      const Coord c = coord_of32((unsigned)p, (unsigned)F.n, DIM);
      t[p] = cadd(cscale(r[p], 1.0f - om), neighbours<DIM>(e, p, c, F.n));
    }
    __syncthreads();
    for (int q = threadIdx.x; q < Ncl; q += CC_NT) {
      const Coord cq = coord_of32((unsigned)q, (unsigned)C.n, DIM);
      R(l + 1)[q] = fw4<DIM>(t, cq, F.n);
    }
    __syncthreads();
  }
  // ---- coarsest: e = M r, rows split over thread groups, partial sums reduced in LDS ----
  {
    const int Nc = Ncst;
    const c32* r = R(a.L - 1);
    c32* e = E(a.L - 1);
    c32* red = T(a.L - 1);
    for (int row0 = 0; row0 < Nc; row0 += CC_NT / groups) {
      const int rows = min(CC_NT / groups, Nc - row0);
      const int g = threadIdx.x / (CC_NT / groups), rr = threadIdx.x % (CC_NT / groups);
      c32 acc = make_float2(0.f, 0.f);
      if (g < groups && rr < rows) {
        if (pre) {
#pragma unroll
          for (int u = 0; u < MK; ++u) {
            const int k = g + u * groups;
            if (k < Nc) acc = cfma(mk[u], r[k], acc);
          }
        } else {
          for (int k = g; k < Nc; k += groups) acc = cfma(a.minvT[(long long)k * Nc + row0 + rr], r[k], acc);
        }
      }
      red[threadIdx.x] = acc;
      __syncthreads();
      if (threadIdx.x < rows) {
        c32 s2 = make_float2(0.f, 0.f);
        for (int q = 0; q < groups; ++q) s2 = cadd(s2, red[q * (CC_NT / groups) + threadIdx.x]);
        e[row0 + threadIdx.x] = s2;
      }
      __syncthreads();
    }
    if (a.lp == a.L - 1) {  // the coarsest level alone
      c32* eg = a.lv[a.lp].e + (long long)b * Nc;
      for (int p = threadIdx.x; p < Nc; p += CC_NT) eg[p] = e[p];
    }
  }
  // ---- up ----
  for (int l = a.L - 2; l >= a.lp; --l) {
    const CoarseLevel& F = a.lv[l];
    const CoarseLevel& C = a.lv[l + 1];
    const int Nf = (int)F.N;
    c32 *r = R(l), *e = E(l), *t = T(l);
    const c32* ec = E(l + 1);
    for (int p = threadIdx.x; p < Nf; p += CC_NT) {
      const Coord c = coord_of32((unsigned)p, (unsigned)F.n, DIM);
      t[p] = cadd(e[p], prolong_at<DIM>(ec, c, C.n));
    }
    __syncthreads();
    if (l == a.lp) {
      c32* eg = F.e + (long long)b * F.N;
      for (int p = threadIdx.x; p < Nf; p += CC_NT) {
        const Coord c = coord_of32((unsigned)p, (unsigned)F.n, DIM);
        eg[p] = cadd(cscale(t[p], 1.0f - om), cmul(F.wd[p], cadd(r[p], neighbours<DIM>(t, p, c, F.n))));
      }
    } else {
      for (int p = threadIdx.x; p < Nf; p += CC_NT) {
        const Coord c = coord_of32((unsigned)p, (unsigned)F.n, DIM);
        e[p] = cadd(cscale(t[p], 1.0f - om), cmul(F.wd[p], cadd(r[p], neighbours<DIM>(t, p, c, F.n))));
      }
      __syncthreads();
    }
  }
}

// ---- the same cycle in two launches, for coarsest grids whose product is the long part ----
// One workgroup per right-hand side reads the whole inverse (8 Nc^2 bytes: 1.3 MB at 20^2)
// through one CU, 26-40 us of the 37-53 us the single launch takes.  Here 32 or 64 rows of
// the product belong to one workgroup: the workgroups of a right-hand side each repeat the
// down part (a few points per thread, in LDS) and form their rows, with their slice of the
// inverse loaded into registers before the down part, so that it is there when the coarsest
// right-hand side is.  The up part is a second launch (it needs every row).  32 rows while
// those workgroups are at most one per CU, else 64, which repeats the down part less (down
// launch at 20^2 x 32: 11.6 us with 32 rows, 9.3 with 64).  Whole solves at 1e-7, single
// launch against two: 128^2 x 1 (22^2 coarsest) 18.9 -> 11.2 ms, 203^2 x 7 FGMRES (17^2) 43.0
// -> 32.9, a gradient at 256^2 x 32 (20^2) 159 -> 99, 64^3 x 8 (8^3, whose vectors did not fit
// the single launch's LDS) 91.8 -> 64.6.
constexpr int CD_MAXN = 640, CD_MP = 4;

// MK: entries of a row per thread, ceil(Nc CD_ROWS / CC_NT) or more
template <int DIM, int CD_ROWS, int MK>
__global__ __launch_bounds__(CC_NT) void k_coarse_down_rows(int B, CoarseCycleArgs a) {
  constexpr int HALF = CD_ROWS / 32;  // columns per thread and pass: 1, or 2 with 64 rows
  extern __shared__ c32 lds[];
  const int b = batch_index();
  if (b >= B || (a.active && !a.active[b])) return;
  const float om = a.omega;
  const int tid = threadIdx.x, Nc = (int)a.lv[a.L - 1].N, row0 = blockIdx.x * CD_ROWS;
  const int rr = tid % CD_ROWS, row = row0 + rr;
  c32* se = lds;                      // W r of the current level; at the end the coarsest right-hand side
  c32* st = lds + (int)a.lv[a.lp].N;  // its residual
  c32 r[CD_MP], w[CD_MP];
  {
    const CoarseLevel& F = a.lv[a.lp];
    const c32* rg = F.rc + (long long)b * F.N;
#pragma unroll
    for (int i = 0; i < CD_MP; ++i) {
      const int p = min(tid + i * CC_NT, (int)F.N - 1);
      r[i] = rg[p];
      w[i] = F.wd[p];
    }
  }
  // this thread's entries of the inverse: row `row`, columns g + 32 u (g the column group; with
  // 64 rows the two groups that two threads of a wavefront hold with 32, so that the sums are
  // the same); issued after the loads above, which the first stage waits for, and used last
  c32 mk[MK];
  const int g = tid / CD_ROWS * HALF;
  auto column = [&](int u) { return g + u % HALF + u / HALF * 32; };
#pragma unroll
  for (int u = 0; u < MK; ++u) mk[u] = a.minvT[(long long)min(column(u), Nc - 1) * Nc + min(row, Nc - 1)];
  __builtin_amdgcn_sched_barrier(0);
  for (int l = a.lp; l < a.L - 1; ++l) {
    const CoarseLevel& F = a.lv[l];
    const CoarseLevel& C = a.lv[l + 1];
    const int Nf = (int)F.N, Nn = (int)C.N, n = F.n;
#pragma unroll
    for (int i = 0; i < CD_MP; ++i)
      if (tid + i * CC_NT < Nf) se[tid + i * CC_NT] = cmul(w[i], r[i]);
    const bool last = l + 1 == a.L - 1;
    if (!last) {
#pragma unroll
      for (int i = 0; i < CD_MP; ++i) w[i] = C.wd[min(tid + i * CC_NT, Nn - 1)];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CD_MP; ++i) {
      const int p = tid + i * CC_NT;
      if (p < Nf) st[p] = cadd(cscale(r[i], 1.0f - om), neighbours<DIM>(se, p, coord_of32((unsigned)p, (unsigned)n, DIM), n));
    }
    __syncthreads();
    c32* rcg = C.rc + (long long)b * C.N;
#pragma unroll
    for (int i = 0; i < CD_MP; ++i) {
      const int q = tid + i * CC_NT;
      if (q < Nn) {
        r[i] = fw4<DIM>(st, coord_of32((unsigned)q, (unsigned)C.n, DIM), n);
        if (last) se[q] = r[i];
        else if (blockIdx.x == 0) rcg[q] = r[i];  // the up part's
      }
    }
    // the next level's first stage writes se (last read before the barrier above)
  }
  __syncthreads();
  c32 part[HALF];
#pragma unroll
  for (int q = 0; q < HALF; ++q) part[q] = make_float2(0.f, 0.f);
#pragma unroll
  for (int u = 0; u < MK; ++u)
    if (column(u) < Nc) part[u % HALF] = cfma(mk[u], se[column(u)], part[u % HALF]);
  // a wavefront holds two column groups; then 16 partial sums per row
  c32 acc = part[0];
  if (HALF == 2) acc = cadd(acc, part[HALF - 1]);
  else acc = cadd(acc, make_float2(__shfl_xor(acc.x, 32, HELM_WAVE), __shfl_xor(acc.y, 32, HELM_WAVE)));
  c32* red = st;  // free since the barrier above
  if (tid % HELM_WAVE < CD_ROWS) red[(tid / HELM_WAVE) * CD_ROWS + rr] = acc;
  __syncthreads();
  if (tid < CD_ROWS && row < Nc) {
    c32 s2 = make_float2(0.f, 0.f);
#pragma unroll
    for (int q = 0; q < CC_NT / HELM_WAVE; ++q) s2 = cadd(s2, red[q * CD_ROWS + tid]);
    a.lv[a.L - 1].e[(long long)b * Nc + row] = s2;
  }
}

template <int DIM>
__global__ __launch_bounds__(CC_NT) void k_coarse_up_rows(CoarseCycleArgs a) {
  extern __shared__ c32 lds[];
  const int b = blockIdx.x;
  if (a.active && !a.active[b]) return;
  const float om = a.omega;
  const int tid = threadIdx.x;
  c32* st = lds;                      // e + P e_coarse of the current level
  c32* se = lds + (int)a.lv[a.lp].N;  // the solution of the level below
  c32 r[CD_MP], w[CD_MP];
  auto fetch = [&](int l) {
    const CoarseLevel& F = a.lv[l];
    const c32* rg = F.rc + (long long)b * F.N;
#pragma unroll
    for (int i = 0; i < CD_MP; ++i) {
      const int p = min(tid + i * CC_NT, (int)F.N - 1);
      r[i] = rg[p];
      w[i] = F.wd[p];
    }
  };
  fetch(a.L - 2);
  {
    const CoarseLevel& Q = a.lv[a.L - 1];
    const c32* eg = Q.e + (long long)b * Q.N;
    for (int p = tid; p < Q.N; p += CC_NT) se[p] = eg[p];
  }
  __syncthreads();
  for (int l = a.L - 2; l >= a.lp; --l) {
    const CoarseLevel& F = a.lv[l];
    const int Nf = (int)F.N, n = F.n, nc = a.lv[l + 1].n;
    c32 tv[CD_MP];
#pragma unroll
    for (int i = 0; i < CD_MP; ++i) {
      const int p = tid + i * CC_NT;
      if (p < Nf) {
        tv[i] = cadd(cmul(w[i], r[i]), prolong_at<DIM>(se, coord_of32((unsigned)p, (unsigned)n, DIM), nc));
        st[p] = tv[i];
      }
    }
    __syncthreads();
    c32* eg = F.e + (long long)b * F.N;
#pragma unroll
    for (int i = 0; i < CD_MP; ++i) {
      const int p = tid + i * CC_NT;
      if (p < Nf) {
        const c32 nb = neighbours<DIM>(st, p, coord_of32((unsigned)p, (unsigned)n, DIM), n);
        const c32 v = cadd(cscale(tv[i], 1.0f - om), cmul(w[i], cadd(r[i], nb)));
        if (l == a.lp) eg[p] = v;
        else se[p] = v;
      }
    }
    if (l > a.lp) {
      fetch(l - 1);
      __syncthreads();
    }
  }
}

}  // namespace

// LDS bytes k_coarse_cycle_lds needs for levels lp .. L-1 (r, e, t per level,
// r, e on the coarsest, CC_NT reduction slots)
size_t coarse_cycle_lds_bytes(const CoarseCycleArgs& a) {
  size_t n = CC_NT;
  for (int l = a.lp; l < a.L; ++l) n += (size_t)(l < a.L - 1 ? 3 : 2) * (size_t)a.lv[l].N;
  return n * sizeof(c32);
}

// Two launches where the coarsest product outweighs a launch (Nc > 128) and the entries fit
// the threads' registers; one launch below (37^2 / 10^2 x 60: 14.3 us in one).
bool coarse_cycle_split(const CoarseCycleArgs& a) {
  const long long Nc = a.lv[a.L - 1].N, Nf = a.lv[a.lp].N;
  return a.lp < a.L - 1 && Nc > 128 && Nc <= CD_MAXN && Nf <= CC_NT * CD_MP;
}

namespace {
template <int DIM, int ROWS, int M0, int M1, int M2, int M3>
void coarse_down_rows(hipStream_t s, int B, size_t lds, int Nc, const CoarseCycleArgs& a) {
  const dim3 grid = batch_grid((Nc + ROWS - 1) / ROWS, B);
  const int mk = (Nc * ROWS + CC_NT - 1) / CC_NT;
  if (mk <= M0) hipLaunchKernelGGL((k_coarse_down_rows<DIM, ROWS, M0>), grid, dim3(CC_NT), lds, s, B, a);
  else if (mk <= M1) hipLaunchKernelGGL((k_coarse_down_rows<DIM, ROWS, M1>), grid, dim3(CC_NT), lds, s, B, a);
  else if (mk <= M2) hipLaunchKernelGGL((k_coarse_down_rows<DIM, ROWS, M2>), grid, dim3(CC_NT), lds, s, B, a);
  else hipLaunchKernelGGL((k_coarse_down_rows<DIM, ROWS, M3>), grid, dim3(CC_NT), lds, s, B, a);
}
template <int DIM>
void coarse_down(hipStream_t s, int B, size_t lds, int Nc, const CoarseCycleArgs& a) {
  if ((long long)B * ((Nc + 31) / 32) <= 256) coarse_down_rows<DIM, 32, 8, 13, 16, 20>(s, B, lds, Nc, a);
  else coarse_down_rows<DIM, 64, 16, 26, 32, 40>(s, B, lds, Nc, a);
}
}  // namespace

void launch_coarse_cycle(hipStream_t s, int B, const CoarseCycleArgs& a) {
  if (coarse_cycle_split(a)) {
    const int Nc = (int)a.lv[a.L - 1].N, Nf = (int)a.lv[a.lp].N;
    // down: two vectors of the finest level (the second at least the 16 partial sums per row);
    // up: one, and one of the level below
    const size_t down = (size_t)(Nf + std::max(Nf, CC_NT)) * sizeof(c32);
    const size_t up = (size_t)(Nf + a.lv[a.lp + 1].N) * sizeof(c32);
    if (a.dim == 2) coarse_down<2>(s, B, down, Nc, a);
    else coarse_down<3>(s, B, down, Nc, a);
    if (a.dim == 2) hipLaunchKernelGGL(k_coarse_up_rows<2>, dim3(B), dim3(CC_NT), up, s, a);
    else hipLaunchKernelGGL(k_coarse_up_rows<3>, dim3(B), dim3(CC_NT), up, s, a);
    return;
  }
  const size_t lds = coarse_cycle_lds_bytes(a);
  const bool in_lds = lds <= kCoarseCycleMaxLds;
  if (a.dim == 2) {
    if (in_lds) hipLaunchKernelGGL(k_coarse_cycle_lds<2>, dim3(B), dim3(CC_NT), lds, s, a);
    else hipLaunchKernelGGL(k_coarse_cycle<2>, dim3(B), dim3(CC_NT), 0, s, a);
  } else {
    if (in_lds) hipLaunchKernelGGL(k_coarse_cycle_lds<3>, dim3(B), dim3(CC_NT), lds, s, a);
    else hipLaunchKernelGGL(k_coarse_cycle<3>, dim3(B), dim3(CC_NT), 0, s, a);
  }
}
