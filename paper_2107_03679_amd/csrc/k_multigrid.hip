// Multigrid kernels for the shifted operator K'_l = -Lap'_l - kappa c_l
// (h_l^2-scaled, Sec. IV-B/IV-C):
//  * fused 2D legs of a V-cycle started from a zero guess with one pre- and
//    one post-relaxation (the paper's nu1 = nu2 = 1, omega_S = 0.8):
//      down: v1 = w D^-1 r;  rc = 4 R (r - K v1)          (LDS tile, 2-cell halo)
//      up:   v2 = w D^-1 r + P e;  z = v2 + w D^-1 (r - K v2)
//    v1 is recomputed by the up-leg instead of being stored.
//  * generic kernels (any dimension, any nu, W-cycles): Jacobi sweeps
//    (eq. dampedJ), residual + full-weighting restriction, prolongation.
//  * the exact coarsest solve as a product with the explicit inverse.
// D = diag(K) includes the Sommerfeld ghost terms: D = 2d - coef - g * #ghosts.
#include "dev_common.h"
#include "kernels.h"
#include "march3.h"

namespace {


// ------------------------------------------------------------ fused 2D legs
// Down-leg on a TCX x TCY tile of coarse points (fine footprint 2 TCX + 1 wide):
//   stage 1: r and v1 = W r on the (2 TCX + 3) x (2 TCY + 3) halo region, v1 -> LDS
//   stage 2: s = r - K v1 = (1 - w) r + sum of in-grid neighbours of v1 (D v1 = w r)
//            on the (2 TCX + 1) x (2 TCY + 1) interior, by the thread that holds r
//   stage 3: rc = 4 R s (scaled coarse right-hand side)
// With RES the leg starts a repeated visit of the level from the current
// solution e (Alg. 2 with a non-zero guess, written as e + MG(r - K e, 0)):
// its right-hand side is r - K e, formed on the halo region from e on a
// one-point wider ring, so that the residual is never stored.
template <int TCX, int TCY, bool RES>
__global__ __launch_bounds__(TCX* TCY) void k_down_fused2(int nrhs, VecSet r, ScaleSet rs, LevelArgs lv,
                                                           float omega, VecSet rc, int nc, const int* active,
                                                           VecSet ev) {
  constexpr int RX = 2 * TCX + 3, RY = 2 * TCY + 3;
  constexpr int SX = 2 * TCX + 1, SY = 2 * TCY + 1;
  constexpr int NT = TCX * TCY, NR = RX * RY, IT = (NR + NT - 1) / NT;
  constexpr int EX = RES ? RX + 2 : 1, EY = RES ? RY + 2 : 1;
  __shared__ c32 sV[RY][RX];
  __shared__ c32 sS[SY][SX];
  __shared__ c32 sE[EY][EX];
  const int n = lv.n;
  const int tiles_x = (nc + TCX - 1) / TCX;
  const unsigned tiles = (unsigned)(tiles_x * ((nc + TCY - 1) / TCY));
  const TileId id = xcd_tile(blockIdx.x, nrhs, tiles, HELM_RHS_GROUP);
  const int b = id.b;
  if (active && !active[b]) return;
  const int cx0 = (id.t % tiles_x) * TCX;
  const int cy0 = (id.t / tiles_x) * TCY;
  const int fx0 = 2 * cx0 - 2, fy0 = 2 * cy0 - 2;
  const float sc = scale_of(rs, b);
  const c32* rb = r.p + (long long)b * r.stride;
  c32 rv[IT], wv[IT], kv[RES ? IT : 1];
  if constexpr (RES) {
    const c32* eb = ev.p + (long long)b * ev.stride;
    for (int idx = threadIdx.x; idx < EX * EY; idx += NT) {
      const int gx = fx0 - 1 + idx % EX, gy = fy0 - 1 + idx / EX;
      const bool ok = gx >= 0 && gx < n && gy >= 0 && gy < n;
      sE[idx / EX][idx % EX] = ok ? eb[(long long)gy * n + gx] : make_float2(0.f, 0.f);
    }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int idx = threadIdx.x + it * NT;
    const int gx = fx0 + idx % RX, gy = fy0 + idx / RX;
    const bool ok = idx < NR && gx >= 0 && gx < n && gy >= 0 && gy < n;
    const long long p = ok ? (long long)gy * n + gx : 0;
    rv[it] = ok ? rb[p] : make_float2(0.f, 0.f);
    wv[it] = ok ? lv.wd[p] : make_float2(0.f, 0.f);
    if constexpr (RES) kv[it] = ok ? lv.coef[p] : make_float2(0.f, 0.f);
  }
  if constexpr (RES) __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int idx = threadIdx.x + it * NT;
    rv[it] = cscale(rv[it], sc);
    if constexpr (RES) {
      // r - K e with K e = D e - (sum of in-grid neighbours); sE is zero outside the grid
      const int lx = idx % RX + 1, ly = idx / RX + 1;
      const int gx = fx0 + idx % RX, gy = fy0 + idx / RX;
      if (idx < NR && gx >= 0 && gx < n && gy >= 0 && gy < n) {
        const int ng = ghosts2(gx, gy, n);
        const c32 D = make_float2(4.0f - kv[it].x - ng * lv.ghost.x, -kv[it].y - ng * lv.ghost.y);
        const c32 nb = cadd(cadd(sE[ly][lx - 1], sE[ly][lx + 1]), cadd(sE[ly - 1][lx], sE[ly + 1][lx]));
        rv[it] = cadd(csub(rv[it], cmul(D, sE[ly][lx])), nb);
      }
    }
    if (idx < NR) sV[idx / RX][idx % RX] = cmul(rv[it], wv[it]);
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int idx = threadIdx.x + it * NT;
    const int lx = idx % RX, ly = idx / RX;
    if (idx >= NR || lx == 0 || lx == RX - 1 || ly == 0 || ly == RY - 1) continue;
    const int gx = fx0 + lx, gy = fy0 + ly;
    c32 s = make_float2(0.f, 0.f);
    if (gx >= 0 && gx < n && gy >= 0 && gy < n) {
      const c32 nb = cadd(cadd(sV[ly][lx - 1], sV[ly][lx + 1]), cadd(sV[ly - 1][lx], sV[ly + 1][lx]));
      s = cadd(cscale(rv[it], 1.0f - omega), nb);
    }
    sS[ly - 1][lx - 1] = s;
  }
  __syncthreads();
  const int tx = threadIdx.x % TCX, ty = threadIdx.x / TCX;
  const int I = cx0 + tx, J = cy0 + ty;
  if (I < nc && J < nc) {
    const int sx = 2 * tx + 1, sy = 2 * ty + 1;
    c32 acc = cscale(sS[sy][sx], 4.0f);
    acc = cadd(acc, cscale(cadd(cadd(sS[sy][sx - 1], sS[sy][sx + 1]), cadd(sS[sy - 1][sx], sS[sy + 1][sx])), 2.0f));
    acc = cadd(acc, cadd(cadd(sS[sy - 1][sx - 1], sS[sy - 1][sx + 1]), cadd(sS[sy + 1][sx - 1], sS[sy + 1][sx + 1])));
    // scaled coarse right-hand side: 4 * (1/16) * stencil sum
    rc.p[(long long)b * rc.stride + (long long)J * nc + I] = cscale(acc, 0.25f);
  }
}

// bilinear prolongation at fine point (gx, gy) from the LDS coarse tile whose
// origin is coarse point (cxs, cys) (printed formula of Sec. IV-C)
template <int CX>
__device__ __forceinline__ c32 prolong_lds(const c32 (*sE)[CX], int gx, int gy, int cxs, int cys) {
  const int I = (gx >> 1) - cxs, J = (gy >> 1) - cys;
  const int ox = gx & 1, oy = gy & 1;
  c32 pe = sE[J][I];
  if (ox && oy) return cscale(cadd(cadd(pe, sE[J][I + 1]), cadd(sE[J + 1][I], sE[J + 1][I + 1])), 0.25f);
  if (ox) return cscale(cadd(pe, sE[J][I + 1]), 0.5f);
  if (oy) return cscale(cadd(pe, sE[J + 1][I]), 0.5f);
  return pe;
}

// Up-leg on a TX x TY tile of fine points; thread (tx, ty0..ty0+PY) owns a
// column segment and keeps r and W of its own points in registers:
//   v2 = W r + P e on the (TX + 2) x (TY + 2) halo region (own points + a ring) -> LDS
//   z  = v2 + W (r - K v2) = (1 - w) v2 + W (r + sum of in-grid neighbours of v2)
// With RES (see k_down_fused2) the right-hand side is r - K e, formed from e
// on a two-point ring, and the leg writes e + z: the result of the repeated
// visit.  z must not alias e (other tiles read e's halo).
template <int TX, int TY, int PY, bool RES>
__global__ __launch_bounds__(TX*(TY / PY)) void k_up_fused2(int nrhs, VecSet r, ScaleSet rs, LevelArgs lv,
                                                             float omega, VecSet ec, int nc, VecSet z,
                                                             const int* active, VecSet ev) {
  constexpr int HX = TX + 2, HY = TY + 2;
  constexpr int CX = TX / 2 + 2, CY = TY / 2 + 2;
  constexpr int NT = TX * (TY / PY);
  constexpr int NRING = 2 * HX + 2 * TY;
  constexpr int FX = RES ? TX + 4 : 1, FY = RES ? TY + 4 : 1;
  static_assert(NRING <= NT, "one ring point per thread");
  __shared__ c32 sE[CY][CX];
  __shared__ c32 sV[HY][HX];
  __shared__ c32 sF[FY][FX];
  const int n = lv.n;
  const int tiles_x = (n + TX - 1) / TX;
  const unsigned tiles = (unsigned)(tiles_x * ((n + TY - 1) / TY));
  const TileId id = xcd_tile(blockIdx.x, nrhs, tiles, HELM_RHS_GROUP);
  const int b = id.b;
  if (active && !active[b]) return;
  const int fx0 = (id.t % tiles_x) * TX;
  const int fy0 = (id.t / tiles_x) * TY;
  const int cxs = fx0 / 2 - 1, cys = fy0 / 2 - 1;
  const c32* eb = ec.p + (long long)b * ec.stride;
  const float sc = scale_of(rs, b);
  const c32* rb = r.p + (long long)b * r.stride;
  const int tx = threadIdx.x % TX, ty0 = (threadIdx.x / TX) * PY;
  // ring point of this thread (halo-local coordinates), if any
  int rlx = -1, rly = -1;
  {
    const int t = threadIdx.x;
    if (t < HX) {
      rlx = t;
      rly = 0;
    } else if (t < 2 * HX) {
      rlx = t - HX;
      rly = HY - 1;
    } else if (t < 2 * HX + TY) {
      rlx = 0;
      rly = t - 2 * HX + 1;
    } else if (t < NRING) {
      rlx = HX - 1;
      rly = t - 2 * HX - TY + 1;
    }
  }
  // issue every global load first, back to back: clamped in-grid addresses without
  // predicates, so that none waits for another; zeros outside the grid are put in at the
  // LDS stores, and values of points outside the grid are never used (every use below is
  // guarded by the same condition); the scale of r is applied after the loads
  constexpr int NE = CX * CY, ITE = (NE + NT - 1) / NT, ITF = RES ? (FX * FY + NT - 1) / NT : 0;
  c32 ev_c[ITE], fv[ITF > 0 ? ITF : 1], rv[PY + 1], wv[PY + 1];
#pragma unroll
  for (int it = 0; it < ITE; ++it) {
    const int idx = min((int)threadIdx.x + it * NT, NE - 1);
    const int I = min(max(cxs + idx % CX, 0), nc - 1), J = min(max(cys + idx / CX, 0), nc - 1);
    ev_c[it] = eb[(long long)J * nc + I];
  }
  c32 kv[RES ? PY + 1 : 1];
  if constexpr (RES) {
    const c32* fb = ev.p + (long long)b * ev.stride;
#pragma unroll
    for (int it = 0; it < ITF; ++it) {
      const int idx = min((int)threadIdx.x + it * NT, FX * FY - 1);
      const int gx = min(max(fx0 - 2 + idx % FX, 0), n - 1), gy = min(max(fy0 - 2 + idx / FX, 0), n - 1);
      fv[it] = fb[(long long)gy * n + gx];
    }
  }
#pragma unroll
  for (int k = 0; k <= PY; ++k) {
    const int gx = min(max(k < PY ? fx0 + tx : fx0 - 1 + rlx, 0), n - 1);
    const int gy = min(max(k < PY ? fy0 + ty0 + k : fy0 - 1 + rly, 0), n - 1);
    const long long p = (long long)gy * n + gx;
    rv[k] = rb[p];
    wv[k] = lv.wd[p];
    if constexpr (RES) kv[k] = lv.coef[p];
  }
#pragma unroll
  for (int it = 0; it < ITE; ++it) {
    const int idx = threadIdx.x + it * NT;
    const int I = cxs + idx % CX, J = cys + idx / CX;
    const bool ok = I >= 0 && I < nc && J >= 0 && J < nc;
    if (idx < NE) sE[idx / CX][idx % CX] = ok ? ev_c[it] : make_float2(0.f, 0.f);
  }
  if constexpr (RES) {
#pragma unroll
    for (int it = 0; it < ITF; ++it) {
      const int idx = threadIdx.x + it * NT;
      const int gx = fx0 - 2 + idx % FX, gy = fy0 - 2 + idx / FX;
      const bool ok = gx >= 0 && gx < n && gy >= 0 && gy < n;
      if (idx < FX * FY) sF[idx / FX][idx % FX] = ok ? fv[it] : make_float2(0.f, 0.f);
    }
  }
#pragma unroll
  for (int k = 0; k <= PY; ++k) rv[k] = cscale(rv[k], sc);
  __syncthreads();
  if constexpr (RES) {
    // r - K e at the own and ring points (sF is zero outside the grid)
#pragma unroll
    for (int k = 0; k <= PY; ++k) {
      const int lx = k < PY ? tx + 1 : rlx, ly = k < PY ? ty0 + k + 1 : rly;
      const int gx = fx0 - 1 + lx, gy = fy0 - 1 + ly;
      if ((k < PY || rlx >= 0) && gx >= 0 && gx < n && gy >= 0 && gy < n) {
        const int ng = ghosts2(gx, gy, n);
        const c32 D = make_float2(4.0f - kv[k].x - ng * lv.ghost.x, -kv[k].y - ng * lv.ghost.y);
        const c32 nb = cadd(cadd(sF[ly + 1][lx], sF[ly + 1][lx + 2]), cadd(sF[ly][lx + 1], sF[ly + 2][lx + 1]));
        rv[k] = cadd(csub(rv[k], cmul(D, sF[ly + 1][lx + 1])), nb);
      }
    }
  }
  c32 v2own[PY];
#pragma unroll
  for (int k = 0; k <= PY; ++k) {
    const int lx = k < PY ? tx + 1 : rlx, ly = k < PY ? ty0 + k + 1 : rly;
    if (k == PY && rlx < 0) continue;
    const int gx = fx0 - 1 + lx, gy = fy0 - 1 + ly;
    c32 v2 = make_float2(0.f, 0.f);
    if (gx >= 0 && gx < n && gy >= 0 && gy < n) v2 = cadd(cmul(rv[k], wv[k]), prolong_lds<CX>(sE, gx, gy, cxs, cys));
    if (k < PY) v2own[k] = v2;
    sV[ly][lx] = v2;
  }
  __syncthreads();
  c32* zb = z.p + (long long)b * z.stride;
#pragma unroll
  for (int k = 0; k < PY; ++k) {
    const int lx = tx + 1, ly = ty0 + k + 1;
    const int gx = fx0 + tx, gy = fy0 + ty0 + k;
    if (gx < n && gy < n) {
      const c32 nb = cadd(cadd(sV[ly][lx - 1], sV[ly][lx + 1]), cadd(sV[ly - 1][lx], sV[ly + 1][lx]));
      c32 zv = cadd(cscale(v2own[k], 1.0f - omega), cmul(wv[k], cadd(rv[k], nb)));
      if constexpr (RES) zv = cadd(zv, sF[ly + 1][lx + 1]);
      zb[(long long)gy * n + gx] = zv;
    }
  }
}

// The same fused up-leg and matvec with a wavefront-wide column layout: the
// region is 64 columns wide (a 60-column tile and a two-point ring), each
// thread owns one column (lane) and every fourth row, so that the v2, z and
// output stages are done by the thread that loaded the point's r, W and A
// coefficient (kept in registers, no reloads), and no index needs a division.
// A block walks K right-hand sides of one tile: the coefficient rows (shared by
// the batch) are loaded once, and the next right-hand side's r and coarse tile
// are loaded while the current one is computed, so that the memory system has
// work in every stage.  A wavefront's rows are uniform (its index is read into
// a scalar register), so every row's base address is scalar and all loads and
// stores of a lane share one 32-bit column offset.  Loads go to the nearest
// in-grid point without predicates; values of points outside the grid are
// never used (every use is guarded by the same condition).
template <int TY, int K>
__global__ __launch_bounds__(256) void k_up_mv2w(int nrhs, VecSet r, ScaleSet rs, LevelArgs lv, LevelArgs la,
                                                 float omega, VecSet ec, int nc, VecSet z, VecSet w,
                                                 const int* active) {
  constexpr int TX = 60, VX = 64, VY = TY + 4, ZY = TY + 2, RPI = 4, IV = VY / RPI;
  static_assert(VY % RPI == 0, "whole row groups");
  constexpr int CX = TX / 2 + 3, CY = TY / 2 + 3, IE = (CX * CY + 255) / 256;
  __shared__ c32 sE[CY][CX];
  __shared__ c32 sV[VY][VX];
  __shared__ c32 sZ[ZY][VX];  // z of region point (lx, ly) at sZ[ly - 1][lx]
  const int n = lv.n;
  // workgroup order (xcd_stretch): "groups of K right-hand sides fastest, then tiles in
  // raster order", one contiguous stretch per XCD
  const unsigned groups = (unsigned)(nrhs + K - 1) / K, tiles_x = (unsigned)(n + TX - 1) / TX;
  const unsigned l = xcd_stretch(blockIdx.x, gridDim.x);
  const unsigned t = l / groups, grp = l - t * groups;
  const int b_end = min(nrhs, (int)(grp + 1) * K);
  int b = (int)grp * K;
  if (active)
    while (b < b_end && !active[b]) ++b;
  if (b >= b_end) return;
  const int fx0 = (int)(t % tiles_x) * TX, fy0 = (int)(t / tiles_x) * TY;
  const int cxs = fx0 / 2 - 1, cys = fy0 / 2 - 1;
  const int lx0 = threadIdx.x & 63;
  const int r0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // the wavefront's first region row
  const unsigned ob0 = (unsigned)min(max(fx0 - 2 + lx0, 0), n - 1) * (unsigned)sizeof(c32);  // nearest in-grid column
  unsigned eo[IE];  // coarse-tile items of this thread: nearest in-grid coarse point
#pragma unroll
  for (int it = 0; it < IE; ++it) {
    const int idx = min((int)threadIdx.x + it * 256, CX * CY - 1);
    const int I = min(max(cxs + idx % CX, 0), nc - 1), J = min(max(cys + idx / CX, 0), nc - 1);
    eo[it] = (unsigned)(J * nc + I);
  }
  auto load_e = [&](int bb, c32* ev_) {  // the coarse tile of right-hand side bb
    const c32* eb = ec.p + (long long)bb * ec.stride;
#pragma unroll
    for (int it = 0; it < IE; ++it) ev_[it] = eb[eo[it]];
  };
  auto load_r = [&](int bb, c32* rv_) {  // r of right-hand side bb on the region
    const c32* rb = r.p + (long long)bb * r.stride;
#pragma unroll
    for (int it = 0; it < IV; ++it) {
      const int gy = fy0 - 2 + r0 + RPI * it;
      if (gy >= 0 && gy < n) rv_[it] = at_byte(rb + (long long)gy * n, ob0);
    }
  };
  c32 rv[IV], evc[IE], wv[IV], kv[IV];
  load_e(b, evc);
  load_r(b, rv);
#pragma unroll
  for (int it = 0; it < IV; ++it) {  // the coefficient rows, once for all right-hand sides
    const int ly = r0 + RPI * it, gy = fy0 - 2 + ly;
    if (gy >= 0 && gy < n) {
      const long long row = (long long)gy * n;
      wv[it] = at_byte(lv.wd + row, ob0);
      if (ly >= 2 && ly < TY + 2) kv[it] = at_byte(la.coef + row, ob0);
    }
  }
  while (true) {
    // the lane's geometry, recomputed every pass from an opaque copy of its column (cheaper
    // than the registers the hoisted addresses and predicates would hold across the loop)
    int lx = lx0;
    asm volatile("" : "+v"(lx));
    const int gx = fx0 - 2 + lx;
    const bool inx = gx >= 0 && gx < n;
    const unsigned ob = (unsigned)min(max(gx, 0), n - 1) * (unsigned)sizeof(c32);
    const bool tcol = lx >= 2 && lx < TX + 2 && gx < n;
    int bn = b + 1;  // the next iterating right-hand side of the block
    if (active)
      while (bn < b_end && !active[bn]) ++bn;
#pragma unroll
    for (int it = 0; it < IE; ++it) {
      const int idx = threadIdx.x + it * 256;
      const int I = cxs + idx % CX, J = cys + idx / CX;
      const bool ok = I >= 0 && I < nc && J >= 0 && J < nc;
      if (idx < CX * CY) sE[idx / CX][idx % CX] = ok ? evc[it] : make_float2(0.f, 0.f);
    }
    __syncthreads();
    c32 rn[IV], en[IE];  // the next right-hand side's r and coarse tile, loaded during the stages below
    if constexpr (K > 1)
      if (bn < b_end) {
        load_e(bn, en);
        load_r(bn, rn);
      }
    const float sc = scale_of(rs, b);
#pragma unroll
    for (int it = 0; it < IV; ++it) {  // v2 = W r + P e (zero outside the grid)
      const int ly = r0 + RPI * it, gy = fy0 - 2 + ly;
      c32 v2 = make_float2(0.f, 0.f);
      if (inx && gy >= 0 && gy < n) {
        rv[it] = cscale(rv[it], sc);
        const int I = (gx >> 1) - cxs, J = (gy >> 1) - cys, ox1 = gx & 1, oy = gy & 1;
        const c32 a = sE[J][I], bb = sE[J][I + ox1], c = sE[J + oy][I], d = sE[J + oy][I + ox1];
        v2 = cadd(cmul(rv[it], wv[it]), cscale(cadd(cadd(a, bb), cadd(c, d)), 0.25f));
      }
      sV[ly][lx] = v2;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IV; ++it) {  // z on the tile and a one-point ring (zero outside the grid)
      const int ly = r0 + RPI * it, gy = fy0 - 2 + ly;
      if (ly < 1 || ly > VY - 2) continue;
      if (lx < 1 || lx > VX - 2) continue;
      c32 zv = make_float2(0.f, 0.f);
      if (inx && gy >= 0 && gy < n) {
        const c32 nb = cadd(cadd(sV[ly][lx - 1], sV[ly][lx + 1]), cadd(sV[ly - 1][lx], sV[ly + 1][lx]));
        zv = cadd(cscale(sV[ly][lx], 1.0f - omega), cmul(wv[it], cadd(rv[it], nb)));
      }
      sZ[ly - 1][lx] = zv;
    }
    __syncthreads();
    c32* zb = z.p + (long long)b * z.stride;
    c32* wb = w.p + (long long)b * w.stride;
#pragma unroll
    for (int it = 0; it < IV; ++it) {  // Z_j and W_{j+1} = A Z_j on the tile
      const int ly = r0 + RPI * it, gy = fy0 - 2 + ly;
      if (ly < 2 || ly >= TY + 2 || gy >= n) continue;
      if (!tcol) continue;
      const long long row = (long long)gy * n;
      const c32 zc = sZ[ly - 1][lx];
      const int ng = ghosts2(gx, gy, n);
      const c32 D = make_float2(4.0f - kv[it].x - ng * la.ghost.x, -kv[it].y - ng * la.ghost.y);
      const c32 nb = cadd(cadd(sZ[ly - 1][lx - 1], sZ[ly - 1][lx + 1]), cadd(sZ[ly - 2][lx], sZ[ly][lx]));
      at_byte(zb + row, ob) = zc;
      at_byte(wb + row, ob) = csub(cmul(D, zc), nb);
    }
    if (K == 1 || bn >= b_end) break;
    b = bn;
#pragma unroll
    for (int it = 0; it < IV; ++it) rv[it] = rn[it];
#pragma unroll
    for (int it = 0; it < IE; ++it) evc[it] = en[it];
  }
}

// Column-layout legs (the autotuner's last variants): the fine region is one
// wavefront wide, each thread owns a column (lane) and every fourth row, so
// the stages need no division and reuse the registers of the loads.  Same
// arithmetic per point as k_down_fused2 / k_up_fused2 (bit-identical results).
// Down-leg: 30 x TCY coarse points, fine region 63 x (2 TCY + 3) at 2 c0 - 2.
// With RES the right-hand side is r - K e (a repeated visit, as in k_down_fused2),
// formed from e staged in LDS on the region and a one-point ring.
template <int TCY, bool RES>
__global__ __launch_bounds__(256) void k_down_col(VecSet r, ScaleSet rs, LevelArgs lv, float omega,
                                                  VecSet rc, int nc, const int* active, VecSet ev) {
  constexpr int TCX = 30, RXU = 2 * TCX + 3, RYU = 2 * TCY + 3, RPI = 4, VY = (RYU + RPI - 1) / RPI * RPI,
                IV = VY / RPI;
  constexpr int FX = RES ? RXU + 2 : 1, FY = RES ? RYU + 2 : 1;
  __shared__ c32 sV[VY][64];
  __shared__ c32 sS[VY][64];
  __shared__ c32 sF[FY][FX];
  const int n = lv.n;
  const int b = blockIdx.x;  // grid (right-hand side, tile column, tile row)
  if (active && !active[b]) return;
  const int cx0 = blockIdx.y * TCX, cy0 = blockIdx.z * TCY;
  const int fx0 = 2 * cx0 - 2, fy0 = 2 * cy0 - 2;
  const float sc = scale_of(rs, b);
  const c32* rb = r.p + (long long)b * r.stride;
  const int lx = threadIdx.x & 63;
  const int r0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // the wavefront's first region row
  const int gx = fx0 + lx;
  const bool inx = lx < RXU && gx >= 0 && gx < n;
  const unsigned ob = (unsigned)min(max(gx, 0), n - 1) * (unsigned)sizeof(c32);  // nearest in-grid column, bytes
  // with RES the fine correction, loaded from clamped in-grid addresses back to back with
  // the row loads; zeros outside the grid are put in at the LDS stores
  constexpr int IF = RES ? (FX * FY + 255) / 256 : 0;
  c32 fv[IF > 0 ? IF : 1];
  if constexpr (RES) {
    const c32* fb = ev.p + (long long)b * ev.stride;
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      const int idx = min((int)threadIdx.x + it * 256, FX * FY - 1);
      const int fx = min(max(fx0 - 1 + idx % FX, 0), n - 1), fy = min(max(fy0 - 1 + idx / FX, 0), n - 1);
      fv[it] = fb[(long long)fy * n + fx];
    }
  }
  // rows are loaded from clamped in-grid columns without lane predicates; values of lanes
  // outside the grid are never used (every use below is guarded by the same condition)
  c32 rv[IV], wv[IV], kv[RES ? IV : 1];
#pragma unroll
  for (int it = 0; it < IV; ++it) {
    const int ly = r0 + RPI * it, gy = fy0 + ly;
    if (ly < RYU && gy >= 0 && gy < n) {
      const long long row = (long long)gy * n;
      rv[it] = at_byte(rb + row, ob);
      wv[it] = at_byte(lv.wd + row, ob);
      if constexpr (RES) kv[it] = at_byte(lv.coef + row, ob);
    }
  }
  if constexpr (RES) {
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      const int idx = threadIdx.x + it * 256;
      const int fx = fx0 - 1 + idx % FX, fy = fy0 - 1 + idx / FX;
      const bool ok = fx >= 0 && fx < n && fy >= 0 && fy < n;
      if (idx < FX * FY) sF[idx / FX][idx % FX] = ok ? fv[it] : make_float2(0.f, 0.f);
    }
    __syncthreads();
  }
#pragma unroll
  for (int it = 0; it < IV; ++it) {
    const int ly = r0 + RPI * it, gy = fy0 + ly;
    c32 v1 = make_float2(0.f, 0.f);  // W r, zero outside the grid
    if (inx && ly < RYU && gy >= 0 && gy < n) {
      rv[it] = cscale(rv[it], sc);
      if constexpr (RES) {
        // r - K e with K e = D e - (sum of in-grid neighbours); sF is zero outside the grid
        const int ng = ghosts2(gx, gy, n);
        const c32 D = make_float2(4.0f - kv[it].x - ng * lv.ghost.x, -kv[it].y - ng * lv.ghost.y);
        const int fx = lx + 1, fy = ly + 1;
        const c32 nb = cadd(cadd(sF[fy][fx - 1], sF[fy][fx + 1]), cadd(sF[fy - 1][fx], sF[fy + 1][fx]));
        rv[it] = cadd(csub(rv[it], cmul(D, sF[fy][fx])), nb);
      }
      v1 = cmul(rv[it], wv[it]);
    }
    sV[ly][lx] = v1;
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IV; ++it) {
    const int ly = r0 + RPI * it, gy = fy0 + ly;
    if (lx < 1 || lx > RXU - 2 || ly < 1 || ly > RYU - 2) continue;
    c32 sv = make_float2(0.f, 0.f);
    if (inx && gy >= 0 && gy < n) {
      const c32 nb = cadd(cadd(sV[ly][lx - 1], sV[ly][lx + 1]), cadd(sV[ly - 1][lx], sV[ly + 1][lx]));
      sv = cadd(cscale(rv[it], 1.0f - omega), nb);
    }
    sS[ly][lx] = sv;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < TCX * TCY; q += 256) {  // 30 x TCY coarse points may exceed the block
    const int tx = q % TCX, ty = q / TCX;
    const int I = cx0 + tx, J = cy0 + ty;
    if (I < nc && J < nc) {
      const int sx = 2 * tx + 2, sy = 2 * ty + 2;
      c32 acc = cscale(sS[sy][sx], 4.0f);
      acc = cadd(acc, cscale(cadd(cadd(sS[sy][sx - 1], sS[sy][sx + 1]), cadd(sS[sy - 1][sx], sS[sy + 1][sx])), 2.0f));
      acc = cadd(acc, cadd(cadd(sS[sy - 1][sx - 1], sS[sy - 1][sx + 1]), cadd(sS[sy + 1][sx - 1], sS[sy + 1][sx + 1])));
      at_byte(rc.p + (long long)b * rc.stride + (long long)J * nc, (unsigned)I * (unsigned)sizeof(c32)) =
          cscale(acc, 0.25f);
    }
  }
}

// Up-leg: 62 x TY fine points, region (tile and a one-point ring) 64 x (TY + 2).
// With RES the right-hand side is r - K e, formed from e on the region and a
// one-point ring, and the leg writes e + z (as k_up_fused2).
template <int TY, bool RES>
__global__ __launch_bounds__(256) void k_up_col(int nrhs, VecSet r, ScaleSet rs, LevelArgs lv, float omega,
                                                VecSet ec, int nc, VecSet z, const int* active, VecSet ev) {
  constexpr int TX = 62, VY = TY + 2, RPI = 4, IV = VY / RPI;
  static_assert(VY % RPI == 0 && TY % 2 == 0, "whole row groups, even tile origin");
  constexpr int CX = TX / 2 + 2, CY = TY / 2 + 2;
  constexpr int FX = RES ? 66 : 1, FY = RES ? VY + 2 : 1;
  __shared__ c32 sE[CY][CX];
  __shared__ c32 sV[VY][64];
  __shared__ c32 sF[FY][FX];
  const int n = lv.n;
  // workgroup order (xcd_stretch): "right-hand sides fastest, then tiles in raster order",
  // one contiguous stretch per XCD
  const unsigned tiles_x = (unsigned)(n + TX - 1) / TX;
  const unsigned l = xcd_stretch(blockIdx.x, gridDim.x);
  const unsigned t = l / (unsigned)nrhs;
  const int b = (int)(l - t * (unsigned)nrhs);
  if (active && !active[b]) return;
  const int fx0 = (int)(t % tiles_x) * TX, fy0 = (int)(t / tiles_x) * TY;
  const int cxs = fx0 / 2 - 1, cys = fy0 / 2 - 1;
  const c32* eb = ec.p + (long long)b * ec.stride;
  const c32* rb = r.p + (long long)b * r.stride;
  const float sc = scale_of(rs, b);
  const int lx = threadIdx.x & 63;
  const int r0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // the wavefront's first region row
  const int gx = fx0 - 1 + lx;
  const bool inx = gx >= 0 && gx < n;
  const unsigned ob = (unsigned)min(max(gx, 0), n - 1) * (unsigned)sizeof(c32);  // nearest in-grid column, bytes
  // the coarse tile (and with RES the fine correction) loaded from clamped in-grid
  // addresses, back to back with the row loads; zeros outside the grid are put in at
  // the LDS stores
  constexpr int IE = (CX * CY + 255) / 256, IF = RES ? (FX * FY + 255) / 256 : 0;
  c32 evc[IE], fv[IF > 0 ? IF : 1];
#pragma unroll
  for (int it = 0; it < IE; ++it) {
    const int idx = min((int)threadIdx.x + it * 256, CX * CY - 1);
    const int I = min(max(cxs + idx % CX, 0), nc - 1), J = min(max(cys + idx / CX, 0), nc - 1);
    evc[it] = eb[(long long)J * nc + I];
  }
  if constexpr (RES) {
    const c32* fb = ev.p + (long long)b * ev.stride;
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      const int idx = min((int)threadIdx.x + it * 256, FX * FY - 1);
      const int fx = min(max(fx0 - 2 + idx % FX, 0), n - 1), fy = min(max(fy0 - 2 + idx / FX, 0), n - 1);
      fv[it] = fb[(long long)fy * n + fx];
    }
  }
  // rows from clamped in-grid columns without lane predicates; values of lanes outside
  // the grid are never used (every use below is guarded by the same condition)
  c32 rv[IV], wv[IV], kv[RES ? IV : 1];
#pragma unroll
  for (int it = 0; it < IV; ++it) {
    const int gy = fy0 - 1 + r0 + RPI * it;
    if (gy >= 0 && gy < n) {
      const long long row = (long long)gy * n;
      rv[it] = at_byte(rb + row, ob);
      wv[it] = at_byte(lv.wd + row, ob);
      if constexpr (RES) kv[it] = at_byte(lv.coef + row, ob);
    }
  }
#pragma unroll
  for (int it = 0; it < IE; ++it) {
    const int idx = threadIdx.x + it * 256;
    const int I = cxs + idx % CX, J = cys + idx / CX;
    const bool ok = I >= 0 && I < nc && J >= 0 && J < nc;
    if (idx < CX * CY) sE[idx / CX][idx % CX] = ok ? evc[it] : make_float2(0.f, 0.f);
  }
  if constexpr (RES) {
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      const int idx = threadIdx.x + it * 256;
      const int fx = fx0 - 2 + idx % FX, fy = fy0 - 2 + idx / FX;
      const bool ok = fx >= 0 && fx < n && fy >= 0 && fy < n;
      if (idx < FX * FY) sF[idx / FX][idx % FX] = ok ? fv[it] : make_float2(0.f, 0.f);
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IV; ++it) {  // v2 = W r + P e on the region (zero outside the grid)
    const int ly = r0 + RPI * it, gy = fy0 - 1 + ly;
    c32 v2 = make_float2(0.f, 0.f);
    if (inx && gy >= 0 && gy < n) {
      rv[it] = cscale(rv[it], sc);
      if constexpr (RES) {
        const int ng = ghosts2(gx, gy, n);
        const c32 D = make_float2(4.0f - kv[it].x - ng * lv.ghost.x, -kv[it].y - ng * lv.ghost.y);
        const int fx = lx + 1, fy = ly + 1;
        const c32 nb = cadd(cadd(sF[fy][fx - 1], sF[fy][fx + 1]), cadd(sF[fy - 1][fx], sF[fy + 1][fx]));
        rv[it] = cadd(csub(rv[it], cmul(D, sF[fy][fx])), nb);
      }
      const int I = (gx >> 1) - cxs, J = (gy >> 1) - cys, ox = gx & 1, oy = gy & 1;
      const c32 a = sE[J][I], bb = sE[J][I + ox], c = sE[J + oy][I], d = sE[J + oy][I + ox];
      v2 = cadd(cmul(rv[it], wv[it]), cscale(cadd(cadd(a, bb), cadd(c, d)), 0.25f));
    }
    sV[ly][lx] = v2;
  }
  __syncthreads();
  c32* zb = z.p + (long long)b * z.stride;
#pragma unroll
  for (int it = 0; it < IV; ++it) {
    const int ly = r0 + RPI * it, gy = fy0 - 1 + ly;
    if (lx < 1 || lx > TX || ly < 1 || ly > TY || gx >= n || gy >= n) continue;
    const c32 nb = cadd(cadd(sV[ly][lx - 1], sV[ly][lx + 1]), cadd(sV[ly - 1][lx], sV[ly + 1][lx]));
    c32 zv = cadd(cscale(sV[ly][lx], 1.0f - omega), cmul(wv[it], cadd(rv[it], nb)));
    if constexpr (RES) zv = cadd(zv, sF[ly + 1][lx + 1]);
    at_byte(zb + (long long)gy * n, ob) = zv;
  }
}

// The finest-level step of the s-step basis in the column layout: up-leg of
// Z_j, W_{j+1} = A Z_j and the down-leg of W_{j+1} in one launch.  A 56 x 12
// tile; the region is 64 x 20 (a four-point ring): v2 on all of it, z on a
// three-point ring, W_{j+1} on a two-point ring (its v1 = W W_{j+1}), s on a
// one-point ring, and the coarse right-hand side of the 28 x 6 coarse points
// whose fine points lie in the tile.  The basis vector W_{j+1} carries scale 1.
// Same arithmetic per point as the separate kernels.
__global__ __launch_bounds__(256) void k_step_col(int nrhs, VecSet r, ScaleSet rs, LevelArgs lv, LevelArgs la,
                                                  float omega, VecSet ec, int nc, VecSet z, VecSet w, VecSet rc,
                                                  const int* active) {
  constexpr int TX = 56, TY = 12, VY = TY + 8, RPI = 4, IV = VY / RPI;
  constexpr int CX = 33, CY = TY / 2 + 5, KX = TX / 2, KY = TY / 2;
  __shared__ c32 sE[CY][CX];
  __shared__ c32 sA[VY][64];  // v2, then v1 = W W_{j+1}
  __shared__ c32 sB[VY][64];  // z, then s
  const int n = lv.n;
  const int tiles_x = (n + TX - 1) / TX;
  const unsigned tiles = (unsigned)(tiles_x * ((n + TY - 1) / TY));
  const TileId id = xcd_tile(blockIdx.x, nrhs, tiles, HELM_RHS_GROUP);
  const int b = id.b;
  if (active && !active[b]) return;
  const int fx0 = (id.t % tiles_x) * TX, fy0 = (id.t / tiles_x) * TY;
  const int cxs = fx0 / 2 - 2, cys = fy0 / 2 - 2;
  const c32* eb = ec.p + (long long)b * ec.stride;
  const c32* rb = r.p + (long long)b * r.stride;
  const float sc = scale_of(rs, b);
  const int lx = threadIdx.x & 63, r0 = threadIdx.x >> 6;
  const int gx = fx0 - 4 + lx;
  const bool inx = gx >= 0 && gx < n;
  constexpr int IE = (CX * CY + 255) / 256;
  c32 evc[IE];
#pragma unroll
  for (int it = 0; it < IE; ++it) {
    const int idx = threadIdx.x + it * 256;
    const int I = cxs + idx % CX, J = cys + idx / CX;
    const bool ok = idx < CX * CY && I >= 0 && I < nc && J >= 0 && J < nc;
    evc[it] = ok ? eb[(long long)J * nc + I] : make_float2(0.f, 0.f);
  }
  c32 rv[IV], wv[IV], kv[IV];
  bool ing[IV];
#pragma unroll
  for (int it = 0; it < IV; ++it) {
    const int ly = r0 + RPI * it, gy = fy0 - 4 + ly;
    ing[it] = inx && gy >= 0 && gy < n;
    const long long p = ing[it] ? (long long)gy * n + gx : 0;
    rv[it] = ing[it] ? cscale(rb[p], sc) : make_float2(0.f, 0.f);
    wv[it] = ing[it] ? lv.wd[p] : make_float2(0.f, 0.f);
    kv[it] = ing[it] && lx >= 2 && lx <= 61 && ly >= 2 && ly <= VY - 3 ? la.coef[p] : make_float2(0.f, 0.f);
  }
#pragma unroll
  for (int it = 0; it < IE; ++it) {
    const int idx = threadIdx.x + it * 256;
    if (idx < CX * CY) sE[idx / CX][idx % CX] = evc[it];
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IV; ++it) {  // v2 = W r + P e
    const int ly = r0 + RPI * it, gy = fy0 - 4 + ly;
    c32 v2 = make_float2(0.f, 0.f);
    if (ing[it]) {
      const int I = (gx >> 1) - cxs, J = (gy >> 1) - cys, ox = gx & 1, oy = gy & 1;
      const c32 a = sE[J][I], bb = sE[J][I + ox], c = sE[J + oy][I], d = sE[J + oy][I + ox];
      v2 = cadd(cmul(rv[it], wv[it]), cscale(cadd(cadd(a, bb), cadd(c, d)), 0.25f));
    }
    sA[ly][lx] = v2;
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IV; ++it) {  // z on the three-point ring
    const int ly = r0 + RPI * it;
    if (lx < 1 || lx > 62 || ly < 1 || ly > VY - 2) continue;
    c32 zv = make_float2(0.f, 0.f);
    if (ing[it]) {
      const c32 nb = cadd(cadd(sA[ly][lx - 1], sA[ly][lx + 1]), cadd(sA[ly - 1][lx], sA[ly + 1][lx]));
      zv = cadd(cscale(sA[ly][lx], 1.0f - omega), cmul(wv[it], cadd(rv[it], nb)));
    }
    sB[ly][lx] = zv;
  }
  __syncthreads();
  c32* zb = z.p + (long long)b * z.stride;
  c32* wb = w.p + (long long)b * w.stride;
  c32 wn[IV];
#pragma unroll
  for (int it = 0; it < IV; ++it) {  // W_{j+1} = A z on the two-point ring; v1 = W W_{j+1}
    const int ly = r0 + RPI * it, gy = fy0 - 4 + ly;
    wn[it] = make_float2(0.f, 0.f);
    if (lx < 2 || lx > 61 || ly < 2 || ly > VY - 3) continue;
    c32 v1 = make_float2(0.f, 0.f);
    if (ing[it]) {
      const c32 zc = sB[ly][lx];
      const int ng = ghosts2(gx, gy, n);
      const c32 D = make_float2(4.0f - kv[it].x - ng * la.ghost.x, -kv[it].y - ng * la.ghost.y);
      const c32 nb = cadd(cadd(sB[ly][lx - 1], sB[ly][lx + 1]), cadd(sB[ly - 1][lx], sB[ly + 1][lx]));
      wn[it] = csub(cmul(D, zc), nb);
      v1 = cmul(wn[it], wv[it]);
      if (lx >= 4 && lx < TX + 4 && ly >= 4 && ly < TY + 4) {
        const long long p = (long long)gy * n + gx;
        zb[p] = zc;
        wb[p] = wn[it];
      }
    }
    sA[ly][lx] = v1;
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < IV; ++it) {  // s = W_{j+1} - K v1 on the one-point ring
    const int ly = r0 + RPI * it;
    if (lx < 3 || lx > 60 || ly < 3 || ly > VY - 4) continue;
    c32 sv = make_float2(0.f, 0.f);
    if (ing[it]) {
      const c32 nb = cadd(cadd(sA[ly][lx - 1], sA[ly][lx + 1]), cadd(sA[ly - 1][lx], sA[ly + 1][lx]));
      sv = cadd(cscale(wn[it], 1.0f - omega), nb);
    }
    sB[ly][lx] = sv;
  }
  __syncthreads();
  if (threadIdx.x < KX * KY) {  // the coarse right-hand side 4 R s
    const int tx = threadIdx.x % KX, ty = threadIdx.x / KX;
    const int I = fx0 / 2 + tx, J = fy0 / 2 + ty;
    if (I < nc && J < nc) {
      const int sx = 2 * tx + 4, sy = 2 * ty + 4;
      c32 acc = cscale(sB[sy][sx], 4.0f);
      acc = cadd(acc, cscale(cadd(cadd(sB[sy][sx - 1], sB[sy][sx + 1]), cadd(sB[sy - 1][sx], sB[sy + 1][sx])), 2.0f));
      acc = cadd(acc, cadd(cadd(sB[sy - 1][sx - 1], sB[sy - 1][sx + 1]), cadd(sB[sy + 1][sx - 1], sB[sy + 1][sx + 1])));
      rc.p[(long long)b * rc.stride + (long long)J * nc + I] = cscale(acc, 0.25f);
    }
  }
}

// ------------------------------------------------------------ fused 3D legs
// The down-leg: DCX x CY coarse points, a fine region of 63 x (R NW) from 2 c0 - 2.  Per fine
// plane f (bottom to top): v1(f) = W r; then s(f - 1) = r - K v1 on the region's interior,
// weighted in z in registers (1/2 for f - 1 = 2K, 1/4 to K - 1 and K for f - 1 = 2K - 1); only a
// finished coarse plane's sum goes through LDS for the in-plane full weighting, one plane
// later, behind that plane's barrier.
constexpr int DCX = 30;
template <int R, int NW>
__global__ __launch_bounds__(64 * NW) void k_down_march3(int nrhs, VecSet r, ScaleSet rs, LevelArgs lv, float omega,
                                                         VecSet rc, int nc, const int* active, int planes) {
  constexpr int CY = (R * NW - 3) / 2, CIT = (DCX * CY + 64 * NW - 1) / (64 * NW);
  __shared__ MarchLds<R, NW> sV;
  __shared__ c32 sS[R * NW][64];
  const int n = lv.n;
  const int tx_n = (nc + DCX - 1) / DCX, ty_n = (nc + CY - 1) / CY;
  const unsigned tiles = (unsigned)(tx_n * ty_n * ((nc + planes - 1) / planes));
  const TileId id = xcd_tile(blockIdx.x, nrhs, tiles, HELM_RHS_GROUP);
  const int b = id.b;
  if (active && !active[b]) return;
  const int cx0 = (id.t % tx_n) * DCX, cy0 = ((id.t / tx_n) % ty_n) * CY, kz0 = (id.t / (tx_n * ty_n)) * planes;
  const int kz1 = min(nc, kz0 + planes);
  const float sc = scale_of(rs, b), om1 = 1.0f - omega;
  const c32* rb = r.p + (long long)b * r.stride;
  c32* cb = rc.p + (long long)b * rc.stride + (long long)cy0 * nc + cx0;
  const long long n2 = (long long)n * n, nc2 = (long long)nc * nc;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gx = 2 * cx0 - 2 + lane, gy0 = 2 * cy0 - 2 + w * R;
  const bool inx = gx >= 0 && gx < n;
  const unsigned xo = inx ? (unsigned)gx * (unsigned)sizeof(c32) : 0u;
  bool in[R];
  int row[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    in[i] = gy0 + i >= 0 && gy0 + i < n;
    row[i] = min(max(gy0 + i, 0), n - 1) * n;
  }
  // the coarse points this thread weights
  unsigned coff[CIT];
  int cl[CIT];
  bool cin[CIT];
#pragma unroll
  for (int it = 0; it < CIT; ++it) {
    const int q = threadIdx.x + it * 64 * NW, tx = q % DCX, ty = q / DCX;
    cin[it] = ty < CY && cx0 + tx < nc && cy0 + ty < nc;
    coff[it] = cin[it] ? (unsigned)(ty * nc + tx) : 0u;
    cl[it] = cin[it] ? (2 * ty + 2) * 64 + 2 * tx + 2 : 65;
  }
  auto weight = [&](int K) {  // coarse plane K from the sums in LDS
#pragma unroll
    for (int it = 0; it < CIT; ++it) {
      const c32* p = &sS[0][0] + cl[it];
      const c32 e = cadd(cadd(p[-1], p[1]), cadd(p[-64], p[64]));
      const c32 d = cadd(cadd(p[-65], p[-63]), cadd(p[63], p[65]));
      const c32 t = cadd(cadd(p[0], cscale(e, 0.5f)), cscale(d, 0.25f));
      if (cin[it]) cb[K * nc2 + coff[it]] = t;
    }
  };
  const int f0 = 2 * kz0 - 2, f1 = 2 * kz1;  // fine planes whose v1 is needed
  c32 rn[R], wn[R], vp[R], a[R], zs[R];
  auto fetch = [&](int f) {
    const long long z = (long long)min(max(f, 0), n - 1) * n2;
    const unsigned x = here(xo);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      rn[i] = at_byte(rb + z + row[i], x);
      wn[i] = at_byte(lv.wd + z + row[i], x);
    }
  };
  fetch(f0);
#pragma unroll
  for (int i = 0; i < R; ++i) vp[i] = a[i] = zs[i] = make_float2(0.f, 0.f);
  // odd: f is odd, so that s of the coarse plane's own fine plane f - 1 is complete; else f - 1
  // closes one coarse plane (its sums go to LDS, weighted in the next step) and opens the next
  auto step = [&](auto odd, int f) {
    c32 v[R], rf[R], nb[R];
    const bool inz = f >= 0 && f < n, ing = f >= 1 && f <= n;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      rf[i] = cscale(rn[i], sc);
      v[i] = select0(inx && inz && in[i], cmul(rf[i], wn[i]));
    }
    fetch(min(f + 1, f1));
    plane_neighbours<decltype(odd)::value>(sV, w, lane, v, nb);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const c32 s = cscale(select0(inx && ing && in[i], cadd(a[i], v[i])), odd ? 0.5f : 0.25f);
      zs[i] = cadd(zs[i], s);
      if (!odd) {
        sS[w * R + i][lane] = zs[i];
        zs[i] = s;
      }
      a[i] = cadd(cadd(cscale(rf[i], om1), nb[i]), vp[i]);
      vp[i] = v[i];
      asm volatile("" : "+v"(a[i].x), "+v"(a[i].y));  // before the branch: the lane shifts fold into the additions
    }
    if constexpr (decltype(odd)::value)
      if (f > f0 + 3) weight((f - 3) >> 1);
  };
  step(std::false_type{}, f0);
  for (int f = f0 + 1; f < f1; f += 2) {
    step(std::true_type{}, f);
    step(std::false_type{}, f + 1);
  }
  __syncthreads();
  weight(kz1 - 1);
}

// The up-leg: own points in lanes 1 .. 62 and rows 1 .. R NW - 2 of the region that starts at
// (x0 - 1, y0 - 1).  The in-plane interpolation of a coarse plane is formed once, from one
// LDS copy, and kept in registers for the (up to three) fine planes that read it: rows start odd
// and R is even, so which rows lie between coarse rows is known at compile time.  Per fine
// plane f: v2(f) = W r + P e, then z(f - 1) from v2(f - 2 .. f), where
// (1 - omega) v2 + W (r + neighbours so far) is all that is kept of plane f - 1.  With acc
// the leg adds z to the output instead of overwriting it (a repeated coarse visit:
// e + MG(r - K e, 0) without a separate pass).
constexpr int UX = 62;
template <int R, int NW>
__global__ __launch_bounds__(64 * NW) void k_up_march3(int nrhs, VecSet r, ScaleSet rs, LevelArgs lv, float omega,
                                                       VecSet ec, int nc, VecSet z, const int* active, int acc,
                                                       int planes) {
  static_assert(R % 2 == 0, "rows in pairs");
  constexpr int UY = R * NW - 2, CX = UX / 2 + 2, CY = R * NW / 2 + 1, NCP = CX * CY,
                ITC = (NCP + 64 * NW - 1) / (64 * NW);
  __shared__ MarchLds<R, NW> sV;
  __shared__ c32 sE[CY * CX];
  const int n = lv.n;
  const int tx_n = (n + UX - 1) / UX, ty_n = (n + UY - 1) / UY;
  const unsigned tiles = (unsigned)(tx_n * ty_n * ((n + planes - 1) / planes));
  const TileId id = xcd_tile(blockIdx.x, nrhs, tiles, HELM_RHS_GROUP);
  const int b = id.b;
  if (active && !active[b]) return;
  const int x0 = (id.t % tx_n) * UX, y0 = ((id.t / tx_n) % ty_n) * UY, z0 = (id.t / (tx_n * ty_n)) * planes;
  const int z1 = min(n, z0 + planes);
  const int cxs = x0 / 2 - 1, cys = y0 / 2 - 1;
  const float sc = scale_of(rs, b), om1 = 1.0f - omega;
  const c32* rb = r.p + (long long)b * r.stride;
  const c32* eb = ec.p + (long long)b * ec.stride;
  c32* zb = z.p + (long long)b * z.stride;
  const long long n2 = (long long)n * n, nc2 = (long long)nc * nc;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gx = x0 - 1 + lane, gy0 = y0 - 1 + w * R;
  const bool inx = gx >= 0 && gx < n, ownx = inx && lane >= 1 && lane <= UX;
  const unsigned xo = inx ? (unsigned)gx * (unsigned)sizeof(c32) : 0u;
  bool in[R], own[R];
  int row[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int ly = w * R + i;
    in[i] = gy0 + i >= 0 && gy0 + i < n;
    own[i] = in[i] && ly >= 1 && ly <= UY;
    row[i] = min(max(gy0 + i, 0), n - 1) * n;
  }
  unsigned coff[ITC];
  bool cin[ITC];
#pragma unroll
  for (int it = 0; it < ITC; ++it) {
    const int q = threadIdx.x + it * 64 * NW;
    const int I = cxs + q % CX, J = cys + q / CX;
    cin[it] = q < NCP && I >= 0 && I < nc && J >= 0 && J < nc;
    coff[it] = cin[it] ? (unsigned)(J * nc + I) * (unsigned)sizeof(c32) : 0u;
  }
  c32 rn[R], wn[R], cn[ITC];
  auto fetch = [&](int f) {
    const long long p = (long long)min(max(f, 0), n - 1) * n2;
    const unsigned x = here(xo);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      rn[i] = at_byte(rb + p + row[i], x);
      wn[i] = at_byte(lv.wd + p + row[i], x);
    }
  };
  auto fetch_coarse = [&](int K) {
    const bool inz = K >= 0 && K < nc;
    const c32* p = eb + (long long)min(max(K, 0), nc - 1) * nc2;
#pragma unroll
    for (int it = 0; it < ITC; ++it) cn[it] = select0(inz && cin[it], at_byte(p, coff[it]));
  };
  auto store_coarse = [&]() {
#pragma unroll
    for (int it = 0; it < ITC; ++it) {
      const int q = threadIdx.x + it * 64 * NW;
      if (q < NCP) sE[q] = cn[it];
    }
  };
  // gx >> 1 and the point above it, gx odd (lane even) only; row i = 0 is odd: it lies between
  // the coarse rows (gy0 >> 1) and (gy0 >> 1) + 1
  const int ex = ((gx + 2) >> 1) - 1 - cxs, exo = lane & 1 ? ex : ex + 1;
  auto interpolate = [&](c32 (&p)[R]) {
    c32 h[R / 2 + 1];
#pragma unroll
    for (int q = 0; q < R / 2 + 1; ++q) {
      const c32* row = sE + (w * (R / 2) + q) * CX;
      h[q] = cscale(cadd(row[ex], row[exo]), 0.5f);
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
      p[i] = i & 1 ? h[(i + 1) / 2] : cscale(cadd(h[i / 2], h[i / 2 + 1]), 0.5f);
  };
  const int fa = z0 - 1, fb = z1;  // planes whose v2 is needed; z0 is even
  c32 pc[R], vp[R], t[R], wc[R];
  fetch(fa);
  fetch_coarse((fa - 1) / 2);
  store_coarse();
  fetch_coarse((fa + 1) / 2);
  __syncthreads();
  interpolate(pc);
  __syncthreads();
  store_coarse();
  __syncthreads();
#pragma unroll
  for (int i = 0; i < R; ++i) vp[i] = t[i] = wc[i] = make_float2(0.f, 0.f);
  auto step = [&](auto odd, int f) {
    c32 v[R], rf[R], wf[R], nb[R];
    const bool inz = f >= 0 && f < n;
    if constexpr (decltype(odd)::value) {  // between two coarse planes: the upper one is in LDS
      c32 pn[R];
      interpolate(pn);
      fetch_coarse((f + 3) >> 1);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        v[i] = cscale(cadd(pc[i], pn[i]), 0.5f);
        pc[i] = pn[i];
      }
    } else {  // on a coarse plane that every thread has read, so that the next can take its place
      store_coarse();
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = pc[i];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
      rf[i] = cscale(rn[i], sc);
      wf[i] = wn[i];
      v[i] = select0(inx && inz && in[i], cadd(cmul(rf[i], wf[i]), v[i]));
    }
    fetch(min(f + 1, fb));
    plane_neighbours<decltype(odd)::value>(sV, w, lane, v, nb);
    c32 zo[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      zo[i] = cadd(t[i], cmul(wc[i], v[i]));
      t[i] = cadd(cscale(v[i], om1), cmul(wf[i], cadd(cadd(rf[i], nb[i]), vp[i])));
      wc[i] = wf[i];
      vp[i] = v[i];
      asm volatile("" : "+v"(t[i].x), "+v"(t[i].y));  // before the branch: the lane shifts fold into the additions
    }
    if (f > z0 && f <= fb && ownx) {  // output plane f - 1
      c32* zp = zb + (long long)(f - 1) * n2;
      const unsigned x = here(xo);
      if (acc)
#pragma unroll
        for (int i = 0; i < R; ++i) zo[i] = cadd(at_byte(zp + row[i], x), zo[i]);
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (own[i]) *(c32*)((char*)(zp + row[i]) + x) = zo[i];
    }
  };
  for (int f = fa; f <= fb; f += 2) {
    step(std::true_type{}, f);
    step(std::false_type{}, f + 1);
  }
}

// ------------------------------------------------------------ generic (2D/3D)
__global__ void k_jacobi_zero(int dim, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet v,
                              const int* active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= lv.N) return;
  const Coord c = coord_of32((unsigned)p, (unsigned)lv.n, dim);
  const c32 rv = cscale(r.p[(long long)b * r.stride + p], scale_of(rs, b));
  v.p[(long long)b * v.stride + p] = cscale(cmul(rv, crcp(diag_at(lv, p, ghosts_of(c, lv.n, dim), dim))), omega);
}

__global__ void k_jacobi(int dim, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet v, VecSet vout,
                         const int* active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= lv.N) return;
  const Coord c = coord_of32((unsigned)p, (unsigned)lv.n, dim);
  const c32* vb = v.p + (long long)b * v.stride;
  const c32 rv = cscale(r.p[(long long)b * r.stride + p], scale_of(rs, b));
  const c32 D = diag_at(lv, p, ghosts_of(c, lv.n, dim), dim);
  // v + w D^-1 (r - K v), K v = D v - sum of neighbours
  const c32 res = csub(cadd(rv, neighbour_sum(vb, p, c, lv.n, dim)), cmul(D, vb[p]));
  vout.p[(long long)b * vout.stride + p] = cadd(vb[p], cscale(cmul(res, crcp(D)), omega));
}

__global__ void k_restrict_residual(int dim, VecSet r, ScaleSet rs, VecSet v, LevelArgs lv, VecSet rc, int nc,
                                    const int* active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long ncN = dim == 2 ? (long long)nc * nc : (long long)nc * nc * nc;
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= ncN) return;
  const Coord C = coord_of32((unsigned)q, (unsigned)nc, dim);
  const int n = lv.n;
  const float sc = scale_of(rs, b);
  const c32* rb = r.p + (long long)b * r.stride;
  const c32* vb = v.p ? v.p + (long long)b * v.stride : nullptr;
  const float w1[3] = {0.25f, 0.5f, 0.25f};
  c32 acc = make_float2(0.f, 0.f);
  const int zlo = dim == 3 ? -1 : 0, zhi = dim == 3 ? 1 : 0;
  for (int dz = zlo; dz <= zhi; ++dz)
    for (int dy = -1; dy <= 1; ++dy)
      for (int dx = -1; dx <= 1; ++dx) {
        Coord f{2 * C.x + dx, 2 * C.y + dy, dim == 3 ? 2 * C.z + dz : 0};
        if (f.x < 0 || f.x >= n || f.y < 0 || f.y >= n || f.z < 0 || f.z >= n) continue;
        const long long p = ((long long)f.z * n + f.y) * n + f.x;
        c32 s = cscale(rb[p], sc);
        if (vb) {
          const c32 D = diag_at(lv, p, ghosts_of(f, n, dim), dim);
          s = cadd(csub(s, cmul(D, vb[p])), neighbour_sum(vb, p, f, n, dim));
        }
        const float wgt = w1[dx + 1] * w1[dy + 1] * (dim == 3 ? w1[dz + 1] : 1.0f);
        acc = cadd(acc, cscale(s, wgt));
      }
  rc.p[(long long)b * rc.stride + q] = cscale(acc, 4.0f);
}

// vout = v + P ec (vout may be v)
__global__ void k_prolong_add(int dim, VecSet ec, int nc, VecSet v, VecSet vout, int n, long long N,
                              const int* active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const Coord f = coord_of32((unsigned)p, (unsigned)n, dim);
  const c32* eb = ec.p + (long long)b * ec.stride;
  c32 acc = make_float2(0.f, 0.f);
  const int oz = dim == 3 ? (f.z & 1) : 0;
  for (int kz = 0; kz <= oz; ++kz)
    for (int ky = 0; ky <= (f.y & 1); ++ky)
      for (int kx = 0; kx <= (f.x & 1); ++kx) {
        const int I = (f.x >> 1) + kx, J = (f.y >> 1) + ky, K = dim == 3 ? (f.z >> 1) + kz : 0;
        float wgt = ((f.x & 1) ? 0.5f : 1.0f) * ((f.y & 1) ? 0.5f : 1.0f) * (oz ? 0.5f : 1.0f);
        acc = cadd(acc, cscale(eb[((long long)K * nc + J) * nc + I], wgt));
      }
  const c32* vb = v.p + (long long)b * v.stride;
  vout.p[(long long)b * vout.stride + p] = cadd(vb[p], acc);
}

// out = s_b b - K v on a level (the right-hand side of a repeated coarse visit:
// MG(b, v) = v + MG(b - K v, 0) for the affine multigrid cycle; the residual
// ahead of a restriction in the generic legs)
__global__ void k_level_residual(int dim, VecSet bvec, ScaleSet bs, VecSet v, LevelArgs lv, VecSet out,
                                 const int* active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= lv.N) return;
  const Coord c = coord_of32((unsigned)p, (unsigned)lv.n, dim);
  const c32* vb = v.p + (long long)b * v.stride;
  const c32 D = diag_at(lv, p, ghosts_of(c, lv.n, dim), dim);
  const c32 kv = csub(cmul(D, vb[p]), neighbour_sum(vb, p, c, lv.n, dim));
  out.p[(long long)b * out.stride + p] = csub(cscale(bvec.p[(long long)b * bvec.stride + p], scale_of(bs, b)), kv);
}

// the same residual in 3D, marching in z
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_level_residual_march3(int nrhs, VecSet bvec, ScaleSet bs, VecSet v,
                                                                   LevelArgs lv, VecSet out, const int* active,
                                                                   int planes) {
  const TileId id = xcd_tile(blockIdx.x, nrhs, march_apply_tiles<NW>(lv.n, planes), HELM_RHS_GROUP);
  const int b = id.b;
  if (active && !active[b]) return;
  march_apply<true, NW>(v.p + (long long)b * v.stride, bvec.p + (long long)b * bvec.stride, scale_of(bs, b), lv, id.t,
                        planes, out.p + (long long)b * out.stride);
}

// y += x for every active right-hand side
__global__ void k_add(VecSet x, VecSet y, long long N, const int* active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  c32* yb = y.p + (long long)b * y.stride;
  yb[p] = cadd(yb[p], x.p[(long long)b * x.stride + p]);
}

// y = out_scale * (D x - sum of neighbours), D = 2d - coef - g #ghosts
__global__ void k_apply(int dim, VecSet x, ScaleSet xs, LevelArgs lv, float out_scale, VecSet y,
                        const int* active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= lv.N) return;
  const Coord c = coord_of32((unsigned)p, (unsigned)lv.n, dim);
  const c32* xb = x.p + (long long)b * x.stride;
  const c32 D = diag_at(lv, p, ghosts_of(c, lv.n, dim), dim);
  const c32 out = csub(cmul(D, xb[p]), neighbour_sum(xb, p, c, lv.n, dim));
  y.p[(long long)b * y.stride + p] = cscale(out, out_scale * scale_of(xs, b));
}

// Z = M R, the exact coarsest solve of a batch, with M given transposed (minvT[k Nc + row] =
// M[row][k]) and read once per BT right-hand sides.  A workgroup takes 16 rows: threads (row,
// column group), 64 groups, each with the entries of its columns loaded straight from memory (128
// bytes a column, KC columns ahead of the products) and R passing through LDS, KC columns at a
// time; then the groups' sums are added in a fixed order.  No partial sums leave the workgroup.  Bound by the inverse's 8 Nc^2 bytes: 24 MB at 12^3, in
// 21 us for 8 right-hand sides (45 + 5 with 64-row tiles, eight column slices and a second
// launch; the same product with one thread per row, for fewer than four right-hand sides, made a
// cycle at 100^3 x 1 208 us, now 126).
constexpr int CS_ROWS = 16, CS_NT = 1024, CS_G = CS_NT / CS_ROWS;
template <int BT, int CS_KC>
__global__ __launch_bounds__(CS_NT) void k_coarse_gemm(const c32* minvT, int Nc, int B, VecSet r, VecSet z,
                                                       const int* active) {
  constexpr int CS_U = CS_KC / CS_G;
  __shared__ __align__(16) c32 sR[CS_KC][BT];
  __shared__ c32 red[CS_NT / HELM_WAVE][CS_ROWS][BT];
  const int tid = threadIdx.x, rr = tid % CS_ROWS, g = tid / CS_ROWS, b0 = blockIdx.y * BT;
  const int row = blockIdx.x * CS_ROWS + rr;
  const c32* mp = minvT + min(row, Nc - 1);
  c32 mn[CS_U];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int u = 0; u < CS_U; ++u) mn[u] = mp[(long long)min(k0 + g + u * CS_G, Nc - 1) * Nc];
  };
  fetch(0);
  c32 acc[BT];
#pragma unroll
  for (int q = 0; q < BT; ++q) acc[q] = make_float2(0.f, 0.f);
  for (int k0 = 0; k0 < Nc; k0 += CS_KC) {
    __syncthreads();
    for (int i = tid; i < CS_KC * BT; i += CS_NT) {
      const int k = i % CS_KC, q = i / CS_KC;
      sR[k][q] = k0 + k < Nc && b0 + q < B ? r.p[(long long)(b0 + q) * r.stride + k0 + k] : make_float2(0.f, 0.f);
    }
    c32 m[CS_U];
#pragma unroll
    for (int u = 0; u < CS_U; ++u) m[u] = mn[u];
    if (k0 + CS_KC < Nc) fetch(k0 + CS_KC);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < CS_U; ++u)
#pragma unroll
      for (int q = 0; q < BT; ++q) acc[q] = cfma(m[u], sR[g + u * CS_G][q], acc[q]);  // zero past the last column
  }
#pragma unroll
  for (int q = 0; q < BT; ++q) {
#pragma unroll
    for (int off = CS_ROWS; off < HELM_WAVE; off <<= 1) {
      acc[q].x += __shfl_xor(acc[q].x, off, HELM_WAVE);
      acc[q].y += __shfl_xor(acc[q].y, off, HELM_WAVE);
    }
    if (tid % HELM_WAVE < CS_ROWS) red[tid / HELM_WAVE][rr][q] = acc[q];
  }
  __syncthreads();
  if (tid < CS_ROWS * BT) {
    const int o = tid % CS_ROWS, q = tid / CS_ROWS, b = b0 + q, row_o = blockIdx.x * CS_ROWS + o;
    if (row_o >= Nc || b >= B || (active && !active[b])) return;
    c32 s = make_float2(0.f, 0.f);
#pragma unroll
    for (int w = 0; w < CS_NT / HELM_WAVE; ++w) s = cadd(s, red[w][o][q]);
    z.p[(long long)b * z.stride + row_o] = s;
  }
}

inline unsigned nblocks(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// Tile shapes of the fused legs the autotuner chooses from (index 0 = default):
// down-leg coarse TCX x TCY per block, up-leg fine TX x TY with PY points per thread.
namespace {
struct DownTile {
  int tcx, tcy;
};
struct UpTile {
  int tx, ty, py;
};
// the last entry of each is the column-layout kernel (k_down_col / k_up_col)
constexpr DownTile kDown[] = {{32, 8}, {16, 16}, {64, 4}, {32, 4}, {16, 8}, {30, 8}, {30, 16}};
constexpr UpTile kUp[] = {{64, 16, 4}, {32, 16, 2}, {64, 8, 2}, {32, 32, 4}, {64, 32, 8}, {62, 14, 0}, {62, 30, 0}};
constexpr int kDownCol = 5, kDownCol16 = 6, kUpCol = 5, kUpCol30 = 6;

// launch shapes of the fused finest up-leg + basis matvec (k_up_mv2w), one autotuner
// choice: tile height and right-hand sides per block
struct UpMvShape {
  int rows, k;
};
constexpr UpMvShape kUpMv[] = {{16, 4}, {12, 1}, {20, 1}, {28, 1}, {12, 2}, {12, 4}, {12, 6}, {20, 2}, {20, 4}};

// Shapes of an untuned launch (cfg < 0): the first of each table, but where that makes fewer than
// 1024 workgroups (four per CU) the launch lasts as long as one workgroup, so a smaller tile: 32 x
// 16 points for the up-leg, 12 rows of one right-hand side for the up-leg with the matvec.  Solves
// at 128^2, first shapes / smaller ones, ms: 1 right-hand side 10.2 / 9.7, 4 of them 12.2 / 9.9
// (matvec shape alone), 16 13.7 / 11.5, 256^2 x 8 29.8 / 26.9, 400^2 x 4 47.5 / 42.7; gradient 256^2
// x 32 95.7 / 91.5, FGMRES 203^2 x 7 31.3 / 29.8.  With 1480 and 2960 workgroups the matvec shape of
// one right-hand side lost 1% (577^2 x 16 and x 30).  The down-legs' smaller tiles changed nothing.
constexpr int SMALL_LAUNCH = 1024;
int up_default(int n, int B) { return (long long)B * ((n + 63) / 64) * ((n + 15) / 16) < SMALL_LAUNCH ? 1 : 0; }

template <int TCX, int TCY>
void down_tile(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet rc, int nc,
               const int* active, VecSet e) {
  const int tiles = ((nc + TCX - 1) / TCX) * ((nc + TCY - 1) / TCY);
  if (e.p)
    hipLaunchKernelGGL((k_down_fused2<TCX, TCY, true>), dim3(B * tiles), dim3(TCX * TCY), 0, s, B, r, rs, lv, omega,
                       rc, nc, active, e);
  else
    hipLaunchKernelGGL((k_down_fused2<TCX, TCY, false>), dim3(B * tiles), dim3(TCX * TCY), 0, s, B, r, rs, lv,
                       omega, rc, nc, active, e);
}
template <int TX, int TY, int PY>
void up_tile(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet ec, int nc, VecSet z,
             const int* active, VecSet e) {
  const int tiles = ((lv.n + TX - 1) / TX) * ((lv.n + TY - 1) / TY);
  if (e.p)
    hipLaunchKernelGGL((k_up_fused2<TX, TY, PY, true>), dim3(B * tiles), dim3(TX * (TY / PY)), 0, s, B, r, rs, lv,
                       omega, ec, nc, z, active, e);
  else
    hipLaunchKernelGGL((k_up_fused2<TX, TY, PY, false>), dim3(B * tiles), dim3(TX * (TY / PY)), 0, s, B, r, rs, lv,
                       omega, ec, nc, z, active, e);
}
}  // namespace

namespace {
template <int R, int NW>
void down_march(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet rc, int nc,
                const int* active) {
  constexpr int CY = (R * NW - 3) / 2;
  const int cols = ((nc + DCX - 1) / DCX) * ((nc + CY - 1) / CY);
  // at most 12 coarse planes: cycle at 128^3 x 8 619 / 617 / 613 / 612 / 611 us with 6 / 8 / 10 / 12 / 16
  const int planes = march_planes((long long)B * cols, nc, 12, 1);
  hipLaunchKernelGGL((k_down_march3<R, NW>), dim3(B * cols * ((nc + planes - 1) / planes)), dim3(64 * NW), 0, s, B, r,
                     rs, lv, omega, rc, nc, active, planes);
}
template <int R, int NW>
void up_march(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet ec, int nc, VecSet z,
              const int* active, int acc) {
  constexpr int UY = R * NW - 2;
  const int n = lv.n, cols = ((n + UX - 1) / UX) * ((n + UY - 1) / UY);
  const int planes = march_planes((long long)B * cols, n, 16, 2);
  hipLaunchKernelGGL((k_up_march3<R, NW>), dim3(B * cols * ((n + planes - 1) / planes)), dim3(64 * NW), 0, s, B, r, rs,
                     lv, omega, ec, nc, z, active, acc, planes);
}
}  // namespace

void launch_down_fused3(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet rc, int nc,
                        const int* active) {
  down_march<2, 8>(s, B, r, rs, lv, omega, rc, nc, active);
}

void launch_up_fused3(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet ec, int nc,
                      VecSet z, const int* active, int acc) {
  // tile heights: cycle at 128^3 x 8 629 us with 6 own rows everywhere, 617 with 14 on the 177^3 level
  // only; 64^3 x 8 solve (113^3 finest) 44.2 ms with 14 rows on it, 44.0 with 6
  if (march_tall(lv.n, B, 2048))
    up_march<2, 8>(s, B, r, rs, lv, omega, ec, nc, z, active, acc);
  else
    up_march<2, 4>(s, B, r, rs, lv, omega, ec, nc, z, active, acc);
}

template <int TY, int K>
void up_mv2(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, LevelArgs la, float omega, VecSet ec, int nc,
            VecSet z, VecSet w, const int* active) {
  constexpr int TX = 60;
  const int n = lv.n;
  const int blocks = (B + K - 1) / K * ((n + TX - 1) / TX) * ((n + TY - 1) / TY);
  hipLaunchKernelGGL((k_up_mv2w<TY, K>), dim3(blocks), dim3(256), 0, s, B, r, rs, lv, la, omega, ec, nc, z, w, active);
}

int mg_up_mv_variants() { return (int)(sizeof(kUpMv) / sizeof(kUpMv[0])); }
int mg_up_mv_rows(int cfg) { return kUpMv[cfg].rows; }
int mg_up_mv_rhs_per_block(int cfg) { return kUpMv[cfg].k; }

void launch_up_mv2(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, LevelArgs la, float omega, VecSet ec,
                   int nc, VecSet z, VecSet w, const int* active, int cfg) {
  if (cfg < 0) cfg = mg_up_mv_default(lv.n, B);
#define HELM_UP_MV(TY_, K_)                                                     \
  if (kUpMv[cfg].rows == TY_ && kUpMv[cfg].k == K_) {                           \
    up_mv2<TY_, K_>(s, B, r, rs, lv, la, omega, ec, nc, z, w, active);          \
    return;                                                                     \
  }
  HELM_UP_MV(12, 1) HELM_UP_MV(20, 1) HELM_UP_MV(28, 1) HELM_UP_MV(12, 2) HELM_UP_MV(12, 4)
  HELM_UP_MV(12, 6) HELM_UP_MV(20, 2) HELM_UP_MV(20, 4)
#undef HELM_UP_MV
  up_mv2<16, 4>(s, B, r, rs, lv, la, omega, ec, nc, z, w, active);
}

void launch_step_fused2(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, LevelArgs la, float omega,
                        VecSet ec, int nc, VecSet z, VecSet w, VecSet rc, const int* active) {
  constexpr int TX = 56, TY = 12;
  const int tiles = ((lv.n + TX - 1) / TX) * ((lv.n + TY - 1) / TY);
  hipLaunchKernelGGL(k_step_col, dim3(B * tiles), dim3(256), 0, s, B, r, rs, lv, la, omega, ec, nc, z, w, rc,
                     active);
}

int mg_down_variants() { return (int)(sizeof(kDown) / sizeof(kDown[0])); }
int mg_up_mv_default(int n, int B) {
  return (long long)((B + 3) / 4) * ((n + 59) / 60) * ((n + 15) / 16) < SMALL_LAUNCH ? 1 : 0;
}
int mg_up_variants() { return (int)(sizeof(kUp) / sizeof(kUp[0])); }
void mg_down_shape(int cfg, int* tcx, int* tcy) {
  *tcx = kDown[cfg].tcx;
  *tcy = kDown[cfg].tcy;
}
void mg_up_shape(int cfg, int* tx, int* ty, int* py) {
  *tx = kUp[cfg].tx;
  *ty = kUp[cfg].ty;
  *py = kUp[cfg].py;
}

void launch_down_fused2(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet rc, int nc,
                        const int* active, int cfg, VecSet e) {
  if (cfg == kDownCol) {
    constexpr int TCX = 30, TCY = 8;
    const dim3 grid(B, (nc + TCX - 1) / TCX, (nc + TCY - 1) / TCY);
    if (e.p)
      hipLaunchKernelGGL((k_down_col<TCY, true>), grid, dim3(256), 0, s, r, rs, lv, omega, rc, nc, active, e);
    else
      hipLaunchKernelGGL((k_down_col<TCY, false>), grid, dim3(256), 0, s, r, rs, lv, omega, rc, nc, active, e);
    return;
  }
  if (cfg == kDownCol16) {  // taller column tile: fewer halo rows per coarse row
    constexpr int TCX = 30, TCY = 16;
    const dim3 grid(B, (nc + TCX - 1) / TCX, (nc + TCY - 1) / TCY);
    if (e.p)
      hipLaunchKernelGGL((k_down_col<TCY, true>), grid, dim3(256), 0, s, r, rs, lv, omega, rc, nc, active, e);
    else
      hipLaunchKernelGGL((k_down_col<TCY, false>), grid, dim3(256), 0, s, r, rs, lv, omega, rc, nc, active, e);
    return;
  }
  switch (cfg) {
    case 1: down_tile<16, 16>(s, B, r, rs, lv, omega, rc, nc, active, e); break;
    case 2: down_tile<64, 4>(s, B, r, rs, lv, omega, rc, nc, active, e); break;
    case 3: down_tile<32, 4>(s, B, r, rs, lv, omega, rc, nc, active, e); break;
    case 4: down_tile<16, 8>(s, B, r, rs, lv, omega, rc, nc, active, e); break;
    default: down_tile<32, 8>(s, B, r, rs, lv, omega, rc, nc, active, e); break;
  }
}

void launch_up_fused2(hipStream_t s, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet ec, int nc,
                      VecSet z, const int* active, int cfg, VecSet e) {
  if (cfg < 0) cfg = up_default(lv.n, B);
  if (cfg == kUpCol) {
    constexpr int TX = 62, TY = 14;
    const int blocks = B * ((lv.n + TX - 1) / TX) * ((lv.n + TY - 1) / TY);
    if (e.p)
      hipLaunchKernelGGL((k_up_col<TY, true>), dim3(blocks), dim3(256), 0, s, B, r, rs, lv, omega, ec, nc, z, active,
                         e);
    else
      hipLaunchKernelGGL((k_up_col<TY, false>), dim3(blocks), dim3(256), 0, s, B, r, rs, lv, omega, ec, nc, z, active,
                         e);
    return;
  }
  if (cfg == kUpCol30) {  // taller column tile
    constexpr int TX = 62, TY = 30;
    const int blocks = B * ((lv.n + TX - 1) / TX) * ((lv.n + TY - 1) / TY);
    if (e.p)
      hipLaunchKernelGGL((k_up_col<TY, true>), dim3(blocks), dim3(256), 0, s, B, r, rs, lv, omega, ec, nc, z, active,
                         e);
    else
      hipLaunchKernelGGL((k_up_col<TY, false>), dim3(blocks), dim3(256), 0, s, B, r, rs, lv, omega, ec, nc, z, active,
                         e);
    return;
  }
  switch (cfg) {
    case 1: up_tile<32, 16, 2>(s, B, r, rs, lv, omega, ec, nc, z, active, e); break;
    case 2: up_tile<64, 8, 2>(s, B, r, rs, lv, omega, ec, nc, z, active, e); break;
    case 3: up_tile<32, 32, 4>(s, B, r, rs, lv, omega, ec, nc, z, active, e); break;
    case 4: up_tile<64, 32, 8>(s, B, r, rs, lv, omega, ec, nc, z, active, e); break;
    default: up_tile<64, 16, 4>(s, B, r, rs, lv, omega, ec, nc, z, active, e); break;
  }
}

void launch_jacobi_zero(hipStream_t s, int dim, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet v,
                        const int* active) {
  hipLaunchKernelGGL(k_jacobi_zero, dim3(nblocks(lv.N, 256), B), dim3(256), 0, s, dim, r, rs, lv, omega, v, active);
}

void launch_jacobi(hipStream_t s, int dim, int B, VecSet r, ScaleSet rs, LevelArgs lv, float omega, VecSet v,
                   VecSet vout, const int* active) {
  hipLaunchKernelGGL(k_jacobi, dim3(nblocks(lv.N, 256), B), dim3(256), 0, s, dim, r, rs, lv, omega, v, vout,
                     active);
}

void launch_restrict_residual(hipStream_t s, int dim, int B, VecSet r, ScaleSet rs, VecSet v, LevelArgs lv,
                              VecSet rc, int nc, const int* active) {
  const long long ncN = dim == 2 ? (long long)nc * nc : (long long)nc * nc * nc;
  hipLaunchKernelGGL(k_restrict_residual, dim3(nblocks(ncN, 256), B), dim3(256), 0, s, dim, r, rs, v, lv, rc, nc,
                     active);
}

void launch_prolong_add(hipStream_t s, int dim, int B, VecSet ec, int nc, VecSet v, int n, const int* active,
                        VecSet vout) {
  const long long N = dim == 2 ? (long long)n * n : (long long)n * n * n;
  hipLaunchKernelGGL(k_prolong_add, dim3(nblocks(N, 256), B), dim3(256), 0, s, dim, ec, nc, v, vout.p ? vout : v, n,
                     N, active);
}

void launch_coarse_solve(hipStream_t s, int B, const c32* minvT, int Nc, VecSet r, VecSet z, const int* active) {
  auto gemm = [&](auto kernel, int bt) {
    hipLaunchKernelGGL(kernel, dim3(nblocks(Nc, CS_ROWS), nblocks(B, bt)), dim3(CS_NT), 0, s, minvT, Nc, B, r, z,
                       active);
  };
  if (B == 1) gemm(k_coarse_gemm<1, 512>, 1);
  else if (B <= 4) gemm(k_coarse_gemm<4, 512>, 4);
  else if (B <= 8) gemm(k_coarse_gemm<8, 512>, 8);
  else gemm(k_coarse_gemm<16, 256>, 16);
}

void launch_apply(hipStream_t s, int dim, int B, VecSet x, ScaleSet xs, LevelArgs lv, float out_scale, VecSet y,
                  const int* active) {
  hipLaunchKernelGGL(k_apply, dim3(nblocks(lv.N, 256), B), dim3(256), 0, s, dim, x, xs, lv, out_scale, y, active);
}

void launch_level_residual(hipStream_t s, int dim, int B, VecSet bvec, VecSet v, LevelArgs lv, VecSet out,
                           const int* active, ScaleSet bs) {
  if (dim == 3) {
    auto march = [&](auto kernel, int nw, int planes, unsigned tiles) {
      hipLaunchKernelGGL(kernel, dim3(B * tiles), dim3(64 * nw), 0, s, B, bvec, bs, v, lv, out, active, planes);
    };
    const int n = lv.n, tall = march_apply_planes<8>(n, B), low = march_apply_planes<4>(n, B);
    if (march_tall(n, B, 1024)) march(k_level_residual_march3<8>, 8, tall, march_apply_tiles<8>(n, tall));
    else march(k_level_residual_march3<4>, 4, low, march_apply_tiles<4>(n, low));
    return;
  }
  hipLaunchKernelGGL(k_level_residual, dim3(nblocks(lv.N, 256), B), dim3(256), 0, s, dim, bvec, bs, v, lv, out,
                     active);
}

void launch_add(hipStream_t s, int B, VecSet x, VecSet y, long long N, const int* active) {
  hipLaunchKernelGGL(k_add, dim3(nblocks(N, 256), B), dim3(256), 0, s, x, y, N, active);
}
