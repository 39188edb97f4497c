// Marches in z over a 3D grid: what the 3D kernels of the multigrid levels and of the Krylov
// basis share.
#pragma once

#include <type_traits>

#include "dev_common.h"

// The 3D kernels below walk a column of the grid plane by plane.  A lane keeps one x and
// R consecutive rows of it, the wavefronts of a workgroup stack up in y: the neighbours in y
// are the lane's own registers, those in x come from the lanes beside it, and only the two
// outer rows of each wavefront pass through LDS.  The sum over the four in-plane neighbours
// is formed as soon as a plane is known, so that one barrier per plane is enough (the next
// plane's rows go to the other half of the buffer).  Loads are read at clamped offsets and
// selected, never branched around, and run one plane ahead.
// Measured against the form before it (a point per thread and ring points of their own, every
// neighbour through LDS behind a branch, two barriers a plane): cycle at 128^3 x 8 714 -> 610 us
// (177^3 up-leg 238 -> 207, down-leg 155 -> 144 us), 64^3 x 8 solve 50.0 -> 44.0 ms (113^3 up-leg
// 73 -> 55, down-leg 44 -> 38, basis product 59 -> 55 us).  The finest legs now move 1.2 GB and
// 0.9 GB through the last-level cache at 6 TB/s (W is read once per XCD); all right-hand sides of
// a tile on one XCD read a third less and took as long.
template <int R, int NW>
struct MarchLds {
  c32 lo[2][NW][64], hi[2][NW][64];  // first and last row of each wavefront
};
// sums over the in-plane neighbours of the rows v[0 .. R) (the outer rows of the workgroup and
// lanes 0 and 63 get sums that mean nothing); the only barrier of a plane
template <bool ODD, int R, int NW>
__device__ __forceinline__ void plane_neighbours(MarchLds<R, NW>& s, int w, int lane, const c32 (&v)[R],
                                                 c32 (&nb)[R]) {
  s.lo[ODD][w][lane] = v[0];
  s.hi[ODD][w][lane] = v[R - 1];
  __syncthreads();
  const c32 down = s.hi[ODD][max(w - 1, 0)][lane], up = s.lo[ODD][min(w + 1, NW - 1)][lane];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const c32 a = i ? v[i ? i - 1 : 0] : down, c = i < R - 1 ? v[i < R - 1 ? i + 1 : 0] : up;
    const c32 y = cadd(a, c);
    nb[i].x = y.x + lane_below(v[i].x) + lane_above(v[i].x);
    nb[i].y = y.y + lane_below(v[i].y) + lane_above(v[i].y);
  }
}
__device__ __forceinline__ c32 select0(bool ok, c32 v) { return make_float2(ok ? v.x : 0.f, ok ? v.y : 0.f); }
// an offset whose widening to 64 bits stays beside its uses: a scalar base and a 32-bit offset
// are one instruction, a 64-bit offset kept in registers takes an addition for each access
__device__ __forceinline__ unsigned here(unsigned x) {
  asm("" : "+v"(x));
  return x;
}

// -------------------------------------------------------------------- K v
// out = K v, or with RHS scale b - K v, in a column of 62 x (MR NW - 2) own points: per plane f
// D v - (in-plane neighbours) - v(f - 1) is formed and kept, and plane f - 1 is finished with v(f).
constexpr int MR = 2, MOX = 62;
template <int NW>
__host__ __device__ __forceinline__ unsigned march_apply_tiles(int n, int planes) {
  constexpr int rows = MR * NW - 2;
  return (unsigned)(((n + MOX - 1) / MOX) * ((n + rows - 1) / rows) * ((n + planes - 1) / planes));
}
template <int NW>
int march_apply_planes(int n, int B) {
  return march_planes((long long)B * march_apply_tiles<NW>(n, n), n, 16, 2);
}
// 14 own rows for a launch that fills the chip several times over (fewer ring rows), else 6 (twice
// the workgroups)
inline bool march_tall(int n, int B, int least) { return (long long)B * march_apply_tiles<8>(n, 16) >= least; }
template <bool RHS, int NW>
__device__ __forceinline__ void march_apply(const c32* v, const c32* bv, float bs, const LevelArgs& lv, int tile,
                                            int planes, c32* out) {
  __shared__ MarchLds<MR, NW> sV;
  constexpr int R = MR, MOY = MR * NW - 2;
  const int n = lv.n, tx_n = (n + MOX - 1) / MOX, ty_n = (n + MOY - 1) / MOY;
  const int x0 = (tile % tx_n) * MOX, y0 = ((tile / tx_n) % ty_n) * MOY, z0 = (tile / (tx_n * ty_n)) * planes;
  const int z1 = min(n, z0 + planes);
  const long long n2 = (long long)n * n;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gx = x0 - 1 + lane, gy0 = y0 - 1 + w * R;
  const bool inx = gx >= 0 && gx < n, ownx = inx && lane >= 1 && lane <= MOX;
  const unsigned xo = inx ? (unsigned)gx * (unsigned)sizeof(c32) : 0u;
  bool in[R], own[R];
  int row[R];
  float ngxy[R];  // Sommerfeld ghost neighbours in the plane
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int gy = gy0 + i, ly = w * R + i;
    in[i] = gy >= 0 && gy < n;
    own[i] = in[i] && ly >= 1 && ly <= MOY;
    row[i] = min(max(gy, 0), n - 1) * n;
    ngxy[i] = (float)((gx == 0) + (gx == n - 1) + (gy == 0) + (gy == n - 1));
  }
  c32 vn[R], kn[R], bn[R], vp[R], t[R];
  auto fetch = [&](int f) {
    const long long p = (long long)min(max(f, 0), n - 1) * n2;
    const unsigned x = here(xo);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      vn[i] = at_byte(v + p + row[i], x);
      kn[i] = at_byte(lv.coef + p + row[i], x);
      if (RHS) bn[i] = at_byte(bv + p + row[i], x);
    }
  };
  auto step = [&](auto odd, int f) {
    c32 c[R], k[R], b[R], nb[R], o[R];
    const bool inz = f >= 0 && f < n;
    const float ngz = (float)((f == 0) + (f == n - 1));
#pragma unroll
    for (int i = 0; i < R; ++i) {
      c[i] = select0(inx && inz && in[i], vn[i]);
      k[i] = kn[i];
      if (RHS) b[i] = cscale(bn[i], bs);
    }
    fetch(min(f + 1, z1));
    plane_neighbours<decltype(odd)::value>(sV, w, lane, c, nb);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      o[i] = RHS ? cadd(t[i], c[i]) : csub(t[i], c[i]);
      const float ng = ngxy[i] + ngz;
      const c32 D = make_float2(6.0f - k[i].x - ng * lv.ghost.x, -k[i].y - ng * lv.ghost.y);
      const c32 kv = csub(cmul(D, c[i]), cadd(nb[i], vp[i]));
      t[i] = RHS ? csub(b[i], kv) : kv;
      vp[i] = c[i];
      asm volatile("" : "+v"(t[i].x), "+v"(t[i].y));  // before the branch: the lane shifts fold into the additions
    }
    if (f > z0 && f <= z1 && ownx) {
      c32* op = out + (long long)(f - 1) * n2;
      const unsigned x = here(xo);
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (own[i]) *(c32*)((char*)(op + row[i]) + x) = o[i];
    }
  };
#pragma unroll
  for (int i = 0; i < R; ++i) vp[i] = t[i] = make_float2(0.f, 0.f);
  fetch(z0 - 1);
  for (int f = z0 - 1; f <= z1; f += 2) {
    step(std::true_type{}, f);
    step(std::false_type{}, f + 1);
  }
}
