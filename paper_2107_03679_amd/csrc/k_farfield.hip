// Sensor operator G~ of eq. DiscreteForward / DiscreteForwardHelm: the field
// scattered by the induced source s = f u (u the total field) on Omega,
// observed at M sensors outside Omega, by the Lippmann-Schwinger integral
// (eq. LSIntegral) with the free-space Green's function (eq. green) and the
// rectangle rule on the grid:
//     y_m = sum_{z in Omega} g(x_m - z) s(z) h^d,
//     g(x) = (j/4) H0^(1)(k_b |x|)  (2D),   e^{j k_b |x|} / (4 pi |x|)  (3D).
// G~ [M][n^dim] is formed once per sensor set (2D: H0^(1) by cubic Hermite
// interpolation in a host FP64 table of H0^(1) and its derivative; 3D: in
// closed form in FP64), then applied as a split-K product and its adjoint, both on the FP32
// matrix cores (v_mfma_f32_16x16x4_f32, whose operands and sums are single precision): lane
// (i16, g) = (l % 16, l / 16) gives row i16 of A and column i16 of B at k = g and holds rows
// 4 g .. 4 g + 3 of column i16 of D.  A complex product is four real ones.
#include <algorithm>

#include "dev_common.h"
#include "kernels.h"

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
// 16 bytes at the 8-byte alignment of a complex field with rows of odd length
typedef f32x4 f32x4_a8 __attribute__((aligned(8)));

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__global__ void k_ff_matrix(int dim, int n, int M, const double* sens, double kbh, double h, const double2* tab,
                            double x0, double dx, int ntab, c32* G) {
  const long long Ni = dim == 2 ? (long long)n * n : (long long)n * n * n;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int m = blockIdx.y;
  if (i >= Ni || m >= M) return;
  const Coord c = coord_of32((unsigned)i, (unsigned)n, dim);
  const double ctr = 0.5 * (n - 1);
  const double ddx = sens[m * dim + 0] - (c.x - ctr), ddy = sens[m * dim + 1] - (c.y - ctr);
  const double ddz = dim == 3 ? sens[m * dim + 2] - (c.z - ctr) : 0.0;
  const double r = sqrt(ddx * ddx + ddy * ddy + ddz * ddz);  // in cells
  double gr, gi;
  if (dim == 2) {
    // H0(x) on the table: value/derivative pairs (tab[2k], tab[2k+1]) at x0 + k dx
    const double x = kbh * r;
    double t = (x - x0) / dx;
    int k = (int)floor(t);
    k = k < 0 ? 0 : (k > ntab - 2 ? ntab - 2 : k);
    t -= k;
    const double h00 = (1 + 2 * t) * (1 - t) * (1 - t), h10 = t * (1 - t) * (1 - t);
    const double h01 = t * t * (3 - 2 * t), h11 = t * t * (t - 1);
    const double2 v0 = tab[2 * k], d0 = tab[2 * k + 1], v1 = tab[2 * k + 2], d1 = tab[2 * k + 3];
    const double hr = h00 * v0.x + h10 * dx * d0.x + h01 * v1.x + h11 * dx * d1.x;
    const double hi = h00 * v0.y + h10 * dx * d0.y + h01 * v1.y + h11 * dx * d1.y;
    // (j/4) H0 = (-Im H0 + j Re H0) / 4, times the cell area h^2
    gr = -0.25 * hi * h * h;
    gi = 0.25 * hr * h * h;
  } else {
    const double rr = r * h, kb = kbh / h;
    double sn, cs;
    sincos(kb * rr, &sn, &cs);
    const double a = h * h * h / (4.0 * 3.14159265358979323846 * rr);
    gr = a * cs;
    gi = a * sn;
  }
  G[(long long)m * Ni + i] = make_float2((float)gr, (float)gi);
}

// s[b][i] = f_i (u_in + u_sc)[b][p(i)] on Omega (compact [B][n^dim])
__global__ void k_ff_source(int dim, int B, int ne, int w, int n, const float* fpl, const c32* uin, const c32* usc,
                            c32* s) {
  const long long Ni = dim == 2 ? (long long)n * n : (long long)n * n * n;
  const long long Ne = dim == 2 ? (long long)ne * ne : (long long)ne * ne * ne;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = blockIdx.y;
  if (i >= Ni) return;
  const Coord c = coord_of32((unsigned)i, (unsigned)n, dim);
  const long long p = dim == 2 ? (long long)(c.y + w) * ne + (c.x + w)
                               : ((long long)(c.z + w) * ne + (c.y + w)) * ne + (c.x + w);
  c32 u = usc[(long long)b * Ne + p];
  if (uin) u = cadd(u, uin[(long long)b * Ne + p]);
  s[(long long)b * Ni + i] = cscale(u, fpl[p]);
}

// part[k][b][m] = sum over pixel chunk k of G[m][i] s[b][i].  A wavefront takes 16 sensors and
// 16 BT right-hand sides, so that G, the large operand, is read once for up to 64 right-hand
// sides: lane group g loads pixels 8 g .. 8 g + 7 of every 32 (64 bytes a lane, 256 a row), the
// next 32 in flight meanwhile.  Bound by the FP32 rate (16 n^d B M operations) and G's 8 M
// bytes per pixel.  180 sensors, 32 right-hand sides, 256^2: 167 us with 32 x 32 LDS tiles on
// the vector units, which read five LDS values for four products, 44 us now (the matrix cores'
// share 20).
struct Px8 {
  c32 v[8];
};
__device__ __forceinline__ Px8 load_px8(const c32* row, long long i, long long i1) {
  Px8 o;
  if (i + 8 <= i1) {
    const f32x4_a8* q = reinterpret_cast<const f32x4_a8*>(row + i);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const f32x4 t = q[u];
      o.v[2 * u] = make_float2(t[0], t[1]);
      o.v[2 * u + 1] = make_float2(t[2], t[3]);
    }
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      o.v[u] = make_float2(0.f, 0.f);
      if (i + u < i1) o.v[u] = row[i + u];
    }
  }
  return o;
}

template <int BT>
__global__ __launch_bounds__(256) void k_ff_apply(int B, int M, long long Ni, long long chunk, const c32* G,
                                                   const c32* s, c32* part) {
  const int lane = threadIdx.x % 64, i16 = lane % 16, g = lane / 16;
  const int m0 = (blockIdx.x * 4 + threadIdx.x / 64) * 16, k = blockIdx.y, b0 = blockIdx.z * 16 * BT;
  if (m0 >= M) return;
  const long long i0 = (long long)k * chunk, i1 = min(i0 + chunk, Ni);
  // rows past the last sensor or right-hand side repeat it; their sums are not stored
  const c32* gr = G + (long long)min(m0 + i16, M - 1) * Ni;
  const c32* sr[BT];
#pragma unroll
  for (int t = 0; t < BT; ++t) sr[t] = s + (long long)min(b0 + 16 * t + i16, B - 1) * Ni;
  f32x4 re[BT], im[BT];
#pragma unroll
  for (int t = 0; t < BT; ++t) re[t] = im[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  Px8 gn = load_px8(gr, i0 + 8 * g, i1), sn[BT];
#pragma unroll
  for (int t = 0; t < BT; ++t) sn[t] = load_px8(sr[t], i0 + 8 * g, i1);
  for (long long ib = i0; ib < i1; ib += 32) {
    const Px8 gv = gn;
    Px8 sv[BT];
#pragma unroll
    for (int t = 0; t < BT; ++t) sv[t] = sn[t];
    if (ib + 32 < i1) {
      gn = load_px8(gr, ib + 32 + 8 * g, i1);
#pragma unroll
      for (int t = 0; t < BT; ++t) sn[t] = load_px8(sr[t], ib + 32 + 8 * g, i1);
    }
#pragma unroll
    for (int v = 0; v < 8; ++v)
#pragma unroll
      for (int t = 0; t < BT; ++t) {
        re[t] = mfma4(gv.v[v].x, sv[t].v[v].x, re[t]);
        im[t] = mfma4(gv.v[v].x, sv[t].v[v].y, im[t]);
        re[t] = mfma4(-gv.v[v].y, sv[t].v[v].y, re[t]);
        im[t] = mfma4(gv.v[v].y, sv[t].v[v].x, im[t]);
      }
  }
#pragma unroll
  for (int t = 0; t < BT; ++t) {
    const int b = b0 + 16 * t + i16;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + 4 * g + r;
      if (b < B && m < M) part[((long long)k * B + b) * M + m] = make_float2(re[t][r], im[t][r]);
    }
  }
}

// y[b][m] = sum over chunks (fixed order: four threads take every fourth chunk, eight loads in
// flight)
__global__ __launch_bounds__(256) void k_ff_reduce(int count, int nsplit, const c32* part, c32* y) {
  __shared__ c32 red[4][64];
  const int e = threadIdx.x % 64, q = threadIdx.x / 64, t = blockIdx.x * 64 + e;
  c32 a = make_float2(0.f, 0.f);
  if (t < count) {
    int k = q;
    for (; k + 28 < nsplit; k += 32) {
      c32 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(long long)(k + 4 * u) * count + t];
#pragma unroll
      for (int u = 0; u < 8; ++u) a = cadd(a, v[u]);
    }
    for (; k < nsplit; k += 4) a = cadd(a, part[(long long)k * count + t]);
  }
  red[q][e] = a;
  __syncthreads();
  if (q == 0 && t < count) y[t] = cadd(cadd(red[0][e], red[1][e]), cadd(red[2][e], red[3][e]));
}

// s_ext[b][p(i)] = sum_m conj(G[m][i]) r[b][m] on Omega, rhs_ext = f s_ext (the layer is zeroed by
// k_ff_zero_layer).  A wavefront takes 32 pixels (two A tiles: lane i16's are 2 i16 and 2 i16 + 1,
// 16 bytes) and 16 BT right-hand sides, G is read once for them, four steps of four sensors
// ahead; r passes through LDS, FA_M sensors at a time, [sensor][right-hand side].  The two
// products of each part have sums of their own (half the chain of rounding).  180 sensors, 32
// right-hand sides, 256^2: 84 us with LDS tiles on the vector units, 44 us now; 82 with every
// lane storing its own eight pixels (64 lines per store) instead of through LDS.
constexpr int FA_M = 128, FA_P = 128;  // sensors per pass, pixels per block
template <int BT>
__global__ __launch_bounds__(256) void k_ff_adjoint(int dim, int B, int M, int ne, int w, int n, const c32* G,
                                                     const c32* r, const float* fpl, c32* s_ext, c32* rhs_ext) {
  constexpr int BW = 16 * BT, U = 4;
  static_assert(FA_M == FA_P, "one buffer for the sensors' values and the pixels' results");
  __shared__ c32 buf[BW * (FA_P + 1) > FA_M * (BW + 1) ? BW * (FA_P + 1) : FA_M * (BW + 1)];
  c32(*sr)[BW + 1] = reinterpret_cast<c32(*)[BW + 1]>(buf);
  const int tid = threadIdx.x, lane = tid % 64, i16 = lane % 16, g = lane / 16, b0 = blockIdx.y * BW;
  const long long Ni = dim == 2 ? (long long)n * n : (long long)n * n * n;
  const long long Ne = dim == 2 ? (long long)ne * ne : (long long)ne * ne * ne;
  const long long i0 = ((long long)blockIdx.x * 4 + tid / 64) * 32;
  // pairs past the last pixel start there (G has one entry more than its rows), and what they
  // add to is not stored
  const c32* gp = G + min(i0 + 2 * i16, Ni - 1);
  f32x4 re[2][2][BT], im[2][2][BT];  // [x or y of G][pixel tile][right-hand sides]
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int t = 0; t < BT; ++t) re[h][q][t] = im[h][q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 gn[U];
  auto fetch = [&](int m0) {  // U steps from sensor m0 (past the last sensor: the last one, r is zero there)
#pragma unroll
    for (int u = 0; u < U; ++u)
      gn[u] = *reinterpret_cast<const f32x4_a8*>(gp + (long long)min(m0 + 4 * u + g, M - 1) * Ni);
  };
  fetch(0);
  for (int mb = 0; mb < M; mb += FA_M) {
    __syncthreads();
    for (int q = tid; q < FA_M * BW; q += 256) {
      const int m = q % FA_M, b = q / FA_M;
      sr[m][b] = mb + m < M && b0 + b < B ? r[(long long)(b0 + b) * M + mb + m] : make_float2(0.f, 0.f);
    }
    __syncthreads();
    const int mend = min(FA_M, M - mb);
    for (int m = 0; m < mend; m += 4 * U) {
      f32x4 gv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) gv[u] = gn[u];
      if (mb + m + 4 * U < M) fetch(mb + m + 4 * U);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        c32 rv[BT];
#pragma unroll
        for (int t = 0; t < BT; ++t) rv[t] = sr[m + 4 * u + g][16 * t + i16];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int t = 0; t < BT; ++t) {
            re[0][q][t] = mfma4(gv[u][2 * q], rv[t].x, re[0][q][t]);
            im[0][q][t] = mfma4(gv[u][2 * q], rv[t].y, im[0][q][t]);
            re[1][q][t] = mfma4(gv[u][2 * q + 1], rv[t].y, re[1][q][t]);
            im[1][q][t] = mfma4(gv[u][2 * q + 1], rv[t].x, im[1][q][t]);
          }
      }
    }
  }
  // through LDS, so that a wavefront stores 64 consecutive pixels of one right-hand side
  c32(*out)[FA_P + 1] = reinterpret_cast<c32(*)[FA_P + 1]>(buf);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int t = 0; t < BT; ++t)
        out[16 * t + i16][(tid / 64) * 32 + 2 * (4 * g + c) + o] =
            make_float2(re[0][o][t][c] + re[1][o][t][c], im[0][o][t][c] - im[1][o][t][c]);
  __syncthreads();
  const int px = tid % FA_P;
  const long long i = (long long)blockIdx.x * FA_P + px;
  if (i >= Ni) return;
  const Coord x = coord_of32((unsigned)i, (unsigned)n, dim);
  const long long p = dim == 2 ? (long long)(x.y + w) * ne + (x.x + w)
                               : ((long long)(x.z + w) * ne + (x.y + w)) * ne + (x.x + w);
  const float f = rhs_ext ? fpl[p] : 0.f;
  for (int b = tid / FA_P; b < BW && b0 + b < B; b += 256 / FA_P) {
    const c32 v = out[b][px];
    s_ext[(long long)(b0 + b) * Ne + p] = v;
    if (rhs_ext) rhs_ext[(long long)(b0 + b) * Ne + p] = cscale(v, f);
  }
}

// zeros outside Omega
__global__ void k_ff_zero_layer(int dim, int B, int ne, int w, int n, long long Ne, c32* s_ext, c32* rhs_ext) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int b = batch_index();
  if (p >= Ne || b >= B) return;
  const Coord c = coord_of32((unsigned)p, (unsigned)ne, dim);
  const bool in = c.x >= w && c.x < w + n && c.y >= w && c.y < w + n && (dim == 2 || (c.z >= w && c.z < w + n));
  if (in) return;
  const long long t = b * Ne + p;
  s_ext[t] = make_float2(0.f, 0.f);
  if (rhs_ext) rhs_ext[t] = make_float2(0.f, 0.f);
}

inline unsigned nb(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

void launch_ff_matrix(hipStream_t s, int dim, int n, int M, const double* sens, double kbh, double h,
                      const double2* tab, double x0, double dx, int ntab, c32* G) {
  const long long Ni = dim == 2 ? (long long)n * n : (long long)n * n * n;
  hipLaunchKernelGGL(k_ff_matrix, dim3(nb(Ni, 256), M), dim3(256), 0, s, dim, n, M, sens, kbh, h, tab, x0, dx, ntab,
                     G);
}

// Pixel chunks of the sensor product: between `least`, 64 of at least 1024 pixels (no FP32 sum runs
// over more than a 64th of a large grid), and `most`, 256 of at least 256.
struct FfChunks {
  long long least, most;
};
static FfChunks ff_chunks(long long Ni) {
  return {std::min(std::max(Ni / 1024, 1LL), 64LL), std::min(std::max(Ni / 256, 1LL), 256LL)};
}
constexpr long long FF_WAVES = 2048;  // two wavefronts per SIMD

// Partial sums per right-hand side for any number of sensors up to M (the chunks that
// launch_ff_forward wants times the sensors are at most FF_WAVES 16)
size_t ff_part_size(long long Ni, int M) {
  const FfChunks c = ff_chunks(Ni);
  return (size_t)std::max(c.least * M, std::min(c.most * M, FF_WAVES * 16));
}

void launch_ff_forward(hipStream_t s, int dim, int B, int M, int ne, int w, int n, const float* fpl, const c32* uin,
                       const c32* usc, const c32* G, c32* src, c32* part, c32* y) {
  const long long Ni = dim == 2 ? (long long)n * n : (long long)n * n * n;
  hipLaunchKernelGGL(k_ff_source, dim3(nb(Ni, 256), B), dim3(256), 0, s, dim, B, ne, w, n, fpl, uin, usc, src);
  // Chunks for FF_WAVES wavefronts over the sensor tiles (up to 64 right-hand sides are one tile of
  // them).  From the pixels and the sensors alone: with the right-hand sides counted too, a source
  // had other last bits in a batch of 65.
  const FfChunks c = ff_chunks(Ni);
  const long long ns = std::max(c.least, std::min(c.most, FF_WAVES / nb(M, 16)));
  const long long chunk = ((Ni + ns - 1) / ns + 31) / 32 * 32;
  const int used = (int)((Ni + chunk - 1) / chunk);
  auto apply = [&](auto kernel, int bt) {
    hipLaunchKernelGGL(kernel, dim3(nb(M, 64), used, nb(B, 16 * bt)), dim3(256), 0, s, B, M, Ni, chunk, G, src, part);
  };
  if (B <= 16) apply(k_ff_apply<1>, 1);
  else if (B <= 32) apply(k_ff_apply<2>, 2);
  else apply(k_ff_apply<4>, 4);
  hipLaunchKernelGGL(k_ff_reduce, dim3(nb((long long)B * M, 64)), dim3(256), 0, s, B * M, used, part, y);
}

void launch_ff_adjoint(hipStream_t s, int dim, int B, int M, int ne, int w, int n, const c32* G, const c32* r,
                       const float* fpl, c32* s_ext, c32* rhs_ext) {
  const long long Ni = dim == 2 ? (long long)n * n : (long long)n * n * n;
  const long long Ne = dim == 2 ? (long long)ne * ne : (long long)ne * ne * ne;
  hipLaunchKernelGGL(k_ff_zero_layer, batch_grid(nb(Ne, 256), B), dim3(256), 0, s, dim, B, ne, w, n, Ne, s_ext, rhs_ext);
  auto adjoint = [&](auto kernel, int bt) {
    hipLaunchKernelGGL(kernel, dim3(nb(Ni, FA_P), nb(B, 16 * bt)), dim3(256), 0, s, dim, B, M, ne, w, n, G, r, fpl, s_ext,
                       rhs_ext);
  };
  if (B <= 16) adjoint(k_ff_adjoint<1>, 1);
  else adjoint(k_ff_adjoint<2>, 2);
}
