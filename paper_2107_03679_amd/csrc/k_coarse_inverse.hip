// The inverse of the coarsest level's operator (Alg. 2's exact solve), in complex double on the
// GPU: blocked Gauss-Jordan in place, GJ_B rows and columns per step, without pivoting, which is
// stable for the diagonally dominant rows the coarse shifted operators have (others go to the
// host's pivoted elimination).  With k the step's block:
//   P = A_kk^-1;  A_kj <- P A_kj (j != k);  A_ij -= A_ik A_kj (i, j != k);  A_ik <- -A_ik P;  A_kk <- P
// Two launches per step: the first inverts the block (every workgroup for itself) and forms
// the block row, keeping a copy of the block column; the second updates the rest.  A step's
// 32 pivots are a serial chain (0.5 us each: one element per thread, the coming pivot's row
// and column in LDS, one barrier; with four elements per thread 0.8 us), so a step takes 17 +
// 6 us up to ~500 points; at 1728 points the update's traffic counts as much.  helm_update_f
// against the host's banded elimination on 16 threads: 10^2 points (512^2) 454 -> 158 us,
// 20^2 1443 -> 369, 8^3 5034 -> 452, 12^3 95.4 -> 2.5 ms.
#include "dev_common.h"
#include "kernels.h"

namespace {

constexpr int GJ_B = 32, GJ_NT = 256, GJ_E = GJ_B * GJ_B / GJ_NT;
constexpr int GR_NT = 1024, GR_E = GJ_B * GJ_B / GR_NT;  // block row

__device__ __forceinline__ double2 dmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 dfms(double2 acc, double2 a, double2 b) {  // acc - a b
  return make_double2(fma(-a.x, b.x, fma(a.y, b.y, acc.x)), fma(-a.x, b.y, fma(-a.y, b.x, acc.y)));
}
__device__ __forceinline__ double2 dfma(double2 acc, double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, acc.x)), fma(a.x, b.y, fma(a.y, b.x, acc.y)));
}
__device__ __forceinline__ double2 drcp(double2 a) {
  // 1 / |a|^2 by two Newton steps on the hardware estimate (the pivots' serial chain)
  const double m = fma(a.x, a.x, a.y * a.y);
  double s = __builtin_amdgcn_rcp(m);
  s = fma(fma(-m, s, 1.0), s, s);
  s = fma(fma(-m, s, 1.0), s, s);
  return make_double2(a.x * s, -a.y * s);
}

// K'_l = -Lap'_l - kappa c_l as a dense matrix (the identity on the padding)
__global__ void k_gj_assemble(int dim, int nl, int NP, const c32* kc, const c32* kclo, double ghost_im, double2* A,
                              int* flag) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)NP * NP) return;
  const int N = dim == 2 ? nl * nl : nl * nl * nl;
  const int r = (int)(t / NP), q = (int)(t % NP);
  double2 v = make_double2(0.0, 0.0);
  if (r < N && q < N) {
    const Coord c = coord_of32((unsigned)r, (unsigned)nl, dim), d = coord_of32((unsigned)q, (unsigned)nl, dim);
    const int dist = abs(c.x - d.x) + abs(c.y - d.y) + abs(c.z - d.z);
    if (dist == 0) {
      const int ng = ghosts_of(c, nl, dim);
      v = make_double2(2.0 * dim - ((double)kc[r].x + kclo[r].x) - ng,
                       -((double)kc[r].y + kclo[r].y) - ng * ghost_im);
      // the off-diagonal row sum is 2 dim - ng; false for a NaN too
      const double m = hypot(v.x, v.y);
      if (!(m > 2.0 * dim - ng && isfinite(m))) *flag = 1;
    } else if (dist == 1) {
      v.x = -1.0;
    }
  } else if (r == q) {
    v.x = 1.0;
  }
  A[t] = v;
}

// Block row k (workgroup j: block column j) and the copy of block column k
__global__ __launch_bounds__(GR_NT) void k_gj_row(int NP, int k, double2* A, double2* C, double2* P) {
  __shared__ double2 sP[GJ_B][GJ_B + 1], sA[GJ_B][GJ_B + 1];
  const int j = blockIdx.x, tid = threadIdx.x, col = tid % GJ_B, row0 = tid / GJ_B;
  constexpr int RS = GR_NT / GJ_B;  // a thread's elements: (row0 + RS e, col)
  // the pivot block in registers; its row and column of the coming pivot in LDS (two of each,
  // so that one barrier separates the pivots)
  __shared__ double2 prow[2][GJ_B], pcol[2][GJ_B];
  double2 x[GR_E], own[GR_E];
  auto publish = [&](int p) {
#pragma unroll
    for (int e = 0; e < GR_E; ++e) {
      const int r = row0 + RS * e;
      if (r == p) prow[p & 1][col] = x[e];
      if (col == p) pcol[p & 1][r] = x[e];
    }
  };
#pragma unroll
  for (int e = 0; e < GR_E; ++e) {
    const int r = row0 + RS * e;
    x[e] = A[(long long)(k * GJ_B + r) * NP + k * GJ_B + col];
    sA[r][col] = A[(long long)(k * GJ_B + r) * NP + j * GJ_B + col];
    if (j != k) C[(long long)(j * GJ_B + r) * GJ_B + col] = A[(long long)(j * GJ_B + r) * NP + k * GJ_B + col];
  }
  publish(0);
  __syncthreads();
  for (int p = 0; p < GJ_B; ++p) {
    const double2 d = drcp(prow[p & 1][p]), rp = dmul(prow[p & 1][col], d);
#pragma unroll
    for (int e = 0; e < GR_E; ++e) {
      const int r = row0 + RS * e;
      const double2 f = pcol[p & 1][r];
      const double2 in = dfms(x[e], f, rp), pc = dmul(make_double2(-f.x, -f.y), d);
      const bool pr = r == p, pl = col == p;  // selected by component: a selected double2 goes through scratch memory
      x[e].x = pr ? (pl ? d.x : rp.x) : (pl ? pc.x : in.x);
      x[e].y = pr ? (pl ? d.y : rp.y) : (pl ? pc.y : in.y);
    }
    if (p + 1 < GJ_B) publish(p + 1);
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < GR_E; ++e) sP[row0 + RS * e][col] = x[e];
  __syncthreads();
  if (j == k) {
#pragma unroll
    for (int e = 0; e < GR_E; ++e) P[(row0 + RS * e) * GJ_B + col] = x[e];
    return;
  }
#pragma unroll
  for (int e = 0; e < GR_E; ++e) own[e] = make_double2(0.0, 0.0);
  for (int q = 0; q < GJ_B; ++q) {
    const double2 v = sA[q][col];
#pragma unroll
    for (int e = 0; e < GR_E; ++e) own[e] = dfma(own[e], sP[row0 + RS * e][q], v);
  }
#pragma unroll
  for (int e = 0; e < GR_E; ++e) A[(long long)(k * GJ_B + row0 + RS * e) * NP + j * GJ_B + col] = own[e];
}

// Every block outside row k
__global__ __launch_bounds__(GJ_NT) void k_gj_update(int NP, int k, double2* A, const double2* C, const double2* P) {
  __shared__ double2 sC[GJ_B][GJ_B + 1], sR[GJ_B][GJ_B + 1];
  const int j = blockIdx.x, i = blockIdx.y, tid = threadIdx.x, col = tid % GJ_B, row0 = tid / GJ_B;
  constexpr int RS = GJ_NT / GJ_B;
  if (i == k) {
    if (j == k)
#pragma unroll
      for (int e = 0; e < GJ_E; ++e)
        A[(long long)(k * GJ_B + row0 + RS * e) * NP + k * GJ_B + col] = P[(row0 + RS * e) * GJ_B + col];
    return;
  }
  double2 acc[GJ_E];
#pragma unroll
  for (int e = 0; e < GJ_E; ++e) {
    const int r = row0 + RS * e;
    sC[r][col] = C[(long long)(i * GJ_B + r) * GJ_B + col];
    const double2* src = j == k ? P + r * GJ_B + col : A + (long long)(k * GJ_B + r) * NP + j * GJ_B + col;
    sR[r][col] = *src;
    acc[e] = A[(long long)(i * GJ_B + r) * NP + j * GJ_B + col];
    if (j == k) acc[e] = make_double2(0.0, 0.0);
  }
  __syncthreads();
#pragma unroll 4
  for (int q = 0; q < GJ_B; ++q) {
    const double2 x = sR[q][col];
#pragma unroll
    for (int e = 0; e < GJ_E; ++e) acc[e] = dfms(acc[e], sC[row0 + RS * e][q], x);
  }
#pragma unroll
  for (int e = 0; e < GJ_E; ++e) A[(long long)(i * GJ_B + row0 + RS * e) * NP + j * GJ_B + col] = acc[e];
}

// minvT[k][r] = inv[r][k]; the operator is complex symmetric and so is its inverse, so the
// entries are read where they are contiguous
__global__ void k_gj_store(int N, int NP, const double2* A, c32* minvT) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)N * N) return;
  const double2 v = A[(t / N) * NP + t % N];
  minvT[t] = make_float2((float)v.x, (float)v.y);
}

int padded(int Nc) { return (Nc + GJ_B - 1) / GJ_B * GJ_B; }

}  // namespace

size_t coarse_inverse_work(int Nc) {
  const size_t NP = padded(Nc);
  return NP * NP + NP * GJ_B + GJ_B * GJ_B;
}

void launch_coarse_inverse(hipStream_t s, int dim, int nl, const c32* kc, const c32* kclo, double ghost_im,
                           double2* work, c32* minvT, int* flag) {
  const int N = dim == 2 ? nl * nl : nl * nl * nl, NP = padded(N), nb = NP / GJ_B;
  double2 *A = work, *C = A + (size_t)NP * NP, *P = C + (size_t)NP * GJ_B;
  hipLaunchKernelGGL(k_gj_assemble, dim3((unsigned)(((long long)NP * NP + 255) / 256)), dim3(256), 0, s, dim, nl, NP, kc,
                     kclo, ghost_im, A, flag);
  for (int k = 0; k < nb; ++k) {
    hipLaunchKernelGGL(k_gj_row, dim3(nb), dim3(GR_NT), 0, s, NP, k, A, C, P);
    hipLaunchKernelGGL(k_gj_update, dim3(nb, nb), dim3(GJ_NT), 0, s, NP, k, A, C, P);
  }
  hipLaunchKernelGGL(k_gj_store, dim3((unsigned)(((long long)N * N + 255) / 256)), dim3(256), 0, s, N, NP, A, minvT);
}
