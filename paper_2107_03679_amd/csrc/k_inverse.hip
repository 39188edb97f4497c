// Inverse-problem steps of Sec. V on the interior grid Omega (n^dim points,
// x fastest): the TV proximal operator with a lower bound (eq. proximalOpt),
// computed by fast gradient projection on its dual, the update of the
// accelerated forward-backward splitting (Alg. 4), the data residual of the
// quadratic fidelity term, and the medium from the scattering potential.
//
// TV(w) = sum_i ||(D w)_i||, (D w)_{a,i} = w_{i+e_a} - w_i (0 across the last
// index of axis a).  Dual field p: dim components per point, ||p_i|| <= 1.
// One FGP step (t the Nesterov sequence, beta = (t - 1) / t'):
//   w = max(v - lam D^T r, lo)
//   q = P_B(r + D w / (4 dim lam));  r = q + beta (q - p);  p = q
// and the answer is max(v - lam D^T p, lo): k_fgp_block, several steps per launch.
#include <algorithm>
#include <cmath>

#include "dev_common.h"
#include "kernels.h"

namespace {

__device__ __forceinline__ long long axis_stride(int a, int n) {
  return a == 0 ? 1LL : (a == 1 ? (long long)n : (long long)n * n);
}
__device__ __forceinline__ int coord_a(const Coord& c, int a) { return a == 0 ? c.x : (a == 1 ? c.y : c.z); }

// w = max(v - lam D^T r, lo); (D^T r)_i = sum_a (r_{a, i - e_a} [i_a > 0] - r_{a,i} [i_a < n - 1])
__global__ void k_fgp_primal(int dim, int n, long long Ni, const float* v, const float* r, float lam, float lo,
                             float* w) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < Ni; i += (long long)gridDim.x * blockDim.x) {
    const Coord c = coord_of32((unsigned)i, (unsigned)n, dim);
    float dt = 0.f;
    for (int a = 0; a < dim; ++a) {
      const float* ra = r + (long long)a * Ni;
      const int ca = coord_a(c, a);
      if (ca > 0) dt += ra[i - axis_stride(a, n)];
      if (ca < n - 1) dt -= ra[i];
    }
    w[i] = fmaxf(v[i] - lam * dt, lo);
  }
}

// Several FGP steps of a region in LDS.  A step reads one neighbour each way, so a launch of
// `units` steps on a region of 64 x 64 (3D: 16^3 or 32 x 16 x 16) points gives the region
// `halo` >= units points on each side (launch_tv_prox chooses it); points nearer the region's
// edge hold values that no kept point reads.  p, v and this point's r, w stay in registers,
// r and w for the neighbours in LDS.  The state (p, r) alternates between two buffers from
// launch to launch, since neighbouring regions read the old one.  A grid that fits one region
// needs no halo and takes up to FGP_MAXU steps per launch.  With a pair of kernels per step
// the prox at 512^2 was 100 launches of about 4 us, half of it the launch, on data that fits
// the L2.  A step is bound by instruction issue (4096 or 8192 points on one CU), so the
// neighbours are read without branches and the projection's scale is rsqrt(|q|^2) (1 ulp; a
// root and a division before): 2.0 -> 0.75 us per step of 4096 points.  One forward-backward
// update with 50 steps: 512^2 487 -> 99 us, 64^2 417 -> 58, 1024^2 with 100 steps 1655 ->
// 293, 48^3 499 -> 177, 128^3 1722 -> 1283.
constexpr int FGP_NT = 1024, FGP_MAXU = 64;
struct FgpArgs {
  int n, halo;
  int tile[2], tiles[2];     // kept points and regions along x, and along the other axes; a region
                             // starts at tile * index - halo
  long long Ni;
  const float* v;            // prox input; or nullptr: v = fbar - gamma grad, stored to vout
  const float *fbar, *grad;
  float gamma;
  float* vout;
  float lam, lo, step;
  const float *p0, *r0;      // state read (first launch: zero) ...
  float *p1, *r1;            // ... and written (not by the last launch)
  int first, last, units;    // dual steps of this launch
  float* w;                  // last launch: the answer; or with f: f, fbar updated (Alg. 4's momentum)
  float *f, *fb;
  float mbeta;
  float beta[FGP_MAXU];
};

template <int DIM, int RX>
__global__ __launch_bounds__(FGP_NT) void k_fgp_block(FgpArgs a) {
  constexpr int RY = DIM == 2 ? 64 : 16, RZ = DIM == 2 ? 1 : 16, RN = RX * RY * RZ, FGP_NP = RN / FGP_NT;
  static_assert(RN == FGP_NT * FGP_NP, "points of a region");
  __shared__ float sR[DIM][RN];
  __shared__ float sW[RN];
  const int n = a.n, tid = threadIdx.x;
  const int bx = blockIdx.x % a.tiles[0], bt = blockIdx.x / a.tiles[0], by = bt % a.tiles[1], bz = bt / a.tiles[1];
  const int gx0 = bx * a.tile[0] - a.halo, gy0 = by * a.tile[1] - a.halo, gz0 = bz * a.tile[1] - a.halo;
  constexpr int ST[3] = {1, RX, RX * RY};  // LDS stride per axis
  // point i of this thread: region index tid + i FGP_NT
  long long g[FGP_NP];
  bool keep[FGP_NP], lo_in[FGP_NP][DIM], hi_in[FGP_NP][DIM];  // neighbours inside the grid
  float v[FGP_NP], pv[FGP_NP][DIM], rv[FGP_NP][DIM];
#pragma unroll
  for (int i = 0; i < FGP_NP; ++i) {
    const int q = tid + i * FGP_NT;
    const int lx = q % RX, ly = q / RX % RY, lz = DIM == 3 ? q / (RX * RY) : 0;
    int c[DIM];
    c[0] = gx0 + lx;
    c[1] = gy0 + ly;
    if (DIM == 3) c[DIM - 1] = gz0 + lz;
    keep[i] = lx >= a.halo && lx < a.halo + a.tile[0] && ly >= a.halo && ly < a.halo + a.tile[1] &&
              (DIM == 2 || (lz >= a.halo && lz < a.halo + a.tile[1]));
    g[i] = 0;
#pragma unroll
    for (int d = DIM - 1; d >= 0; --d) {
      keep[i] = keep[i] && c[d] < n;
      g[i] = g[i] * n + min(max(c[d], 0), n - 1);  // the nearest point of the grid
    }
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      lo_in[i][d] = c[d] > 0;
      hi_in[i][d] = c[d] < n - 1;
      pv[i][d] = rv[i][d] = 0.f;
    }
  }
  if (a.v) {
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i) v[i] = a.v[g[i]];
  } else {
    float gr[FGP_NP];
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i) {
      v[i] = a.fbar[g[i]];
      gr[i] = a.grad[g[i]];
    }
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i) v[i] = fmaf(-a.gamma, gr[i], v[i]);
  }
  if (!a.first) {
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i)
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        pv[i][d] = a.p0[d * a.Ni + g[i]];
        rv[i][d] = a.r0[d * a.Ni + g[i]];
      }
  }
#pragma unroll
  for (int i = 0; i < FGP_NP; ++i)
#pragma unroll
    for (int d = 0; d < DIM; ++d) sR[d][tid + i * FGP_NT] = rv[i][d];
  if (a.vout) {
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i)
      if (keep[i]) a.vout[g[i]] = v[i];
  }
  __syncthreads();
  // max(v - lam D^T r, lo) at point i from r in LDS (own values in registers)
  auto primal = [&](int i, const float (&own)[DIM]) {
    const int q = tid + i * FGP_NT;
    float dt = 0.f;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const float low = sR[d][max(q - ST[d], 0)];  // read without a branch, used inside the grid
      dt += lo_in[i][d] ? low : 0.f;
      dt -= hi_in[i][d] ? own[d] : 0.f;
    }
    return fmaxf(v[i] - a.lam * dt, a.lo);
  };
  for (int u = 0; u < a.units; ++u) {
    const float beta = a.beta[u];
    float w[FGP_NP];
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i) {
      w[i] = primal(i, rv[i]);
      sW[tid + i * FGP_NT] = w[i];
    }
    __syncthreads();
    float high[FGP_NP][DIM];  // read back to back: a read under hi_in would wait by itself
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i)
#pragma unroll
      for (int d = 0; d < DIM; ++d) high[i][d] = sW[min(tid + i * FGP_NT + ST[d], RN - 1)];
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i)
#pragma unroll
      for (int d = 0; d < DIM; ++d) asm volatile("" : "+v"(high[i][d]));
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i) {
      const int q = tid + i * FGP_NT;
      float qd[DIM], nn = 0.f;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const float gr = hi_in[i][d] ? high[i][d] - w[i] : 0.f;
        qd[d] = fmaf(a.step, gr, rv[i][d]);
        nn = fmaf(qd[d], qd[d], nn);
      }
      const float sc = nn > 1.0f ? rsqrtf(nn) : 1.0f;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const float qa = qd[d] * sc;
        rv[i][d] = fmaf(beta, qa - pv[i][d], qa);
        pv[i][d] = qa;
        sR[d][q] = rv[i][d];
      }
    }
    __syncthreads();
  }
  if (!a.last) {
#pragma unroll
    for (int i = 0; i < FGP_NP; ++i) {
      if (!keep[i]) continue;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        a.p1[d * a.Ni + g[i]] = pv[i][d];
        a.r1[d * a.Ni + g[i]] = rv[i][d];
      }
    }
    return;
  }
  // the answer, from p
#pragma unroll
  for (int i = 0; i < FGP_NP; ++i)
#pragma unroll
    for (int d = 0; d < DIM; ++d) sR[d][tid + i * FGP_NT] = pv[i][d];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < FGP_NP; ++i) {
    const float w = primal(i, pv[i]);
    if (!keep[i]) continue;
    if (a.f) {
      a.fb[g[i]] = fmaf(a.mbeta, w - a.f[g[i]], w);
      a.f[g[i]] = w;
    } else {
      a.w[g[i]] = w;
    }
  }
}

__global__ void k_fill(long long count, float val, float* x) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
    x[i] = val;
}

// out = a - s * b
__global__ void k_axmy(long long count, const float* a, float s, const float* b, float* out) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
    out[i] = fmaf(-s, b[i], a[i]);
}

// fbar = f_new + beta (f_new - f);  f = f_new
__global__ void k_fbs_momentum(long long count, const float* f_new, float beta, float* f, float* fbar) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x) {
    const float fn = f_new[i];
    fbar[i] = fmaf(beta, fn - f[i], fn);
    f[i] = fn;
  }
}

// res[q][i] = u[q][idx[i]] - y[q][i];  per-block partial sums of |res|^2 (FP64)
__global__ void k_data_residual(int B, int M, long long N, const int* idx, const c32* u, const c32* y, c32* res,
                                double* part) {
  __shared__ double red[256 / HELM_WAVE];
  double s = 0.0;
  const long long T = (long long)B * M;
  for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < T; t += (long long)gridDim.x * blockDim.x) {
    const int q = (int)(t / M), i = (int)(t - (long long)q * M);
    const c32 d = csub(u[(long long)q * N + idx[i]], y[t]);
    res[t] = d;
    s += (double)d.x * d.x + (double)d.y * d.y;
  }
  s = wave_sum_d(s);
  if (threadIdx.x % HELM_WAVE == 0) red[threadIdx.x / HELM_WAVE] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < 256 / HELM_WAVE; ++q) t += red[q];
    part[blockIdx.x] = t;
  }
}

// n = sqrt(n_b^2 + f / k0^2) (f >= -k0^2 n_b^2 is clamped to n = 0)
__global__ void k_index_from_f(long long count, const float* f, double inv_k02, double nb2, float* nmap) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x)
    nmap[i] = (float)sqrt(fmax(0.0, nb2 + (double)f[i] * inv_k02));
}

inline unsigned grid_of(long long n) {
  const long long g = (n + 255) / 256;
  return (unsigned)(g < 4096 ? (g > 0 ? g : 1) : 4096);
}

}  // namespace

// The launches of `iters` FGP steps: `steps of every launch` + the final primal step (one unit)
// in chunks of the halo (a whole grid in one region: FGP_MAXU).  fm: Alg. 4's update (see
// FbsArgs) around the prox, in its first and last launch.
void launch_tv_prox(hipStream_t s, int dim, int n, const float* v, float lam, float lo, int iters, const FgpBufs& bufs,
                    float* w, const FbsArgs* fm) {
  const long long Ni = dim == 2 ? (long long)n * n : (long long)n * n * n;
  const unsigned g = grid_of(Ni);
  const int region = dim == 2 ? 64 : 16;
  // One region where the grid fits it.  Else the halo trades repeated points for launches of
  // about 6 us plus their steps: while every region runs at once the larger halo wins, beyond
  // that the repeated points count (50 steps, us; 16^3 regions with halo 2 / 3 / 4, then 32 x
  // 16 x 16 ones: 48^3 292 229 177, 362 288 246; 64^3 333 352 303, 419 319 262; 96^3 751 829
  // 970, 596 640 707; 128^3 1789 1812 2514, 1477 1283 1470).
  const bool whole = n <= region, wide = dim == 3 && n > 48;
  const int halo = whole ? 0 : (dim == 2 ? 8 : (n <= 72 ? 4 : 3)), chunk = whole ? FGP_MAXU : halo;
  const bool prox = lam > 0.0f && iters > 0;
  // several regions in one launch: its momentum would overwrite fbar under the neighbours' loads of v
  const bool fused = fm && prox && (whole || iters + 1 > chunk);
  if (fm && !fused) {
    hipLaunchKernelGGL(k_axmy, dim3(g), dim3(256), 0, s, Ni, fm->fbar, fm->gamma, fm->grad, bufs.v);
    v = bufs.v;
    w = bufs.w;
  }
  if (!prox) {
    hipLaunchKernelGGL(k_fill, dim3(g), dim3(256), 0, s, (long long)dim * Ni, 0.0f, bufs.p[0]);
    hipLaunchKernelGGL(k_fgp_primal, dim3(g), dim3(256), 0, s, dim, n, Ni, v, bufs.p[0], 0.0f, lo, w);
  } else {
    FgpArgs a{};
    a.n = n;
    a.halo = halo;
    a.tile[0] = whole ? n : (wide ? 32 : region) - 2 * halo;
    a.tile[1] = whole ? n : region - 2 * halo;
    for (int q = 0; q < 2; ++q) a.tiles[q] = (n + a.tile[q] - 1) / a.tile[q];
    a.Ni = Ni;
    a.lam = lam;
    a.lo = lo;
    a.step = 1.0f / (4.0f * dim * lam);
    a.w = w;
    const unsigned blocks = (unsigned)(a.tiles[0] * a.tiles[1] * (dim == 3 ? a.tiles[1] : 1));
    double t = 1.0;
    for (int done = 0, k = 0;; ++k) {
      a.units = std::min(chunk, iters - done);
      a.first = k == 0;
      a.last = done + a.units == iters && a.units < chunk;  // room for the final primal step
      if (whole && done + a.units == iters) a.last = 1;
      a.v = v;
      a.vout = nullptr;
      a.f = a.fb = nullptr;
      if (fused) {
        a.v = a.first ? nullptr : bufs.v;
        a.fbar = fm->fbar;
        a.grad = fm->grad;
        a.gamma = fm->gamma;
        if (a.first && !a.last) a.vout = bufs.v;
        if (a.last) {
          a.f = fm->f;
          a.fb = fm->fbar;
          a.mbeta = fm->beta;
        }
      }
      a.p0 = bufs.p[k & 1];
      a.r0 = bufs.r[k & 1];
      a.p1 = bufs.p[(k + 1) & 1];
      a.r1 = bufs.r[(k + 1) & 1];
      for (int u = 0; u < a.units; ++u) {
        const double tn = 0.5 * (1.0 + std::sqrt(1.0 + 4.0 * t * t));
        a.beta[u] = (float)((t - 1.0) / tn);
        t = tn;
      }
      if (dim == 2) hipLaunchKernelGGL((k_fgp_block<2, 64>), dim3(blocks), dim3(FGP_NT), 0, s, a);
      else if (wide) hipLaunchKernelGGL((k_fgp_block<3, 32>), dim3(blocks), dim3(FGP_NT), 0, s, a);
      else hipLaunchKernelGGL((k_fgp_block<3, 16>), dim3(blocks), dim3(FGP_NT), 0, s, a);
      done += a.units;
      if (a.last) break;
    }
  }
  if (fm && !fused)
    hipLaunchKernelGGL(k_fbs_momentum, dim3(g), dim3(256), 0, s, Ni, w, fm->beta, fm->f, fm->fbar);
}

namespace {
// per-block partial sums of x[i]^2 (FP64), grid-stride
__global__ void k_sumsq(long long n, const float* x, double* part) {
  __shared__ double red[256 / HELM_WAVE];
  double s = 0.0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    s += (double)x[i] * x[i];
  s = wave_sum_d(s);
  if (threadIdx.x % HELM_WAVE == 0) red[threadIdx.x / HELM_WAVE] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < 256 / HELM_WAVE; ++q) t += red[q];
    part[blockIdx.x] = t;
  }
}

__global__ void k_scale(long long n, float* x, float a) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    x[i] *= a;
}
}  // namespace

int sumsq_blocks(long long n) { return (int)grid_of(n); }
void launch_sumsq(hipStream_t s, long long n, const float* x, double* part) {
  hipLaunchKernelGGL(k_sumsq, dim3(sumsq_blocks(n)), dim3(256), 0, s, n, x, part);
}
void launch_scale(hipStream_t s, long long n, float* x, float a) {
  hipLaunchKernelGGL(k_scale, dim3(grid_of(n)), dim3(256), 0, s, n, x, a);
}

int data_residual_blocks(int B, int M) { return (int)grid_of((long long)B * M); }

void launch_data_residual(hipStream_t s, int B, int M, long long N, const int* idx, const c32* u, const c32* y,
                          c32* res, double* part) {
  hipLaunchKernelGGL(k_data_residual, dim3(data_residual_blocks(B, M)), dim3(256), 0, s, B, M, N, idx, u, y, res,
                     part);
}

void launch_index_from_f(hipStream_t s, long long count, const float* f, double inv_k02, double nb2, float* nmap) {
  hipLaunchKernelGGL(k_index_from_f, dim3(grid_of(count)), dim3(256), 0, s, count, f, inv_k02, nb2, nmap);
}
