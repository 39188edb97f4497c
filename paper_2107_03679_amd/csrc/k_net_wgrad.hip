// Weight and bias gradients of the network's convolutions (BF16 operands, FP32 accumulation,
// v_mfma_f32_16x16x32_bf16): dW[co][tap cin + ci] = sum_p in[p + shift(tap)][ci] g[p][co], a
// product over pixels, db[co] = sum_p g[p][co].
//
// A block takes TH x 32 pixels of one plane at a time: the input's halo tile (its CG tiles of
// 16 channels) and the gradient's tile are staged in LDS pixel by pixel, as they lie in
// memory, and read transposed (ds_read_b64_tr_b16: a lane gets its channel of four pixels), so
// that a tap's shift is an address.  A wavefront owns one input-channel tile, all output
// channels (NCO tiles) and the nine in-plane taps: 9 NCO accumulators, the three halo rows of
// the current pixel row in registers (one row read per pixel row).  With fewer than four
// channel tiles the wavefronts share the rows and their sums are added in LDS at the end.  In
// 3D a block takes one tap plane (grid.z).  The channel tiles beyond CG are grid.y.  A block
// walks several tiles, then writes its partial sums; one launch adds the partials of every
// layer in a fixed order.
// (Fetching both operands element by element for every (16 k-values, 16 channels) tile, the
// weight gradients were 1.35 of the 2.42 ms of a training step on 4 images of 256^2, the
// biases' sums and the 16 reductions 0.25 ms; they are 0.13 and 0.02 ms of 0.89 now.  The
// blocks wait for their tiles' loads: the matrix cores would take 0.02 ms.)
#include <algorithm>

#include "dev_common.h"
#include "net.h"

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int TW = 32;
constexpr int wg_rows(int cg) { return cg == 4 ? 4 : 8; }  // pixel rows of a tile

// Channel l % 16 of pixels 8 (l / 16) .. + 7 for lane l (an MFMA operand over 32 pixels) from
// LDS `p` = &tile[first pixel][first channel], pixel stride ps: two transposed reads, each
// lane addressing 4 channels of one pixel.
__device__ __forceinline__ bf16x8 read_t(const bf16* p, int ps, int lane) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const bf16* q = p + (8 * (lane / 16) + (lane % 16) / 4) * ps + 4 * (lane % 4);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)q);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q + 4 * ps));
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// 8 input channels [ci, ci + 8) of pixel (z, y, x) inside the layer, the values the forward
// convolution stages (MODE 0 plain, 1 averaged, 2 upsampled part then skip)
template <int NDIM, int MODE>
__device__ __forceinline__ bf16x8 input8(const WgradArgs& a, long long img, int z, int y, int x, int ci) {
  const NetSrc& s = a.src;
  const int D = NDIM == 3 ? a.D : 1;
  if (MODE == 1) {
    const int Ds = NDIM == 3 ? s.Ds : 1;
    float acc[8];
#pragma unroll
    for (int v = 0; v < 8; ++v) acc[v] = 0.f;
#pragma unroll
    for (int e = 0; e < (NDIM == 3 ? 2 : 1); ++e)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int zz = NDIM == 3 ? 2 * z + e : 0, yy = 2 * y + q, xx = 2 * x + b;
          const bool ok = zz < Ds && yy < s.Hs && xx < s.Ws;
          const long long p = ((img * Ds + min(zz, Ds - 1)) * s.Hs + min(yy, s.Hs - 1)) * s.Ws + min(xx, s.Ws - 1);
          const bf16x8 t = *reinterpret_cast<const bf16x8*>(s.in + p * s.in_ct + s.in_off + ci);
#pragma unroll
          for (int v = 0; v < 8; ++v) acc[v] += ok ? (float)t[v] : 0.f;
        }
    bf16x8 o;
#pragma unroll
    for (int v = 0; v < 8; ++v) o[v] = (bf16)((NDIM == 3 ? 0.125f : 0.25f) * acc[v]);
    return o;
  }
  if (MODE == 2 && ci < s.cup) {
    const int Du = NDIM == 3 ? (D + 1) / 2 : 1, Hu = (a.H + 1) / 2, Wu = (a.W + 1) / 2;
    const long long p = ((img * Du + (z >> 1)) * Hu + (y >> 1)) * Wu + (x >> 1);
    return *reinterpret_cast<const bf16x8*>(s.up + p * s.up_ct + ci);
  }
  const long long p = ((img * D + z) * a.H + y) * a.W + x;
  return *reinterpret_cast<const bf16x8*>(s.in + p * s.in_ct + s.in_off + ci - s.cup);
}

template <int NDIM, int MODE, int CG, int NCO>
__global__ __launch_bounds__(256) void k_wgrad(WgradArgs a) {
  constexpr int TH = wg_rows(CG), TW2 = TW + 2, WR = 4 / CG, ROWS = TH / WR;  // rows per wavefront
  constexpr int PSI = CG * 16 + 8, PSG = NCO * 16 + 8, CI8 = CG * 2, CO8 = NCO * 2;
  extern __shared__ __align__(16) bf16 sin[];
  bf16* sg = sin + (TH + 2) * TW2 * PSI;
  const int tid = threadIdx.x, lane = tid % 64, i16 = lane % 16, gq = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int cg = wave % CG, rp = wave / CG, ci_base = blockIdx.y * CG * 16;
  const int dz = NDIM == 3 ? (int)blockIdx.z - 1 : 0;
  const int D = NDIM == 3 ? a.D : 1, H = a.H, W = a.W;
  const int txn = (W + TW - 1) / TW, tyn = (H + TH - 1) / TH;
  bf16x8 zero, one;
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    zero[v] = (bf16)0.f;
    one[v] = (bf16)1.f;
  }
  f32x4 acc[9][NCO], bacc[NCO];
#pragma unroll
  for (int n = 0; n < NCO; ++n) {
    bacc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // the bias sums ride on the centre tap plane of the first channel group
  const bool bias = blockIdx.y == 0 && dz == 0 && cg == 0;
  for (int t = blockIdx.x; t < a.ntile; t += a.nchunk) {
    const int x0 = t % txn * TW, y0 = t / txn % tyn * TH;
    const int rz = t / (txn * tyn), z = NDIM == 3 ? rz % D : 0;
    const long long img = NDIM == 3 ? rz / D : rz;
    const int zi = z + dz;
    const bool zin = zi >= 0 && zi < D;
    __syncthreads();  // the last tile's reads are done
    for (int q = tid; q < (TH + 2) * TW2 * CI8; q += 256) {
      const int c = q % CI8, p = q / CI8, yy = y0 - 1 + p / TW2, xx = x0 - 1 + p % TW2, ci = ci_base + 8 * c;
      bf16x8 v = zero;
      if (zin && yy >= 0 && yy < H && xx >= 0 && xx < W && ci < a.cin) v = input8<NDIM, MODE>(a, img, zi, yy, xx, ci);
      *reinterpret_cast<bf16x8*>(sin + p * PSI + 8 * c) = v;
    }
    for (int q = tid; q < TH * TW * CO8; q += 256) {
      const int c = q % CO8, p = q / CO8, yy = y0 + p / TW, xx = x0 + p % TW;
      bf16x8 v = zero;
      if (yy < H && xx < W)
        v = *reinterpret_cast<const bf16x8*>(a.g + (((img * D + z) * H + yy) * W + xx) * a.g_ct + 8 * c);
      *reinterpret_cast<bf16x8*>(sg + p * PSG + 8 * c) = v;
    }
    __syncthreads();
    bf16x8 row[3][3];  // halo rows r, r + 1, r + 2 (index mod 3) at the three x shifts
    const int r0 = rp * ROWS;
    auto load_row = [&](int r, bf16x8 (&o)[3]) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) o[dx] = read_t(sin + (r * TW2 + dx) * PSI + cg * 16, PSI, lane);
    };
    load_row(r0, row[0]);
    load_row(r0 + 1, row[1]);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      load_row(r0 + r + 2, row[(r + 2) % 3]);
      bf16x8 g[NCO];
#pragma unroll
      for (int n = 0; n < NCO; ++n) g[n] = read_t(sg + (r0 + r) * TW * PSG + n * 16, PSG, lane);
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int n = 0; n < NCO; ++n)
          acc[tap][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row[(r + tap / 3) % 3][tap % 3], g[n], acc[tap][n], 0, 0, 0);
      if (bias) {
#pragma unroll
        for (int n = 0; n < NCO; ++n) bacc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(one, g[n], bacc[n], 0, 0, 0);
      }
    }
  }
  // wavefronts that shared the rows: sums added in the order of the row parts
  if constexpr (WR > 1) {
    f32x4* red = reinterpret_cast<f32x4*>(sin);  // [CG][9 NCO + NCO][64]
    for (int q = 1; q < WR; ++q) {
      __syncthreads();
      if (rp == q) {
#pragma unroll
        for (int n = 0; n < NCO; ++n) {
#pragma unroll
          for (int t = 0; t < 9; ++t) red[((cg * NCO + n) * 10 + t) * 64 + lane] = acc[t][n];
          red[((cg * NCO + n) * 10 + 9) * 64 + lane] = bacc[n];
        }
      }
      __syncthreads();
      if (rp == 0) {
#pragma unroll
        for (int n = 0; n < NCO; ++n) {
#pragma unroll
          for (int t = 0; t < 9; ++t) acc[t][n] += red[((cg * NCO + n) * 10 + t) * 64 + lane];
          bacc[n] += red[((cg * NCO + n) * 10 + 9) * 64 + lane];
        }
      }
    }
    if (rp != 0) return;
  }
  // D[i][j]: i = input channel 4 gq + r of the tile, j = output channel i16
  const int ci = ci_base + cg * 16 + 4 * gq;
  float* pb = a.part + (long long)blockIdx.x * a.part_stride;
#pragma unroll
  for (int n = 0; n < NCO; ++n) {
    float* pr = pb + (long long)(n * 16 + i16) * a.kpad + (dz + (NDIM == 3 ? 1 : 0)) * 9 * a.cin + ci;
    if (ci < a.cin) {
#pragma unroll
      for (int t = 0; t < 9; ++t) *reinterpret_cast<f32x4*>(pr + t * a.cin) = acc[t][n];
    }
    if (bias && gq == 0) pb[(long long)a.cout_pad * a.kpad + n * 16 + i16] = bacc[n][0];
  }
}

// dw and db of every layer: the chunk partials added in a fixed order (four threads per entry
// take every fourth chunk, eight loads in flight); zero past the last tap
constexpr int RED_E = 64, RED_Q = 4;
__global__ __launch_bounds__(RED_E* RED_Q) void k_wgrad_reduce(WgradReduceArgs a) {
  __shared__ float sum[RED_Q][RED_E];
  int l = 0;
  while (l + 1 < a.n && (int)blockIdx.x >= a.L[l + 1].block0) ++l;
  const WgradReduceLayer& L = a.L[l];
  const int e = threadIdx.x % RED_E, q = threadIdx.x / RED_E;
  const int nw = L.cout_pad * L.kpad, t = ((int)blockIdx.x - L.block0) * RED_E + e;
  const bool real = t < nw ? t % L.kpad < L.kreal : t - nw < L.cout;
  float s = 0.f;
  if (real) {
    const float* p = L.part + t;
    int c = q;
    for (; c + 7 * RED_Q < L.nchunk; c += 8 * RED_Q) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(long long)(c + u * RED_Q) * L.stride];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; c < L.nchunk; c += RED_Q) s += p[(long long)c * L.stride];
  }
  sum[q][e] = s;
  __syncthreads();
  if (q) return;
  s = (sum[0][e] + sum[1][e]) + (sum[2][e] + sum[3][e]);
  if (t < nw) L.dw[t] = s;
  else if (t - nw < L.cout) L.db[t - nw] = s;
}

template <int NDIM, int MODE, int CG, int NCO>
void wgrad_launch(hipStream_t s, const WgradArgs& a) {
  constexpr int TH = wg_rows(CG);
  const size_t tile = ((TH + 2) * (TW + 2) * (CG * 16 + 8) + TH * TW * (NCO * 16 + 8)) * sizeof(bf16);
  const size_t red = CG == 4 ? 0 : (size_t)CG * NCO * 10 * 64 * sizeof(f32x4);
  const int groups = (a.cin + CG * 16 - 1) / (CG * 16);
  hipLaunchKernelGGL((k_wgrad<NDIM, MODE, CG, NCO>), dim3(a.nchunk, groups, NDIM == 3 ? 3 : 1), dim3(256),
                     std::max(tile, red), s, a);
}

int channel_group(int cin) { return cin % 64 == 0 ? 4 : (cin % 32 == 0 ? 2 : 1); }

}  // namespace

void wgrad_plan(WgradArgs& a) {
  const int cg = channel_group(a.cin), th = wg_rows(cg);
  const long long planes = (long long)a.nimg * (a.dim == 3 ? a.D : 1);
  a.ntile = (int)(planes * ((a.H + th - 1) / th) * ((a.W + TW - 1) / TW));
  a.part_stride = (long long)a.cout_pad * a.kpad + a.cout_pad;
  // about two blocks per CU over the channel groups and tap planes, the partials within 16 MB
  const int groups = (a.cin + cg * 16 - 1) / (cg * 16) * (a.dim == 3 ? 3 : 1);
  const long long most = std::max<long long>(1, (4LL << 20) / a.part_stride);
  a.nchunk = (int)std::max<long long>(1, std::min<long long>({a.ntile, 512 / groups, most}));
}

bool launch_wgrad(hipStream_t s, const WgradArgs& a) {
  const int mode = a.src.pool ? 1 : (a.src.cup > 0 ? 2 : 0), nco = a.cout_pad / 16, cg = channel_group(a.cin);
  // the layers of the two networks
  switch (((a.dim * 10 + mode) * 10 + cg) * 10 + nco) {
    case 2011: wgrad_launch<2, 0, 1, 1>(s, a); return true;  // A0, O
    case 2112: wgrad_launch<2, 1, 1, 2>(s, a); return true;  // A1
    case 2124: wgrad_launch<2, 1, 2, 4>(s, a); return true;  // A2
    case 2144: wgrad_launch<2, 1, 4, 4>(s, a); return true;  // A3
    case 2244: wgrad_launch<2, 2, 4, 4>(s, a); return true;  // B2
    case 2222: wgrad_launch<2, 2, 2, 2>(s, a); return true;  // B1
    case 2211: wgrad_launch<2, 2, 1, 1>(s, a); return true;  // B0
    case 3011: wgrad_launch<3, 0, 1, 1>(s, a); return true;  // A0, O
    case 3111: wgrad_launch<3, 1, 1, 1>(s, a); return true;  // A1
    case 3112: wgrad_launch<3, 1, 1, 2>(s, a); return true;  // A2
    case 3122: wgrad_launch<3, 1, 2, 2>(s, a); return true;  // A3
    case 3242: wgrad_launch<3, 2, 4, 2>(s, a); return true;  // B2
    case 3211: wgrad_launch<3, 2, 1, 1>(s, a); return true;  // B1
    case 3221: wgrad_launch<3, 2, 2, 1>(s, a); return true;  // B0
    default: return false;
  }
}

void launch_wgrad_reduce(hipStream_t s, WgradReduceArgs& a) {
  int blocks = 0;
  for (int l = 0; l < a.n; ++l) {
    a.L[l].block0 = blocks;
    blocks += (a.L[l].cout_pad * a.L[l].kpad + a.L[l].cout + RED_E - 1) / RED_E;
  }
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(blocks), dim3(RED_E * RED_Q), 0, s, a);
}
