// fp32 convolutions with fp64 accumulation: the DAT_F32 path (the tiny CNN of the fp32 configuration, and reduced-size
// runs of the ResNets that cross-check the bf16 MFMA path).  The three contractions run as tiled products on the vector
// units: a workgroup stages a k-chunk of both operands in LDS (the im2col gather happens on the way in, the next chunk
// is in registers meanwhile) and every thread keeps a small block of fp64 sums.  The sum of an output runs over
// (filter row, filter column, channel) in that order, padding adding exact zeros.
//
// What bounds them: at the toy configuration's sizes (32 images of 32x32, 3 -> 16 -> 32 channels) each launch is a
// single round of workgroups and its time is the latency of K/32 chunks.  One thread per output element reading the
// weights at a stride of k*k*Cin floats took 18 / 68 us (forward), 37 / 27 us (backward-data); a wavefront per weight
// walking all pixels 310 / 235 us (backward-weight): the tiles make every global access contiguous and share it
// between the threads of a workgroup, and the pixel range of backward-weight is split over several hundred workgroups.
// The whole iteration of that configuration (FGSM, gradient, update, quantizer): 993 -> 364 us.
#include "kernels.h"

namespace dat {
namespace {
constexpr int kT = 256;
constexpr int KC = 32;        // depth of a staged chunk

// One output tile of  D[m][n] = sum_k A(m, k) B(k, n):  TM x TN outputs per workgroup, MM x MN per thread.
//   forward (DATA = false):       m = output pixel, n = output channel, k = (r, s, input channel)
//   backward-data (DATA = true):  m = input pixel,  n = input channel,  k = (r, s, output channel)
template <int TM, int TN, int MM, int MN, bool DATA>
__global__ __launch_bounds__(kT) void direct_tile_kernel(const float* __restrict__ a, const float* __restrict__ w, const float* __restrict__ res,
                                                         float* __restrict__ d, ConvGeom g) {
  static_assert((TM / MM) * (TN / MN) == kT, "one output block per thread");
  constexpr int LA = TM * KC / kT, LB = (TN * KC + kT - 1) / kT;    // elements per thread and chunk
  constexpr int NT = TN / MN, MT = TM / MM;
  __shared__ float As[KC][TM + 1], Bs[KC][TN + 1];
  const int tid = threadIdx.x;
  const int Hm = DATA ? g.H : g.Ho, Wm = DATA ? g.W : g.Wo;         // grid of the result's pixels
  const int Ha = DATA ? g.Ho : g.H, Wa = DATA ? g.Wo : g.W;         // ... of the gathered operand's
  const int N = DATA ? g.Cin : g.Cout, Ca = DATA ? g.Cout : g.Cin;
  const int K = g.k * g.k * Ca;
  const int64_t M = (int64_t)g.B * Hm * Wm;
  const int64_t m0 = (int64_t)blockIdx.x * TM;
  const int n0 = blockIdx.y * TN;

  // operand loads: consecutive threads walk consecutive k (consecutive channels of one tap)
  const int kk = tid % KC, lrow = tid / KC;
  int hb[LA], wb[LA]; int64_t nb[LA]; bool mv[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int64_t m = m0 + lrow + (kT / KC) * i;
    mv[i] = m < M;
    const int64_t mm = mv[i] ? m : 0;
    const int64_t n = mm / ((int64_t)Hm * Wm); const int rem = (int)(mm - n * Hm * Wm);
    const int h = rem / Wm, x = rem - h * Wm;
    hb[i] = DATA ? h + g.pad : h * g.stride - g.pad;
    wb[i] = DATA ? x + g.pad : x * g.stride - g.pad;
    nb[i] = n * Ha * Wa;
  }
  float ra[LA], rb[LB];
  auto fetch = [&](int k0) {
    const int k = k0 + kk;
    const bool kv = k < K;
    const int tap = (kv ? k : 0) / Ca, c = (kv ? k : 0) - tap * Ca;
    const int r = tap / g.k, s = tap - r * g.k;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      int h = DATA ? hb[i] - r : hb[i] + r, x = DATA ? wb[i] - s : wb[i] + s;
      bool ok = kv && mv[i] && h >= 0 && x >= 0;
      if (DATA && g.stride != 1) {
        ok = ok && h % g.stride == 0 && x % g.stride == 0;
        h /= g.stride; x /= g.stride;
      }
      ok = ok && h < Ha && x < Wa;
      ra[i] = ok ? a[(nb[i] + (int64_t)h * Wa + x) * Ca + c] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int idx = tid + kT * i;
      if (DATA) {        // w[co][r][s][ci]: ci (= n) is contiguous
        const int n = idx % TN, kb = idx / TN, k2 = k0 + kb;
        const bool ok = kb < KC && k2 < K && n0 + n < N;
        const int tap2 = (ok ? k2 : 0) / Ca, co = (ok ? k2 : 0) - tap2 * Ca;
        rb[i] = ok ? w[((int64_t)co * g.k * g.k + tap2) * N + n0 + n] : 0.f;
      } else {           // w[co][k]: k is contiguous
        const int n = idx / KC;
        rb[i] = (n < TN && n0 + n < N && kv) ? w[(int64_t)(n0 + n) * K + k] : 0.f;
      }
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int i = 0; i < LA; ++i) As[kk][lrow + (kT / KC) * i] = ra[i];
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int idx = tid + kT * i;
      if (TN * KC % kT != 0 && idx >= TN * KC) continue;
      if (DATA) Bs[idx / TN][idx % TN] = rb[i]; else Bs[kk][idx / KC] = rb[i];
    }
  };
  const int tn = tid % NT, tm = tid / NT;
  double acc[MM][MN];
#pragma unroll
  for (int i = 0; i < MM; ++i)
#pragma unroll
    for (int j = 0; j < MN; ++j) acc[i][j] = 0.0;
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += KC) {
    stash();
    __syncthreads();
    if (k0 + KC < K) fetch(k0 + KC);
#pragma unroll 8
    for (int k = 0; k < KC; ++k) {
      double av[MM], bv[MN];
#pragma unroll
      for (int i = 0; i < MM; ++i) av[i] = (double)As[k][tm + MT * i];
#pragma unroll
      for (int j = 0; j < MN; ++j) bv[j] = (double)Bs[k][tn + NT * j];
#pragma unroll
      for (int i = 0; i < MM; ++i)
#pragma unroll
        for (int j = 0; j < MN; ++j) acc[i][j] = __builtin_fma(av[i], bv[j], acc[i][j]);   // (the product of two floats is exact in fp64)
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < MM; ++i) {
    const int64_t m = m0 + tm + MT * i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < MN; ++j) {
      const int n = n0 + tn + NT * j;
      if (n >= N) continue;
      double v = acc[i][j];
      if (res) v += (double)res[m * N + n];
      d[m * N + n] = (float)v;
    }
  }
}

template <bool DATA>
dat_status launch_direct(const float* a, const float* w, const float* res, float* d, const ConvGeom& g, hipStream_t st) {
  const int64_t M = (int64_t)g.B * (DATA ? g.H * g.W : g.Ho * g.Wo);
  const int N = DATA ? g.Cin : g.Cout;
  // narrow results (the 3-channel input gradient, the first layers' widths) in narrow tiles: no idle columns
#define DAT_DIRECT(TM, TN, MM, MN) hipLaunchKernelGGL((direct_tile_kernel<TM, TN, MM, MN, DATA>), dim3((unsigned)((M + TM - 1) / TM), (unsigned)((N + TN - 1) / TN)), dim3(kT), 0, st, a, w, res, d, g)
  if (N <= 4) DAT_DIRECT(128, 4, 2, 1);
  else if (N <= 16) DAT_DIRECT(64, 16, 2, 2);
  else DAT_DIRECT(32, 32, 2, 2);
#undef DAT_DIRECT
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

// Backward-weight: dw[co][j] = sum over pixels of dy[p][co] * x(p, j), j = (r, s, ci).  A workgroup sums one 32 x 32
// tile over `pps` pixels (chunks of 32 staged like above) and leaves fp64 partial sums in ws[split][Cout][J];
// direct_wgrad_reduce_kernel adds the splits in order.
__global__ __launch_bounds__(kT) void direct_wgrad_kernel(const float* __restrict__ x, const float* __restrict__ dy, double* __restrict__ ws,
                                                          ConvGeom g, int64_t pps) {
  __shared__ float As[KC][33], Bs[KC][33];        // dY[pixel][co], X[pixel][j]
  const int tid = threadIdx.x;
  const int J = g.k * g.k * g.Cin;
  const int c0 = blockIdx.x * 32, j0 = blockIdx.y * 32;
  const int64_t npix = (int64_t)g.B * g.Ho * g.Wo;
  const int64_t p0 = (int64_t)blockIdx.z * pps, p1 = min(npix, p0 + pps);
  const int col = tid % 32, row = tid / 32;       // loads: channel (resp. j) col of pixels row, row + 8, row + 16, row + 24
  const int j = j0 + col, tap = (j < J ? j : 0) / g.Cin, ci = (j < J ? j : 0) - tap * g.Cin, r = tap / g.k, s = tap - r * g.k;
  float ra[4], rb[4];
  auto fetch = [&](int64_t pb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t p = pb + row + 8 * i;
      const bool pv = p < p1;
      const int64_t pp = pv ? p : 0;
      const int64_t n = pp / ((int64_t)g.Ho * g.Wo); const int rem = (int)(pp - n * g.Ho * g.Wo);
      const int ho = rem / g.Wo, wo = rem - ho * g.Wo;
      const int h = ho * g.stride + r - g.pad, w = wo * g.stride + s - g.pad;
      ra[i] = (pv && c0 + col < g.Cout) ? dy[pp * g.Cout + c0 + col] : 0.f;
      rb[i] = (pv && j < J && h >= 0 && w >= 0 && h < g.H && w < g.W) ? x[((n * g.H + h) * g.W + w) * g.Cin + ci] : 0.f;
    }
  };
  const int tn = tid % 16, tm = tid / 16;
  double acc[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
  fetch(p0);
  for (int64_t pb = p0; pb < p1; pb += KC) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { As[row + 8 * i][col] = ra[i]; Bs[row + 8 * i][col] = rb[i]; }
    __syncthreads();
    if (pb + KC < p1) fetch(pb + KC);
#pragma unroll 8
    for (int k = 0; k < KC; ++k) {
      const double a0 = (double)As[k][tm], a1 = (double)As[k][tm + 16], b0 = (double)Bs[k][tn], b1 = (double)Bs[k][tn + 16];
      acc[0][0] = __builtin_fma(a0, b0, acc[0][0]); acc[0][1] = __builtin_fma(a0, b1, acc[0][1]);
      acc[1][0] = __builtin_fma(a1, b0, acc[1][0]); acc[1][1] = __builtin_fma(a1, b1, acc[1][1]);
    }
    __syncthreads();
  }
  double* dst = ws + (int64_t)blockIdx.z * g.Cout * J;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int co = c0 + tm + 16 * i, jj = j0 + tn + 16 * q;
      if (co < g.Cout && jj < J) dst[(int64_t)co * J + jj] = acc[i][q];
    }
}

// a workgroup owns 8 weights; 32 thread groups each add every 32nd split, then the groups are added in order
__global__ __launch_bounds__(kT) void direct_wgrad_reduce_kernel(const double* __restrict__ ws, int splits, int64_t n, float* __restrict__ dw, double scale) {
  __shared__ double sh[32][8];
  const int cl = threadIdx.x & 7, grp = threadIdx.x >> 3;
  const int64_t i = (int64_t)blockIdx.x * 8 + cl, ic = i < n ? i : n - 1;
  double s = 0.0;
  for (int k0 = grp; k0 < splits; k0 += 128) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + 32 * u;
      v[u] = ws[(int64_t)(k < splits ? k : splits - 1) * n + ic];
      if (k >= splits) v[u] = 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) s += v[u];
  }
  sh[grp][cl] = s;
  __syncthreads();
  if (grp != 0 || i >= n) return;
  s = 0.0;
  for (int q = 0; q < 32; ++q) s += sh[q][cl];
  dw[i] = (float)(s * scale);
}

struct DirectWgradPlan { int gx, gy, splits, max_splits; int64_t pps; };   // max_splits: before rounding, grows with the batch
DirectWgradPlan plan_direct_wgrad(const ConvGeom& g) {
  DirectWgradPlan p;
  const int64_t npix = (int64_t)g.B * g.Ho * g.Wo;
  p.gx = (g.Cout + 31) / 32; p.gy = (g.k * g.k * g.Cin + 31) / 32;
  // two workgroups per CU, at least two chunks of pixels each
  int64_t splits = (512 + (int64_t)p.gx * p.gy - 1) / ((int64_t)p.gx * p.gy);
  if (splits > (npix + 2 * KC - 1) / (2 * KC)) splits = (npix + 2 * KC - 1) / (2 * KC);
  if (splits < 1) splits = 1;
  p.max_splits = (int)splits;
  p.pps = ((npix + splits - 1) / splits + KC - 1) / KC * KC;
  p.splits = (int)((npix + p.pps - 1) / p.pps);
  return p;
}
}  // namespace

dat_status conv_direct_forward(const float* x, const float* w, const float* res, float* y, const ConvGeom& g, hipStream_t st) {
  return launch_direct<false>(x, w, res, y, g, st);
}

dat_status conv_direct_backward_data(const float* dy, const float* w, float* dx, const ConvGeom& g, bool accumulate, hipStream_t st) {
  return launch_direct<true>(dy, w, accumulate ? dx : nullptr, dx, g, st);
}

size_t conv_direct_wgrad_workspace(const ConvGeom& g) {
  return (size_t)plan_direct_wgrad(g).max_splits * g.Cout * g.k * g.k * g.Cin * sizeof(double);
}

dat_status conv_direct_backward_weight(const float* x, const float* dy, float* dw, const ConvGeom& g, float scale, void* ws, hipStream_t st) {
  const DirectWgradPlan p = plan_direct_wgrad(g);
  hipLaunchKernelGGL(direct_wgrad_kernel, dim3((unsigned)p.gx, (unsigned)p.gy, (unsigned)p.splits), dim3(kT), 0, st, x, dy, (double*)ws, g, p.pps);
  DAT_LAUNCH_CHECK();
  const int64_t n = (int64_t)g.Cout * g.k * g.k * g.Cin;
  hipLaunchKernelGGL(direct_wgrad_reduce_kernel, dim3((unsigned)((n + 7) / 8)), dim3(kT), 0, st, (const double*)ws, p.splits, n, dw, (double)scale);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

}  // namespace dat
