// fp32 convolutions with fp64 accumulation: the DAT_F32 path (the tiny CNN of the fp32 configuration, and reduced-size
// runs of the ResNets that cross-check the bf16 MFMA path).  The three contractions run as tiled products on the vector
// units: a workgroup stages a k-chunk of both operands in LDS (the im2col gather happens on the way in, the next chunk
// is in registers meanwhile) and every thread keeps a small block of fp64 sums.  The sum of an output runs over
// (filter row, filter column, channel) in that order.  A tap outside the image is no term of the sum.  It is staged as a
// zero, which adds nothing as long as the other factor is finite; a workgroup that meets an infinity or a NaN in that
// factor (the weights; the output gradient in backward-weight) tests every tap from there on instead, so that border pixels
// and weights that never see the value stay finite.
//
// What bounds them: at the toy configuration's sizes (32 images of 32x32, 3 -> 16 -> 32 channels) each launch is a
// single round of workgroups and its time is the latency of K/32 chunks.  One thread per output element reading the
// weights at a stride of k*k*Cin floats took 18 / 68 us (forward), 37 / 27 us (backward-data); a wavefront per weight
// walking all pixels 310 / 235 us (backward-weight): the tiles make every global access contiguous and share it
// between the threads of a workgroup, and the pixel range of backward-weight is split over several hundred workgroups.
// The whole iteration of that configuration (FGSM, gradient, update, quantizer): 993 -> 364 us, and 257 us since the strided
// layer's backward-data pass walks only the taps a pixel sees (48 -> 18 us) and the layers around it were split further.
#include "kernels.h"

namespace dat {
namespace {
constexpr int kT = 256;
constexpr int KC = 32;        // depth of a staged chunk

__device__ __forceinline__ bool not_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }

// One output tile of  D[m][n] = sum_k A(m, k) B(k, n):  TM x TN outputs per workgroup, MM x MN per thread.
//   forward (DATA = false):       m = output pixel, n = output channel, k = (r, s, input channel)
//   backward-data (DATA = true):  m = input pixel,  n = input channel,  k = (r, s, output channel)
// A strided layer's input pixels fall into stride^2 classes by the remainder of their row and column, and a pixel sees
// only the taps of its class (a quarter of them at stride 2): blockIdx.z is the class, k runs over its taps.
// A thread's two rows or columns are neighbours, one 8-byte LDS read.  (fp64 in LDS saves the conversions and costs as much
// in LDS bandwidth: no faster.)
template <int TM, int TN, int MM, int MN, bool DATA>
__global__ __launch_bounds__(kT) void direct_tile_kernel(const float* __restrict__ a, const float* __restrict__ w, const float* __restrict__ res,
                                                         float* __restrict__ d, ConvGeom g) {
  static_assert((TM / MM) * (TN / MN) == kT, "one output block per thread");
  constexpr int LA = TM * KC / kT, LB = (TN * KC + kT - 1) / kT;    // elements per thread and chunk
  constexpr int NT = TN / MN;
  __shared__ __attribute__((aligned(16))) float As[KC][TM + 2], Bs[KC][TN + 2];
  __shared__ int test_taps;            // a weight that is not finite has been staged
  const int tid = threadIdx.x;
  const int Hm = DATA ? g.H : g.Ho, Wm = DATA ? g.W : g.Wo;         // grid of the result's pixels
  const int Ha = DATA ? g.Ho : g.H, Wa = DATA ? g.Wo : g.W;         // ... of the gathered operand's
  const int N = DATA ? g.Cin : g.Cout, Ca = DATA ? g.Cout : g.Cin;
  // this workgroup's pixels: rows ph, ph + S, ... and columns pw, pw + S, ...; its taps: rf, rf + S, ... and sf, sf + S, ...
  const int S = DATA ? g.stride : 1;
  const int ph = DATA ? (int)blockIdx.z / S : 0, pw = DATA ? (int)blockIdx.z % S : 0;
  const int rf = DATA ? (ph + g.pad) % S : 0, sf = DATA ? (pw + g.pad) % S : 0;
  const int nr = rf < g.k ? (g.k - rf + S - 1) / S : 0, ns = sf < g.k ? (g.k - sf + S - 1) / S : 0;
  const int Hc = (Hm - ph + S - 1) / S, Wc = (Wm - pw + S - 1) / S;
  const int K = nr * ns * Ca, nsd = ns > 0 ? ns : 1;
  const int64_t M = (int64_t)g.B * Hc * Wc;
  const int64_t m0 = (int64_t)blockIdx.x * TM;
  if (m0 >= M) return;
  const int n0 = blockIdx.y * TN;

  // operand loads: consecutive threads walk consecutive k (consecutive channels of one tap)
  const int kk = tid % KC, lrow = tid / KC;
  int hb[LA], wb[LA]; int64_t nb[LA]; bool mv[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int64_t m = m0 + lrow + (kT / KC) * i;
    mv[i] = m < M;
    const int64_t mm = mv[i] ? m : 0;
    const int64_t n = mm / ((int64_t)Hc * Wc); const int rem = (int)(mm - n * Hc * Wc);
    const int h = rem / Wc, x = rem - h * Wc;
    hb[i] = DATA ? (h * S + ph + g.pad - rf) / S : h * g.stride - g.pad;
    wb[i] = DATA ? (x * S + pw + g.pad - sf) / S : x * g.stride - g.pad;
    nb[i] = n * Ha * Wa;
  }
  float ra[LA], rb[LB];
  auto fetch = [&](int k0) {
    const int k = k0 + kk;
    const bool kv = k < K;
    const int tap = (kv ? k : 0) / Ca, c = (kv ? k : 0) - tap * Ca;
    const int r = tap / nsd, s = tap - r * nsd;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int h = DATA ? hb[i] - r : hb[i] + r, x = DATA ? wb[i] - s : wb[i] + s;
      const bool ok = kv && mv[i] && h >= 0 && x >= 0 && h < Ha && x < Wa;
      ra[i] = ok ? a[(nb[i] + (int64_t)h * Wa + x) * Ca + c] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int idx = tid + kT * i;
      if (DATA) {        // w[co][r][s][ci]: ci (= n) is contiguous
        const int n = idx % TN, kb = idx / TN, k2 = k0 + kb;
        const bool ok = kb < KC && k2 < K && n0 + n < N;
        const int t2 = (ok ? k2 : 0) / Ca, co = (ok ? k2 : 0) - t2 * Ca, r2 = t2 / nsd, s2 = t2 - r2 * nsd;
        rb[i] = ok ? w[((int64_t)(co * g.k + rf + r2 * S) * g.k + sf + s2 * S) * N + n0 + n] : 0.f;
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
      if (not_finite(rb[i])) test_taps = 1;
      if (DATA) Bs[idx / TN][idx % TN] = rb[i]; else Bs[kk][idx / KC] = rb[i];
    }
  };
  const int tn = tid % NT, tm = tid / NT;
  double acc[MM][MN];
#pragma unroll
  for (int i = 0; i < MM; ++i)
#pragma unroll
    for (int j = 0; j < MN; ++j) acc[i][j] = 0.0;
  // one chunk, leaving out the taps that lie outside the image
  auto tested_chunk = [&](int k0) {
    const int kend = K - k0 < KC ? K - k0 : KC;
#pragma unroll 1
    for (int i = 0; i < MM; ++i) {
      const int64_t m = m0 + tm * MM + i < M ? m0 + tm * MM + i : 0;
      const int rem = (int)(m % ((int64_t)Hc * Wc)), y = rem / Wc, x = rem - y * Wc;
      const int hp = DATA ? (y * S + ph + g.pad - rf) / S : y * g.stride - g.pad, wp = DATA ? (x * S + pw + g.pad - sf) / S : x * g.stride - g.pad;
#pragma unroll 1
      for (int k = 0; k < kend; ++k) {
        const int tap = (k0 + k) / Ca, r = tap / nsd, s = tap - r * nsd;
        const int h = DATA ? hp - r : hp + r, c = DATA ? wp - s : wp + s;
        if (h < 0 || c < 0 || h >= Ha || c >= Wa) continue;
        for (int j = 0; j < MN; ++j) {
          const double v = (double)As[k][tm * MM + i] * (double)Bs[k][tn * MN + j];
          for (int u = 0; u < MM; ++u)            // (constant indices: the sums stay in registers)
            if (u == i) acc[u][j] += v;
        }
      }
    }
  };
  if (tid == 0) test_taps = 0;
  fetch(0);
  __syncthreads();
  for (int k0 = 0; k0 < K; k0 += KC) {
    stash();
    __syncthreads();
    if (k0 + KC < K) fetch(k0 + KC);
    if (test_taps) {
      tested_chunk(k0);
      __syncthreads();
      continue;
    }
#pragma unroll 8
    for (int k = 0; k < KC; ++k) {
      double av[MM], bv[MN];
      if (MM == 2) { const float2 v = *reinterpret_cast<const float2*>(&As[k][tm * 2]); av[0] = (double)v.x; av[MM - 1] = (double)v.y; }
      else av[0] = (double)As[k][tm];
      if (MN == 2) { const float2 v = *reinterpret_cast<const float2*>(&Bs[k][tn * 2]); bv[0] = (double)v.x; bv[MN - 1] = (double)v.y; }
      else bv[0] = (double)Bs[k][tn];
#pragma unroll
      for (int i = 0; i < MM; ++i)
#pragma unroll
        for (int j = 0; j < MN; ++j) acc[i][j] = __builtin_fma(av[i], bv[j], acc[i][j]);   // (the product of two floats is exact in fp64)
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < MM; ++i) {
    const int64_t m = m0 + tm * MM + i;
    if (m >= M) continue;
    int64_t pix = m;
    if (DATA && S != 1) {
      const int64_t n = m / ((int64_t)Hc * Wc); const int rem = (int)(m - n * Hc * Wc), h = rem / Wc;
      pix = (n * Hm + h * S + ph) * Wm + (rem - h * Wc) * S + pw;
    }
#pragma unroll
    for (int j = 0; j < MN; ++j) {
      const int n = n0 + tn * MN + j;
      if (n >= N) continue;
      double v = acc[i][j];
      if (res) v += (double)res[pix * N + n];
      d[pix * N + n] = (float)v;
    }
  }
}

template <bool DATA>
dat_status launch_direct(const float* a, const float* w, const float* res, float* d, const ConvGeom& g, hipStream_t st) {
  const int S = DATA ? g.stride : 1;                     // (the class of the first row and column is the largest)
  const int64_t M = (int64_t)g.B * (DATA ? ((g.H + S - 1) / S) * ((g.W + S - 1) / S) : g.Ho * g.Wo);
  const int N = DATA ? g.Cin : g.Cout;
  // narrow results (the 3-channel input gradient, the first layers' widths) in narrow tiles: no idle columns
#define DAT_DIRECT(TM, TN, MM, MN) hipLaunchKernelGGL((direct_tile_kernel<TM, TN, MM, MN, DATA>), dim3((unsigned)((M + TM - 1) / TM), (unsigned)((N + TN - 1) / TN), (unsigned)(S * S)), dim3(kT), 0, st, a, w, res, d, g)
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
  __shared__ __attribute__((aligned(16))) float As[KC][34], Bs[KC][34];        // dY[pixel][co], X[pixel][j]
  __shared__ int test_taps;                                                     // a gradient that is not finite has been staged
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
  // one chunk, leaving out the taps that lie outside the image
  auto tested_chunk = [&](int64_t pb) {
    const int kend = p1 - pb < KC ? (int)(p1 - pb) : KC;
#pragma unroll 1
    for (int q = 0; q < 2; ++q) {
      const int jj = j0 + tn * 2 + q, jt = (jj < J ? jj : 0) / g.Cin, jr = jt / g.k, js = jt - jr * g.k;
#pragma unroll 1
      for (int k = 0; k < kend; ++k) {
        const int rem = (int)((pb + k) % ((int64_t)g.Ho * g.Wo)), ho = rem / g.Wo, wo = rem - ho * g.Wo;
        const int h = ho * g.stride + jr - g.pad, w = wo * g.stride + js - g.pad;
        if (h < 0 || w < 0 || h >= g.H || w >= g.W) continue;
        for (int i = 0; i < 2; ++i) {
          const double v = (double)As[k][tm * 2 + i] * (double)Bs[k][tn * 2 + q];
          for (int u = 0; u < 2; ++u)             // (constant indices: the sums stay in registers)
            if (u == q) acc[i][u] += v;
        }
      }
    }
  };
  if (tid == 0) test_taps = 0;
  fetch(p0);
  __syncthreads();
  for (int64_t pb = p0; pb < p1; pb += KC) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (not_finite(ra[i])) test_taps = 1;
      As[row + 8 * i][col] = ra[i]; Bs[row + 8 * i][col] = rb[i];
    }
    __syncthreads();
    if (pb + KC < p1) fetch(pb + KC);
    if (test_taps) {
      tested_chunk(pb);
      __syncthreads();
      continue;
    }
#pragma unroll 8
    for (int k = 0; k < KC; ++k) {
      const float2 af = *reinterpret_cast<const float2*>(&As[k][tm * 2]), bf = *reinterpret_cast<const float2*>(&Bs[k][tn * 2]);
      const double2 av = make_double2((double)af.x, (double)af.y), bv = make_double2((double)bf.x, (double)bf.y);
      acc[0][0] = __builtin_fma(av.x, bv.x, acc[0][0]); acc[0][1] = __builtin_fma(av.x, bv.y, acc[0][1]);
      acc[1][0] = __builtin_fma(av.y, bv.x, acc[1][0]); acc[1][1] = __builtin_fma(av.y, bv.y, acc[1][1]);
    }
    __syncthreads();
  }
  double* dst = ws + (int64_t)blockIdx.z * g.Cout * J;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int co = c0 + tm * 2 + i, jj = j0 + tn * 2 + q;
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
