// After the worker block: the server's aggregation of quantized gradients, Eq. (grad_agg), and the
// outer-minimisation oracle A(.) as the layer-wise adaptive learning rate of Eq. (3) with the LAMB
// direction of Alg. A2.  All kernels stream the flat parameter vector once (HBM-bound) and walk the
// tensor table like the quantizer does; per-tensor squared norms are accumulated in fp64, first in
// LDS slots per workgroup, then with one global atomic per workgroup and tensor.
#include "kernels.h"
#include "tensor_table.h"

namespace dat {
namespace {

constexpr int kT = 256;
constexpr int kIter = 8;
constexpr int kSlots = 128;

__device__ __forceinline__ void atomic_add_f64(double* p, double v) { atomicAdd(p, v); }

// m, v, u updated in place; norms[0][t] += sum theta^2, norms[1][t] += sum u^2.
__global__ __launch_bounds__(kT) void lamb_direction_kernel(const float* __restrict__ theta, const float* __restrict__ g,
                                                            float* __restrict__ m, float* __restrict__ v,
                                                            float* __restrict__ u, const int64_t* __restrict__ off,
                                                            int T, int64_t d, LambParams hp, double* __restrict__ norms) {
  __shared__ double s_n[2][kSlots];
  __shared__ int s_tfirst;
  const int64_t i_begin = (int64_t)blockIdx.x * (kT * kIter);
  if (threadIdx.x == 0) s_tfirst = find_tensor(off, T, min(i_begin, d - 1));
  if (threadIdx.x < kSlots) { s_n[0][threadIdx.x] = 0.0; s_n[1][threadIdx.x] = 0.0; }
  __syncthreads();
  const int tfirst = s_tfirst;
  int t = tfirst;
  int64_t next = off[t + 1];
  double a_th = 0.0, a_u = 0.0;
  auto flush = [&]() {
    if (a_th != 0.0 || a_u != 0.0) {
      const int slot = t - tfirst;
      if (slot < kSlots) { atomic_add_f64(&s_n[0][slot], a_th); atomic_add_f64(&s_n[1][slot], a_u); }
      else { atomic_add_f64(norms + t, a_th); atomic_add_f64(norms + T + t, a_u); }
    }
    a_th = 0.0; a_u = 0.0;
  };
  for (int it = 0; it < kIter; ++it) {
    const int64_t i = i_begin + (int64_t)it * kT + threadIdx.x;
    if (i >= d) break;
    while (i >= next) { flush(); ++t; next = off[t + 1]; }
    const float th = theta[i], gi = g[i];
    float ui;
    if (hp.use_adam) {
      const float mi = hp.b1 * m[i] + (1.0f - hp.b1) * gi;
      const float vi = hp.b2 * v[i] + (1.0f - hp.b2) * gi * gi;
      m[i] = mi; v[i] = vi;
      ui = (mi * hp.inv_bc1) / (sqrtf(vi * hp.inv_bc2) + hp.zeta);
    } else {
      ui = gi;
    }
    ui += hp.wd * th;
    u[i] = ui;
    a_th += (double)th * (double)th;
    a_u += (double)ui * (double)ui;
  }
  flush();
  __syncthreads();
  if (threadIdx.x < kSlots && tfirst + (int)threadIdx.x < T) {
    if (s_n[0][threadIdx.x] != 0.0) atomic_add_f64(norms + tfirst + threadIdx.x, s_n[0][threadIdx.x]);
    if (s_n[1][threadIdx.x] != 0.0) atomic_add_f64(norms + T + tfirst + threadIdx.x, s_n[1][threadIdx.x]);
  }
}

// theta_i <- theta_i - eta * tau(||theta_i||) / ||u_i|| * u_i
__global__ __launch_bounds__(kT) void lalr_apply_kernel(float* __restrict__ theta, const float* __restrict__ u,
                                                        const int64_t* __restrict__ off, int T, int64_t d,
                                                        LambParams hp, const double* __restrict__ norms) {
  const int64_t i_begin = (int64_t)blockIdx.x * (kT * kIter);
  int64_t i = i_begin + threadIdx.x;
  if (i >= d) return;
  int t = find_tensor(off, T, i);
  int64_t next = off[t + 1];
  auto rate_of = [&](int tt) -> float {
    const double nth = sqrt(norms[tt]), nu = sqrt(norms[T + tt]);
    if (!(nu > 0.0)) return 0.0f;
    const double tau = fmin(fmax(nth, (double)hp.c_l), (double)hp.c_u);
    return (float)((double)hp.eta * tau / nu);
  };
  float rate = rate_of(t);
  for (int it = 0; it < kIter; ++it, i += kT) {
    if (i >= d) break;
    while (i >= next) { ++t; next = off[t + 1]; rate = rate_of(t); }
    theta[i] = theta[i] - rate * u[i];
  }
}

__global__ void zero_f64_kernel(double* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

// ---- aggregation of M quantized gradients ------------------------------------------------------
// out[e] = (sum over workers w, in order, of code_w[e] * (scale_w[t] / S)) / M.  Bound by HBM: M*BITS/8 bytes read and
// four written per element.  A thread owns kWords words, kT words apart; where they all lie inside one tensor (nearly
// everywhere: a workgroup covers 4 K elements) the quotient scale_w / S is formed once per worker instead of once per
// element, and the words of kGroup workers are in flight while the group before is added; the first group is requested
// before the tensor table (searched in LDS) is even read.  25.6 M elements, 8 bit, M = 8 (307 MB): 171 us with a division
// and two dependent loads per element and worker; 101 us with one worker ahead and eight words per thread (85 registers);
// 68 us = 4.5 TB/s like this, a large copy's rate.
template <int BITS> struct AggFmt {
  static constexpr int kEpw = 32 / BITS;                                 // codes per 32-bit word
  static constexpr int kWords = BITS >= 8 ? 4 : BITS == 4 ? 2 : 1;       // words per thread: at most 16 sums in registers
  static constexpr int kGroup = 4;                                       // workers whose words are in flight together
};

template <int BITS>
__global__ __launch_bounds__(kT) void aggregate_kernel(AggregateArgs a) {
  constexpr int EPW = AggFmt<BITS>::kEpw, NW = AggFmt<BITS>::kWords, G = AggFmt<BITS>::kGroup;
  constexpr int S = (1 << (BITS - 1)) - 1;
  __shared__ int64_t s_off[kTabMax + 1];
  const int64_t nwords = (a.d * BITS + 31) / 32;
  int64_t wi = (int64_t)blockIdx.x * (kT * NW) + threadIdx.x;
  // the first group's words do not depend on the table: requested before it is searched (words past the end: word 0)
  const bool whole = (wi + (int64_t)(NW - 1) * kT) * EPW + (EPW - 1) < a.d;
  uint32_t cur[G][NW];
  auto load = [&](uint32_t (&dst)[G][NW], int w0) {
#pragma unroll
    for (int v = 0; v < G; ++v) {
      const uint32_t* src = reinterpret_cast<const uint32_t*>(a.q[w0 + v < a.M ? w0 + v : a.M - 1]) + wi;
#pragma unroll
      for (int u = 0; u < NW; ++u) dst[v][u] = src[u * kT];
    }
  };
  if (whole) load(cur, 0);
  const int64_t* off = stage_offsets(a.offsets, a.T, s_off);
  if (wi >= nwords) return;
  int t = find_tensor(off, a.T, wi * EPW);
  int64_t next = off[t + 1];
  auto code_of = [](uint32_t word, int j) { return (float)(((int)(word << (32 - BITS * (j + 1)))) >> (32 - BITS)); };
  // division by the number of workers: by a power of two it is the multiplication with the exact reciprocal
  const bool pow2 = (a.M & (a.M - 1)) == 0;
  const float fm = (float)a.M, inv = 1.0f / fm;
  const int64_t ilast = (wi + (int64_t)(NW - 1) * kT) * EPW + (EPW - 1);
  if (ilast < next && whole && (reinterpret_cast<uintptr_t>(a.out) & 15) == 0) {
    float acc[NW][EPW];
#pragma unroll
    for (int u = 0; u < NW; ++u)
#pragma unroll
      for (int j = 0; j < EPW; ++j) acc[u][j] = 0.0f;
    for (int w0 = 0; w0 < a.M; w0 += G) {
      float sc[G];
#pragma unroll
      for (int v = 0; v < G; ++v) sc[v] = a.scales[w0 + v < a.M ? w0 + v : a.M - 1][t];
      uint32_t nxt[G][NW];
      if (w0 + G < a.M) load(nxt, w0 + G);
#pragma unroll
      for (int v = 0; v < G; ++v) {
        if (w0 + v >= a.M) break;
        const float step = __fdiv_rn(sc[v], (float)S);
#pragma unroll
        for (int u = 0; u < NW; ++u)
#pragma unroll
          for (int j = 0; j < EPW; ++j) acc[u][j] = __fadd_rn(acc[u][j], __fmul_rn(code_of(cur[v][u], j), step));
      }
#pragma unroll
      for (int v = 0; v < G; ++v)
#pragma unroll
        for (int u = 0; u < NW; ++u) cur[v][u] = nxt[v][u];
    }
#pragma unroll
    for (int u = 0; u < NW; ++u) {
      float r[EPW];
#pragma unroll
      for (int j = 0; j < EPW; ++j) r[j] = pow2 ? __fmul_rn(acc[u][j], inv) : __fdiv_rn(acc[u][j], fm);
      float* o = a.out + (wi + (int64_t)u * kT) * EPW;
      if (EPW == 2) *reinterpret_cast<float2*>(o) = make_float2(r[0], r[1]);
      else {
#pragma unroll
        for (int j = 0; j + 4 <= EPW; j += 4) *reinterpret_cast<float4*>(o + j) = make_float4(r[j], r[j + 1], r[j + 2], r[j + 3]);
      }
    }
    return;
  }
  // words that reach into another tensor, or past the end of the vector
  const int64_t nbytes = (a.d * BITS + 7) / 8;
  for (int it = 0; it < NW; ++it, wi += kT) {
    if (wi >= nwords) break;
    const int64_t i0 = wi * EPW;
    float acc[EPW];
    int tt[EPW];
#pragma unroll
    for (int j = 0; j < EPW; ++j) {
      acc[j] = 0.0f;
      const int64_t i = i0 + j;
      if (i < a.d) { while (i >= next) { ++t; next = off[t + 1]; } }
      tt[j] = t;
    }
    const bool full = (wi + 1) * 4 <= nbytes;
    for (int w = 0; w < a.M; ++w) {
      uint32_t word = 0;
      if (full) word = reinterpret_cast<const uint32_t*>(a.q[w])[wi];
      else for (int b = 0; b < 4 && wi * 4 + b < nbytes; ++b) word |= (uint32_t)a.q[w][wi * 4 + b] << (8 * b);
#pragma unroll
      for (int j = 0; j < EPW; ++j) acc[j] = __fadd_rn(acc[j], __fmul_rn(code_of(word, j), __fdiv_rn(a.scales[w][tt[j]], (float)S)));
    }
#pragma unroll
    for (int j = 0; j < EPW; ++j)
      if (i0 + j < a.d) a.out[i0 + j] = __fdiv_rn(acc[j], fm);
  }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + (int64_t)kT * kIter - 1) / ((int64_t)kT * kIter)); }

}  // namespace

dat_status launch_lamb(float* theta, const float* g, float* m, float* v, float* u, const int64_t* off, int T, int64_t d,
                       const LambParams& hp, double* norms, hipStream_t st) {
  hipLaunchKernelGGL(zero_f64_kernel, dim3((2 * T + 255) / 256), dim3(256), 0, st, norms, 2 * T);
  DAT_LAUNCH_CHECK();
  hipLaunchKernelGGL(lamb_direction_kernel, dim3(blocks_for(d)), dim3(kT), 0, st, theta, g, m, v, u, off, T, d, hp, norms);
  DAT_LAUNCH_CHECK();
  hipLaunchKernelGGL(lalr_apply_kernel, dim3(blocks_for(d)), dim3(kT), 0, st, theta, u, off, T, d, hp, norms);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

}  // namespace dat

using namespace dat;

extern "C" dat_status dat_aggregate(const uint8_t* const* q, const float* const* scales, int M, const int64_t* offsets_dev,
                                    int num_tensors, int64_t d, int bits, float* out, void* stream) {
  if (!q || !scales || !offsets_dev || !out || M < 1 || M > DAT_MAX_WORKERS || num_tensors < 1 || d < 0) return DAT_ERR_ARG;
  if (bits != 2 && bits != 4 && bits != 8 && bits != 16) return DAT_ERR_ARG;
  AggregateArgs a;
  for (int i = 0; i < M; ++i) {
    if (!q[i] || !scales[i] || !aligned(q[i], 4)) return DAT_ERR_ARG;
    a.q[i] = q[i]; a.scales[i] = scales[i];
  }
  a.M = M; a.offsets = offsets_dev; a.T = num_tensors; a.d = d; a.out = out;
  if (d == 0) return DAT_OK;
  const int64_t nwords = (d * bits + 31) / 32;
  hipStream_t st = (hipStream_t)stream;
#define DAT_AGG(B) hipLaunchKernelGGL(aggregate_kernel<B>, dim3((unsigned)((nwords + kT * AggFmt<B>::kWords - 1) / (kT * AggFmt<B>::kWords))), dim3(kT), 0, st, a)
  switch (bits) {
    case 2: DAT_AGG(2); break;
    case 4: DAT_AGG(4); break;
    case 8: DAT_AGG(8); break;
    default: DAT_AGG(16); break;
  }
#undef DAT_AGG
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}
