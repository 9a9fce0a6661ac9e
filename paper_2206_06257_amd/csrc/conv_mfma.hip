// bf16 convolutions as implicit GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16,
// fp32 accumulate): forward, backward-data and backward-weight of the conv layers that make
// up dat_attack / dat_step.  Written for 64-wide wavefronts: a 256-thread workgroup is four
// waves (2x2, or 1x4 for 32-channel tiles), each wave owning a block of 32x32 MFMA accumulators.
//
// Forward / backward-data:
//   D[c][p] = sum_k Wt[c][k] * X[p][k],  k = (r, s, ci) flattened, ci fastest.
//   Wt rows are output channels ([Cout][k*k*Cin], K-contiguous); X[p][k] is the im2col view of
//   the NHWC input, gathered on the fly: 8 consecutive k are 8 consecutive channels of one tap,
//   i.e. one 16-byte vector.  Both operands sit in LDS as [row][BK k] tiles (BK = 32 or 64) with
//   an XOR swizzle of the 16-byte slots so that the 16-byte fragment reads of the 32 lanes
//   sharing a k-slot hit distinct banks.  Three kernels fill those tiles:
//   * `igemm_dma_kernel` (contraction channels a multiple of BK): global memory -> LDS directly
//     (buffer_load_dwordx4 ... lds), one LDS stage, four or more workgroups resident per CU;
//   * `igemm_ring_kernel` (layers with at most a few workgroups per CU, and the wide ResNets' multiples of 160
//     channels): one or two workgroups per CU, a ring of LDS stages filled by the same direct loads;
//   * `igemm_kernel` (any channel count, and the long 1x1 contractions into <= 64 channels):
//     global -> registers -> LDS, double buffered, loads running PF k-tiles ahead.
//   Backward-data is the same contraction over the output gradient: stride 1 with the flipped,
//   transposed filter ([Cin][k][k][Cout]); stride 2 over the four parity classes of the input pixels,
//   each a dense stride-1 convolution with that class's sub-filter, in one launch (four where the
//   register-staged kernel runs).
//   The shared epilogue adds an optional residual (or the previously stored gradient) in fp32,
//   rounds once to bf16, transposes through LDS, writes 16-byte channel vectors and can emit the
//   per-channel (sum, sum of squares) of what it stored: the batch statistics of the BN that follows.
//   Workgroups are numbered so that the channel tiles of one pixel tile land on the same XCD
//   (ids congruent mod 8 share an L2), which keeps the gathered activations L2-resident; in the
//   single-stage and register-staged kernels, layers with a filter window also give every XCD one
//   contiguous range of pixel tiles, so that the rows neighbouring tiles share are re-read from that L2.
//   (Not in the multi-stage kernel, measured both ways: 0 to 2.5 % slower with it, 160 channels at 32x32,
//   256 images 138.2 / 137.5 us, 640 at 8x8, 100 images 61.0 / 59.6, 256 at 14x14, 256 images 56.7 / 56.0.)
//
// Backward-weight (`wgrad_kernel`): dW[co][(r,s,ci)] = sum_p dY[p][co] * X[p][(r,s,ci)], a
// contraction over pixels, which are the strided dimension of both operands.  The tiles land in
// LDS as they are in memory ([pixel][channel], direct-to-LDS loads) and the MFMA fragments are
// read with the LDS transpose reads of gfx950 (ds_read_b64_tr_b16), which hand every lane four
// consecutive pixels of its channel.  The pixel range is split over workgroups; partial tiles go to a workspace
// and a second kernel sums them in a fixed order (deterministic).
#include <atomic>
#include <mutex>
#include <cstdlib>
#include "kernels.h"

namespace dat {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kThreads = 256;


typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native 16-byte vector (stays in registers)
union Frag { u32x4 u; bf16x8 v; };

// 16-byte slot permutation of a [row][NS slots] LDS tile (NS = 4: 64-byte rows, NS = 8: 128-byte
// rows).  Chosen so that the lanes of a fragment read (consecutive rows, same logical slot) touch
// distinct 16-byte bank groups both within any 8 consecutive rows x 128 bytes and within any 16
// consecutive rows x 256 bytes (LDS bank sweeps of 32 and of 64 banks).  Uses row bits 0..3 only.
template <int NS> __device__ __forceinline__ int swz(int row, int slot);
template <> __device__ __forceinline__ int swz<4>(int row, int slot) {
  const int f = (((row >> 2) & 1) << 1) | (((row >> 1) ^ (row >> 3)) & 1);
  return row * 64 + ((slot ^ f) << 4);
}
template <> __device__ __forceinline__ int swz<8>(int row, int slot) {
  const int f = (row & 7) ^ ((row >> 3) & 1);
  return row * 128 + ((slot ^ f) << 4);
}

// Out-of-range and padding vectors of igemm_kernel are read from this zero page instead of being masked.
__device__ __attribute__((aligned(16))) uint32_t g_zero_page[4] = {0u, 0u, 0u, 0u};

struct IgemmArgs {
  const bf16_t* in;     // [B][Hin][Win][Cin]
  const bf16_t* wt;     // [Cout][KH*KW*Cin]
  const bf16_t* res;    // optional [M][Cout] added before rounding
  const uint8_t* res_mask;   // optional: bit j of byte e/8 gates element e of `res` (a ReLU mask: res*mask is added)
  int res_even_only;         // `res` holds values only at pixels with even row and even column (ostep 1); the rest counts as zero
  bf16_t* out;          // [M][Cout], M = B*Hout*Wout
  int B, Hin, Win, Cin, Hout, Wout, Cout;   // Hout x Wout = grid of output pixels this launch computes
  int KH, KW, ostride, pad_h, pad_w;
  // Elements between neighbouring input pixels of a row (0: Cin, the ordinary case).  With 0 < xstride < Cin the
  // "Cin channels" of pixel w are the stored values of the pixels w .. w + Cin/xstride - 1, i.e. a filter row of
  // Cin/xstride taps read as one contiguous vector (igemm_dma_kernel with Cin equal to its k-tile only); a 16-byte
  // vector then lies in pixel w + offset/xstride and is zero when that pixel is outside the row.
  int xstride;
  // output pixel (n, a, b) is stored at row (n*outH + a*ostep + oh0)*outW + b*ostep + ow0 of `out`
  int outH, outW, ostep, oh0, ow0;
  int M, Ktot, nct, npt;
  // pixel tile -> XCD: interleaved (tile t on XCD t mod 8) or one contiguous range of tiles per XCD (neighbouring
  // tiles, which share filter-window rows, then share an L2)
  int xcd_contiguous;
  // Optional per-channel sums (sum v, sum v^2) of the stored (bf16-rounded) outputs -- the batch
  // statistics of the normalisation that follows -- one [2][Cout] slab per pixel tile at
  // stat_partial + (stat_slab0 + pixel_tile) * 2 * Cout.
  int stat_mode, stat_slab0;
  float* stat_partial;
  // stat_mode 2: the stored tensor is the output gradient of a batch normalisation with input stat_x (same
  // layout as `out`), ReLU mask stat_mask (or nullptr) and batch statistics stat_mean / stat_rstd; the slabs then
  // hold (sum v*m, sum v*m*xhat), the two sums of that normalisation's backward pass.
  const bf16_t* stat_x; const uint8_t* stat_mask; const float* stat_mean; const float* stat_rstd;
  // stat_mode 3 (results with more than 64 channels only): a second normalisation (input stat_x2, statistics stat_mean2 / stat_rstd2)
  // shares that output gradient; slabs are [3][Cout]: (sum v*m, sum v*m*xhat, sum v*m*xhat2).
  const bf16_t* stat_x2; const float* stat_mean2; const float* stat_rstd2;
  // Optional operand transform (1x1 stride-1 layers, igemm_kernel only): `in` is the output gradient of a batch
  // normalisation, and the operand actually contracted is that normalisation's input gradient,
  // bn_input_grad(in .* mask, xf_x, constants of the channel), rounded to bf16 -- formed while the tile moves from
  // registers to LDS instead of being written to memory by a pass of its own.
  const bf16_t* xf_x;        // [M][Cin] the normalisation's input
  const uint8_t* xf_mask;    // one bit per element of `in` (ReLU mask), or nullptr
  const float* xf_tab;       // 4*Cin floats, layout of bn_input_grad's constants
};

// Several launches of one kernel as one grid: what differs between them.  The four parity classes of a stride-2
// backward-data pass go this way, the classes with most taps first (their workgroups run longest).  Each class has
// blocks [begin, next begin), a multiple of 8, so a class's tiles meet the XCDs as in a launch of its own (whether
// interleaved or in ranges, xcd_contiguous, is decided for all classes by the one with most taps).
struct IgemmClass { const bf16_t* wt; int Hout, Wout, KH, KW, pad_h, pad_w, oh0, ow0, M, Ktot, stat_slab0, with_res, npt, begin; };
struct IgemmClasses { int n; IgemmClass c[4]; };
// An ordinary launch: a kernel of its own, without the table.  With the table as an argument of every launch and all four
// entries read (n = 0: none), the 64- and 32-channel single-stage kernels spilled 9 and 8 vector registers instead of 2 and 4
// and the 256 x 256 multi-stage kernel 16 scalar ones.  (Over 500 layer shapes: ordinary launches 0 to 1.5 % faster without
// it, launches in classes 1 to 2 % since they read their own entry only.)
struct NoClasses { static constexpr int n = 0; };

__device__ __forceinline__ int enter_class(IgemmArgs&, const NoClasses&, int bid) { return bid; }
// Block number within its class, whose values replace those of `a` (read from the argument block at an index that is the
// same for all lanes: scalar loads of one class only).
__device__ __forceinline__ int enter_class(IgemmArgs& a, const IgemmClasses& cl, int bid) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < 4; ++i) k += i < cl.n && bid >= cl.c[i].begin;
  const IgemmClass& c = cl.c[k];
  a.wt = c.wt; a.Hout = c.Hout; a.Wout = c.Wout; a.KH = c.KH; a.KW = c.KW; a.pad_h = c.pad_h; a.pad_w = c.pad_w;
  a.oh0 = c.oh0; a.ow0 = c.ow0; a.M = c.M; a.Ktot = c.Ktot; a.stat_slab0 = c.stat_slab0; a.npt = c.npt;
  if (!c.with_res) a.res = nullptr;
  return bid - c.begin;
}

// dat_conv_plan: while set, the launches of this thread are noted here instead of being made.
struct LaunchRecord { int launches, kernel, tile_c, tile_p, stages, k_tile, straddle, classes; int64_t slabs; };
thread_local LaunchRecord* t_record = nullptr;
enum { kRegisterStaged = 0, kSingleStage = 1, kMultiStage = 2 };

int64_t slabs_of(const IgemmArgs& a, const NoClasses&) { return a.npt; }
int64_t slabs_of(const IgemmArgs&, const IgemmClasses& cl) { int64_t s = 0; for (int i = 0; i < cl.n; ++i) s += cl.c[i].npt; return s; }

template <class CL>
bool recorded(const IgemmArgs& a, const CL& cl, int kernel, int tile_c, int tile_p, int stages, int k_tile, int straddle) {
  if (!t_record) return false;
  LaunchRecord& r = *t_record;
  ++r.launches;
  r.kernel = kernel; r.tile_c = tile_c; r.tile_p = tile_p; r.stages = stages; r.k_tile = k_tile; r.straddle = straddle; r.classes = cl.n;
  r.slabs += slabs_of(a, cl);
  return true;
}

__device__ __forceinline__ int64_t out_row(const IgemmArgs& a, int m) {
  if (a.ostep == 1 && a.outH == a.Hout && a.outW == a.Wout) return m;
  const int HW = a.Hout * a.Wout;
  const int n = m / HW, rem = m - n * HW;
  const int ya = rem / a.Wout, xb = rem - ya * a.Wout;
  return ((int64_t)n * a.outH + ya * a.ostep + a.oh0) * a.outW + xb * a.ostep + a.ow0;
}

// ---- epilogue shared by the convolution kernels: (+res) -> bf16 -> LDS transpose -> 16-byte stores ----
// `lds` must hold TP rows of STG_STRIDE = 2*TC + 16 bytes (and [kThreads/(TC/8)][2][TC] floats for the
// statistics); every wave must be done with whatever else lived there (the caller ends on a barrier).
template <int TC, int TP, int WGC, int NT = kThreads>
__device__ __forceinline__ void igemm_epilogue(const IgemmArgs& a, f32x16 (&acc)[TC / WGC / 32][TP / (NT / 64 / WGC) / 32],
                                               unsigned char* lds, int c0, int m0, int pt) {
  constexpr int WGP = NT / 64 / WGC;
  constexpr int WC = TC / WGC, WP = TP / WGP;
  constexpr int NI = WC / 32, NJ = WP / 32;
  constexpr int STG_STRIDE = TC * 2 + 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wc = wave % WGC, wp = wave / WGC;
  // ---- epilogue: (+res) -> bf16 -> LDS transpose -> 16-byte stores -------------------------
  // accumulator element e of lane l in tile (i,j): channel = 8*(e/4) + 4*(l/32) + e%4, pixel = l%32.
  // All four waves stage their block at once (one barrier), then every thread streams 16-byte
  // channel vectors of whole pixel rows to global memory.
  // A residual (or the previously stored gradient) is first brought into the staging buffer with
  // the same coalesced 16-byte accesses the stores use; each lane then adds its accumulators to
  // the values at its own staging slots in fp32 and rounds once, in place.
  constexpr int CV = TC / 8;                       // channel vectors per pixel row
  constexpr int RPP = NT / CV;                     // pixel rows per store sweep
  constexpr int NU = (TP + RPP - 1) / RPP;         // sweeps
  // tile widths that are no power of two (160 channels: 20 vectors per row, 12 rows per sweep): the last
  // threads have no vector and the last sweep is short
  constexpr bool EXACT = NT % CV == 0 && TP % RPP == 0;
  const int cv = tid % CV, pr0 = tid / CV;
  auto row_ok = [&](int u) { return EXACT || (pr0 < RPP && pr0 + u * RPP < TP); };
  const int ch = c0 + cv * 8;
  if (a.res) {
    uint4 rv[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int m = m0 + pr0 + u * RPP;
      rv[u] = make_uint4(0u, 0u, 0u, 0u);
      bool take = row_ok(u) && m < a.M && ch < a.Cout;
      if (a.res_even_only && take) { const int q = m / a.Wout; take = !(((m - q * a.Wout) | (q % a.Hout)) & 1); }
      if (take) {
        const int64_t e = out_row(a, m) * a.Cout + ch;
        rv[u] = *reinterpret_cast<const uint4*>(a.res + e);
        if (a.res_mask) {
          const uint32_t k = a.res_mask[e >> 3];
          rv[u].x &= ((k & 1u) ? 0xffffu : 0u) | ((k & 2u) ? 0xffff0000u : 0u);
          rv[u].y &= ((k & 4u) ? 0xffffu : 0u) | ((k & 8u) ? 0xffff0000u : 0u);
          rv[u].z &= ((k & 16u) ? 0xffffu : 0u) | ((k & 32u) ? 0xffff0000u : 0u);
          rv[u].w &= ((k & 64u) ? 0xffffu : 0u) | ((k & 128u) ? 0xffff0000u : 0u);
        }
      }
    }
    // (the main loop ended with a barrier: every wave is done with the operand tiles)
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (row_ok(u)) *reinterpret_cast<uint4*>(lds + (pr0 + u * RPP) * STG_STRIDE + cv * 16) = rv[u];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int prow = wp * WP + j * 32 + (lane & 31);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int chl = wc * WC + i * 32 + 8 * g + 4 * (lane >> 5);
        float v[4] = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        uint2* slot = reinterpret_cast<uint2*>(lds + prow * STG_STRIDE + chl * 2);
        if (a.res) {
          const uint2 r = *slot;
          v[0] += __uint_as_float(r.x << 16); v[1] += __uint_as_float(r.x & 0xffff0000u);
          v[2] += __uint_as_float(r.y << 16); v[3] += __uint_as_float(r.y & 0xffff0000u);
        }
        uint2 pk;
        pk.x = f2bf_pack(v[0], v[1]);
        pk.y = f2bf_pack(v[2], v[3]);
        *slot = pk;
      }
    }
  __syncthreads();
  float s1[8], s2[8], s3[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) { s1[j] = 0.f; s2[j] = 0.f; s3[j] = 0.f; }
  if (a.stat_mode == 3) {
    // as mode 2 below, for two normalisations sharing d(out)
    float mu[8], rs[8], mu2[8], rs2[8];
    if (ch < a.Cout) {
#pragma unroll
      for (int j = 0; j < 8; ++j) { mu[j] = a.stat_mean[ch + j]; rs[j] = a.stat_rstd[ch + j]; mu2[j] = a.stat_mean2[ch + j]; rs2[j] = a.stat_rstd2[ch + j]; }
    }
    constexpr int H = (NU + 1) / 2;              // rows in two batches: half the operand registers
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      uint4 xv[H], yv[H]; uint32_t mk[H];
#pragma unroll
      for (int u = 0; u < H; ++u) {
        const int m = m0 + pr0 + (b * H + u) * RPP;
        xv[u] = make_uint4(0u, 0u, 0u, 0u); yv[u] = xv[u]; mk[u] = 0u;
        if (b * H + u < NU && row_ok(b * H + u) && m < a.M && ch < a.Cout) {
          const int64_t e = out_row(a, m) * a.Cout + ch;
          xv[u] = *reinterpret_cast<const uint4*>(a.stat_x + e);
          yv[u] = *reinterpret_cast<const uint4*>(a.stat_x2 + e);
          mk[u] = a.stat_mask ? (uint32_t)a.stat_mask[e >> 3] : 0xffu;
        }
      }
#pragma unroll
      for (int u = 0; u < H; ++u) {
        const int prow = pr0 + (b * H + u) * RPP, m = m0 + prow;
        if (b * H + u < NU && row_ok(b * H + u) && m < a.M && ch < a.Cout) {
          const uint4 pk = *reinterpret_cast<const uint4*>(lds + prow * STG_STRIDE + cv * 16);
          *reinterpret_cast<uint4*>(a.out + out_row(a, m) * a.Cout + ch) = pk;
          const uint32_t w[4] = {pk.x, pk.y, pk.z, pk.w}, xw[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w}, yw[4] = {yv[u].x, yv[u].y, yv[u].z, yv[u].w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float v0 = ((mk[u] >> (2 * j)) & 1u) ? __uint_as_float(w[j] << 16) : 0.f;
            const float v1 = ((mk[u] >> (2 * j + 1)) & 1u) ? __uint_as_float(w[j] & 0xffff0000u) : 0.f;
            s1[2 * j] += v0; s1[2 * j + 1] += v1;
            s2[2 * j] = __builtin_fmaf(v0, (__uint_as_float(xw[j] << 16) - mu[2 * j]) * rs[2 * j], s2[2 * j]);
            s2[2 * j + 1] = __builtin_fmaf(v1, (__uint_as_float(xw[j] & 0xffff0000u) - mu[2 * j + 1]) * rs[2 * j + 1], s2[2 * j + 1]);
            s3[2 * j] = __builtin_fmaf(v0, (__uint_as_float(yw[j] << 16) - mu2[2 * j]) * rs2[2 * j], s3[2 * j]);
            s3[2 * j + 1] = __builtin_fmaf(v1, (__uint_as_float(yw[j] & 0xffff0000u) - mu2[2 * j + 1]) * rs2[2 * j + 1], s3[2 * j + 1]);
          }
        }
      }
    }
  } else if (a.stat_mode == 2) {
    // BN backward sums of the tile just computed: the normalisation's input and mask are fetched for all of this
    // thread's rows before the first one is used
    float mu[8], rs[8];
    if (ch < a.Cout) {
      const float4 m0v = *reinterpret_cast<const float4*>(a.stat_mean + ch), m1v = *reinterpret_cast<const float4*>(a.stat_mean + ch + 4);
      const float4 r0v = *reinterpret_cast<const float4*>(a.stat_rstd + ch), r1v = *reinterpret_cast<const float4*>(a.stat_rstd + ch + 4);
      mu[0] = m0v.x; mu[1] = m0v.y; mu[2] = m0v.z; mu[3] = m0v.w; mu[4] = m1v.x; mu[5] = m1v.y; mu[6] = m1v.z; mu[7] = m1v.w;
      rs[0] = r0v.x; rs[1] = r0v.y; rs[2] = r0v.z; rs[3] = r0v.w; rs[4] = r1v.x; rs[5] = r1v.y; rs[6] = r1v.z; rs[7] = r1v.w;
    }
    uint4 xv[NU]; uint32_t mk[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int m = m0 + pr0 + u * RPP;
      xv[u] = make_uint4(0u, 0u, 0u, 0u); mk[u] = 0u;
      if (row_ok(u) && m < a.M && ch < a.Cout) {
        const int64_t e = out_row(a, m) * a.Cout + ch;
        xv[u] = *reinterpret_cast<const uint4*>(a.stat_x + e);
        mk[u] = a.stat_mask ? (uint32_t)a.stat_mask[e >> 3] : 0xffu;
      }
    }
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int prow = pr0 + u * RPP, m = m0 + prow;
      if (row_ok(u) && m < a.M && ch < a.Cout) {
        const uint4 pk = *reinterpret_cast<const uint4*>(lds + prow * STG_STRIDE + cv * 16);
        *reinterpret_cast<uint4*>(a.out + out_row(a, m) * a.Cout + ch) = pk;
        const uint32_t w[4] = {pk.x, pk.y, pk.z, pk.w}, xw[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v0 = ((mk[u] >> (2 * j)) & 1u) ? __uint_as_float(w[j] << 16) : 0.f;
          const float v1 = ((mk[u] >> (2 * j + 1)) & 1u) ? __uint_as_float(w[j] & 0xffff0000u) : 0.f;
          const float x0 = __uint_as_float(xw[j] << 16), x1 = __uint_as_float(xw[j] & 0xffff0000u);
          s1[2 * j] += v0; s2[2 * j] = __builtin_fmaf(v0, (x0 - mu[2 * j]) * rs[2 * j], s2[2 * j]);
          s1[2 * j + 1] += v1; s2[2 * j + 1] = __builtin_fmaf(v1, (x1 - mu[2 * j + 1]) * rs[2 * j + 1], s2[2 * j + 1]);
        }
      }
    }
  } else {
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int prow = pr0 + u * RPP, m = m0 + prow;
    if (row_ok(u) && m < a.M && ch < a.Cout) {
      const uint4 pk = *reinterpret_cast<const uint4*>(lds + prow * STG_STRIDE + cv * 16);
      *reinterpret_cast<uint4*>(a.out + out_row(a, m) * a.Cout + ch) = pk;
      if (a.stat_mode) {
        const uint32_t w[4] = {pk.x, pk.y, pk.z, pk.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v0 = __uint_as_float(w[j] << 16), v1 = __uint_as_float(w[j] & 0xffff0000u);
          s1[2 * j] += v0; s2[2 * j] = __builtin_fmaf(v0, v0, s2[2 * j]); s1[2 * j + 1] += v1; s2[2 * j + 1] = __builtin_fmaf(v1, v1, s2[2 * j + 1]);
        }
      }
    }
  }
  }
  if (a.stat_mode) {
    // fold the RPP row groups in a fixed order through LDS, one slab per pixel tile
    __syncthreads();
    const int ns = a.stat_mode == 3 ? 3 : 2;        // sums per channel
    float* red = reinterpret_cast<float*>(lds);     // [RPP][ns][TC]
    if (EXACT || pr0 < RPP) {
      // 16-byte stores: as single floats the lanes of a wave (8 floats apart, rows a multiple of 64 floats apart) would
      // land eight to a bank
      auto put = [&](int which, const float (&v)[8]) {
        float4* dst = reinterpret_cast<float4*>(red + (pr0 * ns + which) * TC + cv * 8);
        dst[0] = make_float4(v[0], v[1], v[2], v[3]);
        dst[1] = make_float4(v[4], v[5], v[6], v[7]);
      };
      put(0, s1); put(1, s2);
      if (ns == 3) put(2, s3);
    }
    __syncthreads();
    for (int q = tid; q < ns * TC; q += NT) {
      const int which = q / TC, c = q % TC;
      float t = 0.f;
      for (int g = 0; g < RPP; ++g) t += red[(g * ns + which) * TC + c];
      if (c0 + c < a.Cout) a.stat_partial[((int64_t)(a.stat_slab0 + pt) * ns + which) * a.Cout + c0 + c] = t;
    }
  }
}

template <int TC, int TP, int WGC, int PF, bool FAST, int BKT, int OCC, bool XF = false>
__global__ __launch_bounds__(kThreads, OCC) void igemm_kernel(IgemmArgs a) {
  static_assert(!XF || FAST, "the operand transform needs whole k-tiles of one tap");
  constexpr int WGP = 4 / WGC;                     // waves along channels x waves along pixels
  constexpr int WC = TC / WGC, WP = TP / WGP;      // wave tile
  constexpr int NI = WC / 32, NJ = WP / 32;        // MFMA tiles per wave
  constexpr int NS = BKT / 8;                      // 16-byte slots per tile row
  constexpr int RB = BKT * 2;                      // bytes per tile row
  constexpr int RPG = kThreads / NS;               // tile rows covered by one load per thread
  constexpr int KS = BKT / 16;                     // MFMA k-steps per tile
  constexpr int VW = (TC * NS + kThreads - 1) / kThreads, VX = TP * NS / kThreads;   // 16-byte vectors per thread per tile
  constexpr int TILE_BYTES = (TC + TP) * RB;
  constexpr int STG_STRIDE = TC * 2 + 16;
  constexpr int LDS_BYTES = (2 * TILE_BYTES > TP * STG_STRIDE) ? 2 * TILE_BYTES : TP * STG_STRIDE;
  __shared__ __attribute__((aligned(16))) unsigned char lds[LDS_BYTES];

  // XCD-aware tile numbering: workgroup ids congruent mod 8 run on the same XCD (one L2 each), so
  // all channel tiles of a pixel tile get ids 8 apart and share the gathered activations in one L2.
  // Pixel tiles are dealt to the XCDs round robin, or (layers with a filter window) in one contiguous
  // range per XCD.
  const int bid = blockIdx.x;
  const int q = bid >> 3;
  const int ct = q % a.nct;
  const int pt = a.xcd_contiguous ? (bid & 7) * ((a.npt + 7) >> 3) + (q / a.nct) : (q / a.nct) * 8 + (bid & 7);
  if (pt >= a.npt) return;
  const int c0 = ct * TC, m0 = pt * TP;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wc = wave % WGC, wp = wave / WGC;
  const int kvec = tid % NS, lrow = tid / NS;      // this thread's slot in the global->LDS copy

  // im2col row state for the activation vectors this thread fetches (32-bit element offsets)
  int hb[VX], wb[VX], nb[VX]; bool mv[VX];
  const int HW = a.Hout * a.Wout;
#pragma unroll
  for (int i = 0; i < VX; ++i) {
    const int m = m0 + lrow + RPG * i;
    mv[i] = m < a.M;
    const int mm = mv[i] ? m : 0;
    const int n = mm / HW, rem = mm - n * HW;
    const int ho = rem / a.Wout, wo = rem - ho * a.Wout;
    hb[i] = ho * a.ostride - a.pad_h; wb[i] = wo * a.ostride - a.pad_w;
    nb[i] = n * a.Hin * a.Win;
  }
  const int ntiles = (a.Ktot + BKT - 1) / BKT;
  // (the symbol itself, not a pointer hidden from the compiler: it must see that both sides of the selects below are global
  // memory, or the loads become flat ones, which also count as LDS accesses: 1x1 256 -> 64 at 56x56, 256 images 94 us, flat 101)
  const u32x4* zero_page = reinterpret_cast<const u32x4*>(g_zero_page);

  // Weight rows of this thread: offset of (row, k = kvec*8) and row validity; advances by BK per tile.
  int woff[VW]; bool wrow[VW];
#pragma unroll
  for (int i = 0; i < VW; ++i) {
    const int c = c0 + lrow + RPG * i;
    wrow[i] = (lrow + RPG * i < TC) & (c < a.Cout);
    woff[i] = (wrow[i] ? c : 0) * a.Ktot + kvec * 8;
  }
  // Activation state.  FAST (Cin % 32 == 0): a k-tile never straddles a filter tap, so the tap
  // (r,s), the bounds test and the pixel offset change only every Cin/32 tiles (a uniform branch);
  // in between the offset just advances by 32 channels.  Otherwise every vector decodes its own tap.
  int xoff[VX]; bool xok[VX];
  int kc0 = 0, kr = 0, ks = 0;                      // FAST: channel offset of the tile, current tap
  int kc, gr, gs;                                   // generic: this thread's channel / tap
  {
    const int k = kvec * 8;
    const int tap = k / a.Cin;
    kc = k - tap * a.Cin; gr = tap / a.KW; gs = tap - gr * a.KW;
  }
  auto retap = [&](int r, int s_, int cofs) {
#pragma unroll
    for (int i = 0; i < VX; ++i) {
      const int hi = hb[i] + r, wi = wb[i] + s_;
      xok[i] = mv[i] & (hi >= 0) & (wi >= 0) & (hi < a.Hin) & (wi < a.Win);
      xoff[i] = (nb[i] + hi * a.Win + wi) * a.Cin + cofs;
    }
  };

  // Global loads run PF tiles ahead of the MFMAs: tile t+1 sits in LDS (other buffer) while tiles
  // t+2 .. t+1+PF are in flight into PF register sets.  Every step issues the same number of
  // unconditional loads (invalid vectors read the zero page), so nothing waits on a load early.
  struct RegSet { u32x4 w[VW]; u32x4 x[VX]; u32x4 y[XF ? VX : 1]; uint32_t mk[XF ? VX : 1]; int kch; };
  RegSet rs[PF];
  extern __shared__ __attribute__((aligned(16))) float xf_tab_lds[];   // XF: the constants of all Cin channels
  int kf = 0;                                      // next tile to fetch
  auto fetch = [&](RegSet& r) {
    const bool tile_ok = kf < ntiles;
#pragma unroll
    for (int i = 0; i < VW; ++i) {
      const bool ok = tile_ok & wrow[i] & (FAST || kf * BKT + kvec * 8 < a.Ktot);
      const u32x4* p = ok ? reinterpret_cast<const u32x4*>(a.wt + woff[i]) : zero_page;
      r.w[i] = *p;
      woff[i] += BKT;
    }
    if (FAST) {
      if (kc0 == 0) retap(kr, ks, kvec * 8);       // uniform: first tile of a tap
      if (XF) r.kch = tile_ok ? kc0 : 0;
#pragma unroll
      for (int i = 0; i < VX; ++i) {
        const bool ok = tile_ok & xok[i];
        const u32x4* p = ok ? reinterpret_cast<const u32x4*>(a.in + xoff[i]) : zero_page;
        r.x[i] = *p;
        if (XF) {
          const u32x4* py = ok ? reinterpret_cast<const u32x4*>(a.xf_x + xoff[i]) : zero_page;
          r.y[i] = *py;
          const uint8_t* pm = (ok && a.xf_mask) ? a.xf_mask + (xoff[i] >> 3) : reinterpret_cast<const uint8_t*>(g_zero_page);
          r.mk[i] = a.xf_mask ? (uint32_t)*pm : (ok ? 0xffu : 0u);
        }
        xoff[i] += BKT;
      }
      kc0 += BKT;
      if (kc0 == a.Cin) { kc0 = 0; if (++ks == a.KW) { ks = 0; ++kr; } }
    } else {
      retap(gr, gs, kc);
      const bool kvalid = tile_ok & (kf * BKT + kvec * 8 < a.Ktot);
#pragma unroll
      for (int i = 0; i < VX; ++i) {
        const u32x4* p = (kvalid & xok[i]) ? reinterpret_cast<const u32x4*>(a.in + xoff[i]) : zero_page;
        r.x[i] = *p;
      }
      kc += BKT;
      while (kc >= a.Cin) { kc -= a.Cin; if (++gs == a.KW) { gs = 0; ++gr; } }
    }
    ++kf;
  };
  const int st_w = swz<NS>(lrow, kvec), st_x = TC * RB + swz<NS>(lrow, kvec);   // rows lrow + RPG*i share the swizzle (RPG % 16 == 0)
  auto stash = [&](int buf, const RegSet& r) {
    unsigned char* base = lds + buf * TILE_BYTES;
#pragma unroll
    for (int i = 0; i < VW; ++i)
      if (lrow + RPG * i < TC) *reinterpret_cast<u32x4*>(base + st_w + i * (RPG * RB)) = r.w[i];
    if (XF) {
      // the 8 channels of this thread's vectors: kch + kvec*8 .. +7
      const float* tb = xf_tab_lds + ((r.kch >> 3) + kvec) * 32;
      float ka[8], kp[8], kq[8], mu[8];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float4 va = reinterpret_cast<const float4*>(tb)[h], vp = reinterpret_cast<const float4*>(tb + 8)[h];
        const float4 vq = reinterpret_cast<const float4*>(tb + 16)[h], vm = reinterpret_cast<const float4*>(tb + 24)[h];
        ka[4 * h] = va.x; ka[4 * h + 1] = va.y; ka[4 * h + 2] = va.z; ka[4 * h + 3] = va.w;
        kp[4 * h] = vp.x; kp[4 * h + 1] = vp.y; kp[4 * h + 2] = vp.z; kp[4 * h + 3] = vp.w;
        kq[4 * h] = vq.x; kq[4 * h + 1] = vq.y; kq[4 * h + 2] = vq.z; kq[4 * h + 3] = vq.w;
        mu[4 * h] = vm.x; mu[4 * h + 1] = vm.y; mu[4 * h + 2] = vm.z; mu[4 * h + 3] = vm.w;
      }
#pragma unroll
      for (int i = 0; i < VX; ++i) {
        u32x4 o;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t gw = r.x[i][d], yw = r.y[i][d];
          const float g0 = ((r.mk[i] >> (2 * d)) & 1u) ? __uint_as_float(gw << 16) : 0.f;
          const float g1 = ((r.mk[i] >> (2 * d + 1)) & 1u) ? __uint_as_float(gw & 0xffff0000u) : 0.f;
          const float v0 = bn_input_grad(g0, __uint_as_float(yw << 16), ka[2 * d], kp[2 * d], kq[2 * d], mu[2 * d]);
          const float v1 = bn_input_grad(g1, __uint_as_float(yw & 0xffff0000u), ka[2 * d + 1], kp[2 * d + 1], kq[2 * d + 1], mu[2 * d + 1]);
          o[d] = f2bf_pack(v0, v1);
        }
        *reinterpret_cast<u32x4*>(base + st_x + i * (RPG * RB)) = o;
      }
    } else {
#pragma unroll
      for (int i = 0; i < VX; ++i) *reinterpret_cast<u32x4*>(base + st_x + i * (RPG * RB)) = r.x[i];
    }
  };
  // fragment read offsets (bytes inside a tile) per MFMA k-step
  int fa_off[KS][NI], fb_off[KS][NJ];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    const int slot = kk * 2 + (lane >> 5);
#pragma unroll
    for (int i = 0; i < NI; ++i) fa_off[kk][i] = swz<NS>(wc * WC + i * 32 + (lane & 31), slot);
#pragma unroll
    for (int j = 0; j < NJ; ++j) fb_off[kk][j] = TC * RB + swz<NS>(wp * WP + j * 32 + (lane & 31), slot);
  }

  f32x16 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  {
    // tiles 0 .. PF are all requested before the first one is waited for
    RegSet first;
    fetch(first);
#pragma unroll
    for (int p = 0; p < PF; ++p) fetch(rs[p]);
    if (XF) {
      for (int i = tid; i < a.Cin; i += kThreads)
        reinterpret_cast<float4*>(xf_tab_lds)[i] = reinterpret_cast<const float4*>(a.xf_tab)[i];
      __syncthreads();
    }
    stash(0, first);
  }
  __syncthreads();
  auto step = [&](int t, RegSet& r) {
    const unsigned char* base = lds + (t & 1) * TILE_BYTES;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      Frag fa[NI], fb[NJ];
#pragma unroll
      for (int i = 0; i < NI; ++i) fa[i].u = *reinterpret_cast<const u32x4*>(base + fa_off[kk][i]);
#pragma unroll
      for (int j = 0; j < NJ; ++j) fb[j].u = *reinterpret_cast<const u32x4*>(base + fb_off[kk][j]);
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i].v, fb[j].v, acc[i][j], 0, 0, 0);
    }
    stash((t + 1) & 1, r);     // this register set holds tile t+1 (all zero past the end)
    fetch(r);                  // ... and now receives tile t+1+PF
    __syncthreads();
  };
  // main loop: whole groups of PF steps, no conditionals, so that the number of loads in flight
  // is the same on every path; then at most PF-1 guarded tail steps
  int kt = 0;
  for (; kt + PF <= ntiles; kt += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) step(kt + u, rs[u]);
  }
#pragma unroll
  for (int u = 0; u < PF - 1; ++u)
    if (kt + u < ntiles) step(kt + u, rs[u]);

  igemm_epilogue<TC, TP, WGC>(a, acc, lds, c0, m0, pt);
}

// ---- direct-to-LDS variant (contraction channels a multiple of 64) ---------------------------------
// Operand tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds: every lane names
// its own 16-byte source, the 64 vectors of a wave land contiguously at a wave-uniform LDS address):
// no staging registers and no ds_write, so four workgroups stay resident per CU with 64-wide k-tiles,
// whose 128-byte rows use whole cache lines (the vector L1 moves ~0.45 lines per clock whether a wave
// uses all of a line or half of it).  One LDS stage per workgroup: load tile t, wait, compute, and
// only then overwrite it; the load latency is covered by the other resident workgroups.
// The XOR swizzle of the 16-byte slots is applied on the source side: the lane that fills physical
// slot p of a row fetches logical k-slot p ^ f(row).
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// The loads go through buffer descriptors (buffer_load_dwordx4 ... lds): a lane's byte offset changes only with the
// filter tap, the position inside the tap is the scalar offset of the instruction, and a vector outside the image or
// the tensor carries the offset kOob, which lies beyond every descriptor's range: the hardware's range check then
// delivers zeros.  With flat addresses every load cost about nine vector instructions (64-bit address, zero-page
// select) and every k-tile a scalar load of the zero page's address.  Measured (3x3, us, flat -> buffer): 64 channels at
// 32x32, 512 images 66 -> 56; 128 at 16x16 46 -> 40; 64 at 56x56, 256 images 100 -> 88; 128 at 28x28 71 -> 64.
constexpr uint32_t kOob = 0xfffffff0u;     // operands hold fewer than 2^31 elements in whole vectors: at most kOob bytes
typedef __amdgpu_buffer_rsrc_t BufRsrc;
__device__ __forceinline__ BufRsrc buffer_of(const bf16_t* p, int64_t elements) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p), 0, (int)(uint32_t)(elements * 2), 0x00020000);
}
__device__ __forceinline__ void load_to_lds(BufRsrc r, unsigned char* dst, uint32_t lane_off, uint32_t uniform_off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_ptr)dst, 16, (int)lane_off, (int)uniform_off, 0, 0);
}

template <int TC, int TP, int WGC, int OCC, int BKT, class CL>
__global__ __launch_bounds__(kThreads, OCC) void igemm_dma_kernel(IgemmArgs a, CL cl) {
  constexpr int KS = BKT / 16, NS = BKT / 8;              // MFMA k-steps per tile; 16-byte slots per tile row
  constexpr int WGP = 4 / WGC;
  constexpr int WC = TC / WGC, WP = TP / WGP;
  constexpr int NI = WC / 32, NJ = WP / 32;
  constexpr int RB = BKT * 2, RPG = kThreads / NS;        // bytes per tile row; tile rows covered by one load per thread
  constexpr int VW = (TC + RPG - 1) / RPG, VX = TP / RPG;
  constexpr int TILE_BYTES = (VW * RPG + TP) * RB;       // weight rows rounded up to whole load sweeps
  constexpr int XBASE = VW * RPG * RB;
  constexpr int STG_STRIDE = TC * 2 + 16;
  constexpr int RED_BYTES = (kThreads / (TC / 8)) * (TC >= 128 ? 3 : 2) * TC * 4;
  constexpr int E_BYTES = TP * STG_STRIDE > RED_BYTES ? TP * STG_STRIDE : RED_BYTES;
  constexpr int LDS_BYTES = TILE_BYTES > E_BYTES ? TILE_BYTES : E_BYTES;
  static_assert(TP % RPG == 0 && (BKT == 32 || BKT == 64), "tile rows must be whole load sweeps");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS_BYTES];

  const int bid = enter_class(a, cl, blockIdx.x);
  const int q = bid >> 3;
  const int ct = q % a.nct;
  const int pt = a.xcd_contiguous ? (bid & 7) * ((a.npt + 7) >> 3) + (q / a.nct) : (q / a.nct) * 8 + (bid & 7);
  if (pt >= a.npt) return;
  const int c0 = ct * TC, m0 = pt * TP;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % WGC, wp = wave / WGC;
  const int lrow = tid / NS;
  // logical k-slot behind physical slot tid % NS of row lrow: the XOR of swz<NS> is its own inverse
  const int kvec = (swz<NS>(lrow, tid % NS) - lrow * RB) >> 4;

  int hb[VX], wb[VX], nb[VX]; bool mv[VX];
  const int HW = a.Hout * a.Wout;
#pragma unroll
  for (int i = 0; i < VX; ++i) {
    const int m = m0 + lrow + RPG * i;
    mv[i] = m < a.M;
    const int mm = mv[i] ? m : 0;
    const int n = mm / HW, rem = mm - n * HW;
    const int ho = rem / a.Wout, wo = rem - ho * a.Wout;
    hb[i] = ho * a.ostride - a.pad_h; wb[i] = wo * a.ostride - a.pad_w;
    nb[i] = n * a.Hin * a.Win;
  }
  const int ntiles = a.Ktot / BKT;
  const int ps = a.xstride ? a.xstride : a.Cin;         // elements between neighbouring input pixels
  const int xcol = (kvec * 8) / ps;                     // pixel this thread's vector lies in, relative to the tap (0 unless xstride is set)
  const BufRsrc wbuf = buffer_of(a.wt, (int64_t)a.Cout * a.Ktot), xbuf = buffer_of(a.in, (int64_t)a.B * a.Hin * a.Win * ps);
  uint32_t woff[VW], xoff[VX];                            // byte offsets of this thread's vectors (kOob: zeros)
#pragma unroll
  for (int i = 0; i < VW; ++i) {
    const int c = c0 + lrow + RPG * i;
    woff[i] = ((lrow + RPG * i < TC) & (c < a.Cout)) ? (uint32_t)(c * a.Ktot + kvec * 8) * 2u : kOob;
  }
  uint32_t wk = 0;                                        // bytes into the weight rows
  int kc0 = 0, kr = 0, ks = 0;
  unsigned char* const wave_base = lds + wave * 1024;     // a wave's 64 vectors = 1 KB of consecutive tile rows
  // all loads of the next k-tile (a tile never straddles a filter tap: the tap, the bounds test and the
  // pixel offset change only every Cin/64 tiles, a uniform branch)
  auto fetch = [&]() {
#pragma unroll
    for (int i = 0; i < VW; ++i)
      load_to_lds(wbuf, wave_base + i * (RPG * RB), woff[i], wk);
    wk += BKT * 2;
    if (kc0 == 0) {
#pragma unroll
      for (int i = 0; i < VX; ++i) {
        const int hi = hb[i] + kr, wi = wb[i] + ks;
        const bool ok = mv[i] & (hi >= 0) & (wi + xcol >= 0) & (hi < a.Hin) & (wi + xcol < a.Win);
        xoff[i] = ok ? (uint32_t)((nb[i] + hi * a.Win + wi) * ps + kvec * 8) * 2u : kOob;
      }
    }
#pragma unroll
    for (int i = 0; i < VX; ++i) load_to_lds(xbuf, wave_base + XBASE + i * (RPG * RB), xoff[i], (uint32_t)kc0 * 2u);
    kc0 += BKT;
    if (kc0 == a.Cin) { kc0 = 0; if (++ks == a.KW) { ks = 0; ++kr; } }
  };
  // fragment byte offsets for k-step 0; k-step kk is the slot pair 2*kk further on, i.e. offset ^ (kk * 32)
  int fa_off[NI], fb_off[NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i) fa_off[i] = swz<NS>(wc * WC + i * 32 + (lane & 31), lane >> 5);
#pragma unroll
  for (int j = 0; j < NJ; ++j) fb_off[j] = XBASE + swz<NS>(wp * WP + j * 32 + (lane & 31), lane >> 5);

  f32x16 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  for (int t = 0; t < ntiles; ++t) {
    fetch();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's vectors have landed ...
    __builtin_amdgcn_s_barrier();                         // ... and so have everyone else's
    Frag fa[2][NI], fb[2][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i) fa[0][i].u = *reinterpret_cast<const u32x4*>(lds + fa_off[i]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) fb[0][j].u = *reinterpret_cast<const u32x4*>(lds + fb_off[j]);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      if (kk + 1 < KS) {                                   // fragments of the next k-step under this one's MFMAs
#pragma unroll
        for (int i = 0; i < NI; ++i) fa[(kk + 1) & 1][i].u = *reinterpret_cast<const u32x4*>(lds + (fa_off[i] ^ ((kk + 1) * 32)));
#pragma unroll
        for (int j = 0; j < NJ; ++j) fb[(kk + 1) & 1][j].u = *reinterpret_cast<const u32x4*>(lds + (fb_off[j] ^ ((kk + 1) * 32)));
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1][i].v, fb[kk & 1][j].v, acc[i][j], 0, 0, 0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();                         // everyone is done reading before the stage is overwritten
  }
  igemm_epilogue<TC, TP, WGC>(a, acc, lds, c0, m0, pt);
}

// Blocks of a launch in tiles of TP pixels; for a launch in classes also their block ranges.
template <int TP>
unsigned plan_blocks(IgemmArgs& a, NoClasses&) {
  a.npt = (a.M + TP - 1) / TP;
  return (unsigned)((a.npt + 7) / 8 * 8 * a.nct);
}
template <int TP>
unsigned plan_blocks(IgemmArgs& a, IgemmClasses& cl) {
  int blocks = 0;
  for (int i = 0; i < cl.n; ++i) {
    cl.c[i].npt = (cl.c[i].M + TP - 1) / TP;
    cl.c[i].begin = blocks;
    blocks += (cl.c[i].npt + 7) / 8 * 8 * a.nct;
  }
  return (unsigned)blocks;
}

template <int TC, int TP, int WGC, int OCC, int BKT = 64, class CL = NoClasses>
dat_status launch_igemm_dma(IgemmArgs a, hipStream_t st, CL cl = CL{}) {
  if ((int64_t)a.B * a.Hin * a.Win * a.Cin >= (1ll << 31) || (int64_t)a.Cout * a.Ktot >= (1ll << 31)) return DAT_ERR_UNSUPPORTED;
  if (a.Cin % BKT != 0 || a.Ktot < BKT || a.Ktot % BKT != 0) return DAT_ERR_UNSUPPORTED;
  if (a.xstride && (a.Cin != BKT || a.xstride % 8 != 0 || a.Cin % a.xstride != 0)) return DAT_ERR_UNSUPPORTED;   // one tap per k-tile
  a.nct = (a.Cout + TC - 1) / TC;
  const unsigned blocks = plan_blocks<TP>(a, cl);
  if (blocks == 0) return DAT_OK;
  a.xcd_contiguous = a.KH * a.KW > 1;   // filter windows: neighbouring tiles re-read each other's rows
  if (recorded(a, cl, kSingleStage, TC, TP, 1, BKT, 0)) return DAT_OK;
  hipLaunchKernelGGL((igemm_dma_kernel<TC, TP, WGC, OCC, BKT, CL>), dim3(blocks), dim3(kThreads), 0, st, a, cl);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

// ---- ring variant: layers with at most a few workgroups per CU --------------------------------------------------
// S LDS stages of 64-wide k-tiles filled by the same direct-to-LDS loads, NT / 64 waves, one or two workgroups per CU.
// The single-stage kernel hides its load latency behind other workgroups; a layer that has none to offer (few tiles)
// or that is faster in tiles too large for four workgroups per CU hides it behind the S - 1 k-tiles in flight here.
// What then bounds a k-tile is the chain barrier -> LDS reads -> MFMA.  So the fragments of the next group of G
// k-steps are read (into the other half of a register double buffer) before the current group is multiplied, across
// the tile boundary too: the barrier stands in front of a tile's last group, when every wave has finished reading the
// stage, so that the next tile's first reads and the refill of the stage run under that group's MFMAs.  G = 4 (a whole
// tile) where two sets of fragments fit the registers, else 1.
// Measured (3x3 layers, forward, us; single-stage kernels -> ring): 512 channels at 4x4, 13 images 47 -> 18
// (32 x 128 tiles), 512 images 63 -> 38 (128 x 128); 7x7, 85 images 51 -> 33; 5x5, 50 images 49 -> 20; 256 channels at
// 14x14, 85 images 40 -> 28 (256 x 128); 320 channels at 16x16, 256 images 138 -> 106 and 640 at 8x8 133 -> 100 = 1.2
// PFLOP/s (160 x 256).
// ANYC: the contraction channels are no multiple of the k-tile (160 channels, 64-wide tiles), so a tile straddles
// filter taps: every lane follows the tap and channel of its own 16-byte vector (a vector never straddles: Cin % 8
// == 0), and the last tile is padded with zeros.
template <int TC, int TP, int WGC, int S, int NT, int G, bool ANYC, class CL>
__global__ __launch_bounds__(NT) void igemm_ring_kernel(IgemmArgs a, CL cl) {
  constexpr int BKT = 64, KS = BKT / 16, NG = KS / G;       // MFMA k-steps per tile, in NG groups of G
  constexpr int WGP = NT / 64 / WGC;
  constexpr int WC = TC / WGC, WP = TP / WGP;
  constexpr int NI = WC / 32, NJ = WP / 32;
  constexpr int RB = 128, RPG = NT / 8;                   // bytes per tile row; tile rows covered by one load per thread
  constexpr int VW = (TC + RPG - 1) / RPG, VX = TP / RPG;
  constexpr int NL = VW + VX;                             // loads per thread per tile
  constexpr bool PART = TC % RPG != 0;                    // the last weight sweep is short: its upper waves have no load
  constexpr int NLMIN = PART ? NL - 1 : NL;               // loads every wave issues per tile
  constexpr int TILE_BYTES = (TC + TP) * RB;
  constexpr int STG_BYTES = TP * (TC * 2 + 16);
  constexpr int RED_BYTES = (NT / (TC / 8)) * 3 * TC * 4;
  constexpr int E_BYTES = STG_BYTES > RED_BYTES ? STG_BYTES : RED_BYTES;
  constexpr int LDS_BYTES = (S * TILE_BYTES > E_BYTES) ? S * TILE_BYTES : E_BYTES;
  static_assert(TC % 8 == 0 && TP % RPG == 0, "pixel rows must be whole load sweeps, weight rows whole waves");
  static_assert(S >= 2 && (S - 1) * NL <= 63, "vmcnt range");
  static_assert(LDS_BYTES <= 163840, "LDS of a CU");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS_BYTES];

  const int bid = enter_class(a, cl, blockIdx.x);
  const int q = bid >> 3;
  const int ct = q % a.nct, pt = (q / a.nct) * 8 + (bid & 7);
  if (pt >= a.npt) return;
  const int c0 = ct * TC, m0 = pt * TP;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % WGC, wp = wave / WGC;
  const int lrow = tid >> 3;
  const int kvec = (swz<8>(lrow, tid & 7) - lrow * RB) >> 4;   // logical k-slot behind physical slot tid & 7 of row lrow

  int hb[VX], wb[VX], nb[VX]; bool mv[VX];
  const int HW = a.Hout * a.Wout;
#pragma unroll
  for (int i = 0; i < VX; ++i) {
    const int m = m0 + lrow + RPG * i;
    mv[i] = m < a.M;
    const int mm = mv[i] ? m : 0;
    const int n = mm / HW, rem = mm - n * HW;
    const int ho = rem / a.Wout, wo = rem - ho * a.Wout;
    hb[i] = ho * a.ostride - a.pad_h; wb[i] = wo * a.ostride - a.pad_w;
    nb[i] = n * a.Hin * a.Win;
  }
  const int ntiles = ANYC ? (a.Ktot + BKT - 1) / BKT : a.Ktot / BKT;
  const BufRsrc wbuf = buffer_of(a.wt, (int64_t)a.Cout * a.Ktot), xbuf = buffer_of(a.in, (int64_t)a.B * a.Hin * a.Win * a.Cin);
  uint32_t woff[VW], xoff[VX];                            // byte offsets of this thread's vectors (kOob: zeros)
#pragma unroll
  for (int i = 0; i < VW; ++i) {
    const int c = c0 + lrow + RPG * i;
    woff[i] = ((lrow + RPG * i < TC) & (c < a.Cout)) ? (uint32_t)(c * a.Ktot + kvec * 8) * 2u : kOob;
  }
  int kc0 = 0, kr = 0, ks = 0, kf = 0;
  uint32_t wk = 0;                                        // bytes into the weight rows
  int kc, gr, gs, kw = kvec * 8;                          // ANYC: channel and tap of this lane's vector, its k index
  {
    const int tap = kw / a.Cin;
    kc = kw - tap * a.Cin; gr = tap / a.KW; gs = tap - gr * a.KW;
  }
  unsigned char* sb = lds;
  // the loads of tile kf into ring stage `stage`, one at a time (past the end the last tile is fetched again, so that
  // every tile issues the same number of loads and the vmcnt arithmetic stays exact)
  auto fetch_begin = [&](int stage) { sb = lds + stage * TILE_BYTES + wave * 1024; };
  auto fetch_w = [&](int i) {
    if (PART && i == VW - 1 && wave * 8 + RPG * i >= TC) return;   // (uniform: a wave's load is 8 rows)
    load_to_lds(wbuf, sb + i * (RPG * RB), (!ANYC || kw < a.Ktot) ? woff[i] : kOob, wk);
  };
  auto fetch_tap = [&]() {
    if (!ANYC && kc0 != 0) return;
#pragma unroll
    for (int i = 0; i < VX; ++i) {
      const int r = ANYC ? gr : kr, c = ANYC ? gs : ks;
      const int hi = hb[i] + r, wi = wb[i] + c;
      const bool ok = mv[i] & (r < a.KH) & (hi >= 0) & (wi >= 0) & (hi < a.Hin) & (wi < a.Win);
      xoff[i] = ok ? (uint32_t)((nb[i] + hi * a.Win + wi) * a.Cin + (ANYC ? kc : kvec * 8)) * 2u : kOob;
    }
  };
  auto fetch_x = [&](int i) { load_to_lds(xbuf, sb + TC * RB + i * (RPG * RB), xoff[i], ANYC ? 0u : (uint32_t)kc0 * 2u); };
  auto fetch_end = [&]() {
    if (++kf >= ntiles) return;
    wk += BKT * 2;
    if (ANYC) {
      kw += BKT; kc += BKT;
      while (kc >= a.Cin) { kc -= a.Cin; if (++gs == a.KW) { gs = 0; ++gr; } }
    } else {
      kc0 += BKT;
      if (kc0 == a.Cin) { kc0 = 0; if (++ks == a.KW) { ks = 0; ++kr; } }
    }
  };
  int fa_off[NI], fb_off[NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i) fa_off[i] = swz<8>(wc * WC + i * 32 + (lane & 31), lane >> 5);
#pragma unroll
  for (int j = 0; j < NJ; ++j) fb_off[j] = TC * RB + swz<8>(wp * WP + j * 32 + (lane & 31), lane >> 5);

  f32x16 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

#pragma unroll 1
  for (int p = 0; p < S; ++p) {
    fetch_begin(p);
#pragma unroll
    for (int i = 0; i < VW; ++i) fetch_w(i);
    fetch_tap();
#pragma unroll
    for (int i = 0; i < VX; ++i) fetch_x(i);
    fetch_end();
  }
  Frag fa[2][G][NI], fb[2][G][NJ];
  auto read_group = [&](const unsigned char* base, int g, int buf) {
#pragma unroll
    for (int u = 0; u < G; ++u) {
#pragma unroll
      for (int i = 0; i < NI; ++i) fa[buf][u][i].u = *reinterpret_cast<const u32x4*>(base + (fa_off[i] ^ ((g * G + u) * 32)));
#pragma unroll
      for (int j = 0; j < NJ; ++j) fb[buf][u][j].u = *reinterpret_cast<const u32x4*>(base + (fb_off[j] ^ ((g * G + u) * 32)));
    }
  };
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * NLMIN) : "memory");
  __builtin_amdgcn_s_barrier();
  read_group(lds, 0, 0);
  int stage = 0;
  auto tile = [&](int par) {                              // par: register buffer that holds the tile's first group
    const unsigned char* cur = lds + stage * TILE_BYTES;
    const int nstage = stage + 1 == S ? 0 : stage + 1;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int buf = (par + g) & 1;
      if (g == NG - 1) {
        // all of this wave's reads of the stage are done and its part of tile t+1 has landed (at most S-2 tiles of
        // loads outstanding); behind the barrier that holds for every wave: the next tile can be read, the stage refilled
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * NLMIN) : "memory");
        __builtin_amdgcn_s_barrier();
        read_group(lds + nstage * TILE_BYTES, 0, buf ^ 1);
        fetch_begin(stage);
      } else {
        read_group(cur, g + 1, buf ^ 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < G; ++u)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][u][i].v, fb[buf][u][j].v, acc[i][j], 0, 0, 0);
          if (g == NG - 1) {   // tile t+S, spread over this group's MFMAs: weights first, then pixels
#pragma unroll
            for (int l = 0; l < NL; ++l)
              if (l * (G * NI) / NL == u * NI + i) {
                if (l < VW) fetch_w(l);
                else { if (l == VW) fetch_tap(); fetch_x(l - VW); }
              }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    fetch_end();
    stage = nstage;
  };
  if (NG & 1) {
    int t = 0;
    for (; t + 2 <= ntiles; t += 2) { tile(0); tile(1); }
    if (t < ntiles) tile(0);
  } else {
    for (int t = 0; t < ntiles; ++t) tile(0);
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // the loads past the end land in LDS too
  __builtin_amdgcn_s_barrier();
  igemm_epilogue<TC, TP, WGC, NT>(a, acc, lds, c0, m0, pt);
}

template <int TC, int TP, int WGC, int S, int NT, int G, bool ANYC = false, class CL = NoClasses>
dat_status launch_igemm_ring(IgemmArgs a, hipStream_t st, CL cl = CL{}) {
  if ((int64_t)a.B * a.Hin * a.Win * a.Cin >= (1ll << 31) || (int64_t)a.Cout * a.Ktot >= (1ll << 31)) return DAT_ERR_UNSUPPORTED;
  if (a.Ktot < 64 || a.xf_tab || a.xstride) return DAT_ERR_UNSUPPORTED;
  if (ANYC ? (a.Cin % 8 != 0 || a.Ktot != a.KH * a.KW * a.Cin) : a.Cin % 64 != 0) return DAT_ERR_UNSUPPORTED;
  a.nct = (a.Cout + TC - 1) / TC;
  const unsigned blocks = plan_blocks<TP>(a, cl);
  if (blocks == 0) return DAT_OK;
  if (recorded(a, cl, kMultiStage, TC, TP, S, 64, ANYC)) return DAT_OK;
  hipLaunchKernelGGL((igemm_ring_kernel<TC, TP, WGC, S, NT, G, ANYC, CL>), dim3(blocks), dim3(NT), 0, st, a, cl);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

__global__ void widen_kernel(const bf16_t* __restrict__ src, float* __restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = bf2f(src[i]);
}

// OCC: waves per SIMD the register allocation is held to (1 = no constraint)
// 1x1 stride-1 layers whose operand is transformed on the way into LDS (see IgemmArgs::xf_x)
template <int TC, int TP, int WGC, int PF, int BKT, int OCC>
dat_status launch_igemm_xf(IgemmArgs a, hipStream_t st) {
  if ((int64_t)a.B * a.Hin * a.Win * a.Cin >= (1ll << 31) || (int64_t)a.Cout * a.Ktot >= (1ll << 31)) return DAT_ERR_UNSUPPORTED;
  if (a.KH != 1 || a.KW != 1 || a.ostride != 1 || a.Cin % BKT != 0 || a.Ktot != a.Cin) return DAT_ERR_UNSUPPORTED;
  const size_t tab_bytes = (size_t)a.Cin * kBnTabFloatsPerChannel * sizeof(float);
  if (tab_bytes > 32768) return DAT_ERR_UNSUPPORTED;
  a.nct = (a.Cout + TC - 1) / TC;
  a.npt = (a.M + TP - 1) / TP;
  if (a.npt == 0) return DAT_OK;
  a.xcd_contiguous = 0;
  if (recorded(a, NoClasses{}, kRegisterStaged, TC, TP, 1, BKT, 0)) return DAT_OK;
  const int npt8 = (a.npt + 7) / 8 * 8;
  hipLaunchKernelGGL((igemm_kernel<TC, TP, WGC, PF, true, BKT, OCC, true>), dim3((unsigned)(npt8 * a.nct)), dim3(kThreads), tab_bytes, st, a);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

template <int TC, int TP, int WGC, int PF, int BKT, int OCC = 1>
dat_status launch_igemm(IgemmArgs a, hipStream_t st) {
  // 32-bit element offsets inside the kernel
  if ((int64_t)a.B * a.Hin * a.Win * a.Cin >= (1ll << 31) || (int64_t)a.Cout * a.Ktot >= (1ll << 31)) return DAT_ERR_UNSUPPORTED;
  a.nct = (a.Cout + TC - 1) / TC;
  a.npt = (a.M + TP - 1) / TP;
  if (a.npt == 0) return DAT_OK;
  a.xcd_contiguous = a.KH * a.KW > 1;   // filter windows: neighbouring tiles re-read each other's rows
  if (recorded(a, NoClasses{}, kRegisterStaged, TC, TP, 1, BKT, a.Cin % BKT != 0)) return DAT_OK;
  const int npt8 = (a.npt + 7) / 8 * 8;
  if (a.Cin % BKT == 0 && a.Ktot > 0)
    hipLaunchKernelGGL((igemm_kernel<TC, TP, WGC, PF, true, BKT, OCC>), dim3((unsigned)(npt8 * a.nct)), dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL((igemm_kernel<TC, TP, WGC, PF, false, BKT, OCC>), dim3((unsigned)(npt8 * a.nct)), dim3(kThreads), 0, st, a);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

template <int TC, int TP, int WGC>
dat_status pick_depth(const IgemmArgs& a, hipStream_t st) {
  // short contractions (1x1 layers with few input channels) gain nothing from deep prefetch;
  // long ones use 64-wide k-tiles (half the barriers per MFMA) when a tile cannot straddle a tap
  if (a.Ktot <= 128) return launch_igemm<TC, TP, WGC, 1, 32>(a, st);
  if (a.Cin % 64 == 0) return launch_igemm<TC, TP, WGC, 2, 64>(a, st);
  return launch_igemm<TC, TP, WGC, 3, 32>(a, st);
}

// 128-channel tiles, measured over the ResNet-50 layer shapes: four resident workgroups per CU beat
// two workgroups with deep register prefetch on every layer; when the contraction channels are a
// multiple of 64 the direct-to-LDS kernel (whole cache lines, no staging registers) is another
// ~10 % faster than the register-staged one with 32-wide k-tiles.
dat_status pick_depth_wide(const IgemmArgs& a, hipStream_t st) {
  if (a.Cin % 64 == 0 && a.Ktot >= 64) return launch_igemm_dma<128, 128, 2, 4>(a, st);
  return launch_igemm<128, 128, 2, 1, 32, 4>(a, st);
}

std::atomic<int64_t> g_launches{0};

int compute_units() {
  static std::atomic<int> cached{0};
  int n = cached.load(std::memory_order_relaxed);
  if (n == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached.store(n, std::memory_order_relaxed);
  }
  return n;
}

std::atomic<bool> g_ring_enabled{true};
std::atomic<bool> g_tile160{true};
std::atomic<bool> g_narrow_underfilled{true};

// The switches of dat_set_kernel_option, read once per convolution: the slab count a reduction is given and the tiles that
// write the slabs follow from the same values, whatever another thread sets meanwhile.
struct Switches { bool ring, tile160, narrow; };
Switches read_switches() {
  return {g_ring_enabled.load(std::memory_order_relaxed), g_tile160.load(std::memory_order_relaxed), g_narrow_underfilled.load(std::memory_order_relaxed)};
}

// Which ring configuration, if any, runs this launch.  The lines are drawn by tiles per CU (256 CUs), measured on the
// 3x3 and 1x1 layers of every network at batches of 13 to 512, us:
//  * kR160x256 / kR160x128: widths that are a multiple of 160 (the wide ResNets).  Every wave takes all 160 channels of 32
//    pixels: no empty MFMA rows, and the gathered activations are fetched once per 160 channels.  One 256-pixel tile
//    per CU at a time, or two 128-pixel ones; the same work per round, the larger tile 2-5 % faster (640 channels, 256
//    images 99.7 / 106.7).  With an odd number of 128-pixel tiles per CU the larger tile would leave half of its last
//    round idle (640 channels, 128 images, one tile per CU: 72 / 63).
//  * kR256x256, kR256x128: contraction >= 1024 into a multiple of 256 channels, one round over at least 60 % (more than half)
//    of the CUs.  (On exactly half of them the 128x128 tiles below are one full round: 4x4 512 -> 512 at 512 images 50.8, 128x128
//    37.4; 8x8 256 -> 256 at 256 images 29.0, 22.0; 1x1 2048 -> 512 at 8x8, 128 images 27.9, 21.0.)
//    14x14 256 -> 256 at 256 images 65 (128x128 tiles) -> 56, 7x7 512 -> 512 75 -> 58; 14x14 at 85 images (131 tiles) 40 -> 28.
//  * at most one 128x128 tile per CU, contraction >= 256: the largest tile that still gives half of the CUs one.
//    128x128 above half a tile per CU (20x20 128 -> 128 at 50 images 16.1 -> 12.4; 64x128 tiles 12.9), 64x128 above a
//    quarter (10x10 256 -> 256 at 50 images 22.8 -> 15.4; 32x128 17.2, 128x128 19.1), else 32x128 (5x5 512 -> 512 at 50
//    images 48.8 -> 19.6; 64x128 25.6).  The line is at one tile per CU: between 1.0 and 1.5 the single-stage 128x128 kernel is
//    ahead (16x16 128 -> 128 at 160 images 21.2, ring 128x128 25.1, 64x128 24.1, 32x128 28.2, single-stage 32x128 24.8; 28x28
//    at 42 and 61 images 19.0 and 20.3, next best 22.1 and 22.8; the only tie 1x1 1024 -> 128 at 28x28, 60 images, 22.2, 64x128
//    22.0).
enum RingPick { kRNone, kR32, kR64, kR128, kR256x128, kR256x256, kR160x128, kR160x256, kR160x128Any, kR160x256Any };

RingPick pick_ring(const IgemmArgs& a, const Switches& sw) {
  if (a.xf_tab || a.xstride || a.Cin % 8 != 0 || a.Ktot < 256 || a.KH * a.KW * a.Cin != a.Ktot) return kRNone;
  const int64_t cus = compute_units(), p128 = ((int64_t)a.M + 127) / 128, p256 = ((int64_t)a.M + 255) / 256;
  const bool one_grid = a.ostep == 1 && a.stat_slab0 == 0;       // 256-pixel tiles: the whole tensor is this launch
  if (a.Cout % 160 == 0 && (a.Cin % 64 == 0 || a.Ktot >= 512) && sw.tile160) {
    const int64_t per_cu = (p128 * (a.Cout / 160) + cus - 1) / cus;
    const bool any = a.Cin % 64 != 0;
    // 640 channels over few pixels: 128 divides them too, and the narrower tiles below give more CUs work
    if (a.Cout % 128 != 0 || any || 2 * p128 * (a.Cout / 160) > cus) {
      if (one_grid && per_cu % 2 == 0) return any ? kR160x256Any : kR160x256;
      return any ? kR160x128Any : kR160x128;
    }
  }
  if (a.Cin % 64 != 0) return kRNone;
  if (one_grid && a.Ktot >= 1024 && a.Cout % 256 == 0 && sw.ring) {
    const int64_t nct = a.Cout / 256, t256 = p256 * nct, t128 = p128 * nct;
    if (t256 <= cus && 5 * t256 >= 3 * cus) return kR256x256;
    if (t128 <= cus && 2 * t128 > cus) return kR256x128;
  }
  if (!sw.narrow) return kRNone;
  // A backward-data pass that igemm_kernel may also run with its operand transform (conv_mfma_bn_operand_ok) leaves its
  // batch-norm sums in the same order either way: 64-channel tiles of 256 threads, or the 128-channel single-stage kernel
  // (whose 128x128 tiles the 512-thread multi-stage ones would beat: 1x1 512 -> 128 at 28x28, 21 images 12.3 us, multi-stage 8.4;
  // but a thread's rows there are others, and the two settings of the operand transform promise identical bits).
  if (a.stat_mode >= 2 && a.KH * a.KW == 1 && a.ostep == 1 && a.Cout > 32 && a.Cout <= 128 && a.Cin >= 2 * a.Cout)
    return a.Cout <= 64 && 2 * p128 <= cus ? kR64 : kRNone;
  const int64_t t = p128 * ((a.Cout + 127) / 128);
  if (a.Cout > 64 && t <= cus) return 2 * t > cus ? kR128 : 4 * t > cus ? kR64 : kR32;
  if (a.Cout <= 64 && 2 * p128 <= cus) return kR32;
  return kRNone;
}

// pixel rows per tile (= per slab of epilogue statistics) of the configuration run_igemm launches
int pixel_tile(RingPick r) {
  return r == kR256x256 || r == kR160x256 || r == kR160x256Any ? 256 : 128;
}

dat_status run_igemm(const IgemmArgs& a, const Switches& sw, RingPick ring, hipStream_t st) {
  if (!t_record) g_launches.fetch_add(1, std::memory_order_relaxed);
  if (a.Cin % 8 != 0 || a.Cout % 8 != 0) return DAT_ERR_UNSUPPORTED;
  if (a.stat_mode == 3 && (a.Cout <= 64 || a.xf_tab)) return DAT_ERR_UNSUPPORTED;   // three sums: the <= 64-channel kernels have no LDS for them
  if (a.xstride) {   // overlapping input pixels: the direct-to-LDS kernel with one tap per 64-wide k-tile
    if (a.Cout > 64 || a.xf_tab) return DAT_ERR_UNSUPPORTED;
    return a.Cout <= 32 ? launch_igemm_dma<32, 128, 1, 6>(a, st) : launch_igemm_dma<64, 128, 2, 5>(a, st);
  }
  switch (ring) {
    case kR32: return launch_igemm_ring<32, 128, 1, 4, 256, 4>(a, st);
    case kR64: return launch_igemm_ring<64, 128, 2, 3, 256, 4>(a, st);
    case kR128: return launch_igemm_ring<128, 128, 2, 4, 512, 4>(a, st);
    case kR256x128: return launch_igemm_ring<256, 128, 4, 3, 512, 1>(a, st);
    case kR256x256: return launch_igemm_ring<256, 256, 2, 2, 512, 1>(a, st);
    case kR160x128: return launch_igemm_ring<160, 128, 1, 2, 256, 1>(a, st);
    case kR160x256: return launch_igemm_ring<160, 256, 1, 3, 512, 1>(a, st);
    case kR160x128Any: return launch_igemm_ring<160, 128, 1, 2, 256, 1, true>(a, st);
    case kR160x256Any: return launch_igemm_ring<160, 256, 1, 3, 512, 1, true>(a, st);
    case kRNone: break;
  }
  if (a.xf_tab) {
    // 64-channel results (contraction 256, four k-tiles): one register set in flight and three workgroups per CU
    // beat two sets at two workgroups (15.6 -> 14.8 ms per step over these launches); for the 128-channel results the
    // same change gained nothing
    if (a.Cout <= 64) return launch_igemm_xf<64, 128, 2, 1, 64, 3>(a, st);
    return launch_igemm_xf<128, 128, 2, 2, 32, 2>(a, st);
  }
  // short contractions into a multiple of 160 channels that 128 does not divide: 160-channel tiles, direct to LDS where a
  // 64-wide k-tile divides the contraction (14x14, 128 images, us, register-staged -> direct: 1x1 192 -> 160 9.6 -> 8.3,
  // 128 -> 480 13.2 -> 12.1; 16 images 64 -> 160 6.3 -> 5.8)
  if (a.Cout % 160 == 0 && a.Cout % 128 != 0 && sw.tile160) {
    if (a.Cin % 64 == 0 && a.Ktot >= 64) return launch_igemm_dma<160, 128, 1, 3>(a, st);
    return launch_igemm<160, 128, 1, 1, 32, 3>(a, st);
  }
  // narrow channel tiles: the direct-to-LDS kernel wherever its k-tile divides the contraction channels,
  // except 1x1 layers with a long contraction into <= 64 channels (HBM-bound reads: deep register
  // prefetch with two workgroups per CU streams them at the copy rate)
  if (a.Cout <= 32) {
    if (a.Cin % 64 == 0 && a.Ktot >= 64) return launch_igemm_dma<32, 128, 1, 6>(a, st);
    return pick_depth<32, 128, 1>(a, st);
  }
  if (a.Cout <= 64) {
    if (a.Cin % 64 == 0 && a.Ktot >= 64 && (a.KH * a.KW > 1 || a.Ktot < 256)) return launch_igemm_dma<64, 128, 2, 5>(a, st);
    if (a.Cin % 64 != 0 && a.Cin % 32 == 0 && a.Ktot >= 32) return launch_igemm_dma<64, 128, 2, 5, 32>(a, st);
    return pick_depth<64, 128, 2>(a, st);
  }
  return pick_depth_wide(a, st);
}

// The classes of one backward-data pass as one launch, if a kernel takes them that way (*done); `a` carries the values of
// the class with most taps.  128-pixel tiles; the rules are those of pick_ring and run_igemm for the sum of the tiles.
dat_status run_igemm_classes(const IgemmArgs& a, const Switches& sw, const IgemmClasses& cl, hipStream_t st, bool* done) {
  *done = false;
  const bool tile160 = a.Cout % 160 == 0 && sw.tile160, any = a.Cin % 64 != 0;
  if (any && !(tile160 && a.Ktot >= 512)) return DAT_OK;
  if (a.Ktot < 64 || a.Cin % 8 != 0 || a.Cout % 8 != 0 || a.xf_tab || a.xstride || (a.stat_mode == 3 && a.Cout <= 64)) return DAT_OK;
  *done = true;
  if (!t_record) g_launches.fetch_add(1, std::memory_order_relaxed);
  int64_t tiles = 0;
  for (int i = 0; i < cl.n; ++i) tiles += (cl.c[i].M + 127) / 128;
  const int64_t cus = compute_units(), t = tiles * ((a.Cout + 127) / 128);
  if (any) return launch_igemm_ring<160, 128, 1, 2, 256, 1, true>(a, st, cl);
  if (tile160 && (a.Cout % 128 != 0 || 2 * tiles * (a.Cout / 160) > cus)) return launch_igemm_ring<160, 128, 1, 2, 256, 1>(a, st, cl);
  if (sw.narrow && a.Cout > 64 && t <= cus) {
    if (2 * t > cus) return launch_igemm_ring<128, 128, 2, 4, 512, 4>(a, st, cl);
    if (4 * t > cus) return launch_igemm_ring<64, 128, 2, 3, 256, 4>(a, st, cl);
    return launch_igemm_ring<32, 128, 1, 4, 256, 4>(a, st, cl);
  }
  if (sw.narrow && a.Cout <= 64 && 2 * tiles <= cus) return launch_igemm_ring<32, 128, 1, 4, 256, 4>(a, st, cl);
  if (a.Cout <= 32) return launch_igemm_dma<32, 128, 1, 6>(a, st, cl);
  if (a.Cout <= 64) return launch_igemm_dma<64, 128, 2, 5>(a, st, cl);
  return launch_igemm_dma<128, 128, 2, 4>(a, st, cl);
}

// ---- weight layouts ---------------------------------------------------------------------------
// master fp32 [Cout][k][k][cin_real] -> w [Cout][k][k][Cin] bf16 (zero padded channels) and the
// backward-data operand wT.
//   stride 1: wT [Cin][k][k][Cout], wT[ci][r'][s'][co] = w[co][k-1-r'][k-1-s'][ci].
//   stride 2: the input pixels split into four parity classes (h%2, w%2); class (ph,pw) only sees
//     the taps r = rf + 2i, s = sf + 2j with rf = (ph+pad)%2, sf = (pw+pad)%2, and is a dense
//     stride-1 convolution of dY with that nr x ns sub-filter.  wT holds the four flipped
//     sub-filters back to back: class q = 2*ph+pw at offset Cin*Cout*(taps of earlier classes),
//     laid out [Cin][nr][ns][Cout].
struct ParityClass { int rf, nr, pad; };
__host__ __device__ inline ParityClass parity_class(int p, int k, int pad) {
  ParityClass c;
  c.rf = (p + pad) & 1;
  c.nr = (k - c.rf + 1) / 2;
  if (c.rf >= k) c.nr = 0;
  const int off = (p + pad - c.rf) / 2;
  c.pad = c.nr - 1 - off;
  return c;
}

__global__ void weight_transform_kernel(const float* __restrict__ master, bf16_t* __restrict__ w, bf16_t* __restrict__ wT,
                                        int Cout, int k, int cin_real, int Cin, int stride, int pad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)Cout * k * k * Cin) return;
  const int ci = (int)(i % Cin);
  int64_t p = i / Cin;
  const int s = (int)(p % k); p /= k;
  const int r = (int)(p % k);
  const int co = (int)(p / k);
  const bf16_t v = ci < cin_real ? f2bf(master[(((int64_t)co * k + r) * k + s) * cin_real + ci]) : (bf16_t)0;
  w[i] = v;
  if (stride == 1) {
    wT[(((int64_t)ci * k + (k - 1 - r)) * k + (k - 1 - s)) * Cout + co] = v;
  } else {
    // the class whose first tap has the parity of r (resp. s)
    const int ph = (r + pad) & 1, pw = (s + pad) & 1;      // (ph+pad)%2 == r%2  <=>  ph == (r+pad)%2
    int64_t base = 0;
    for (int q = 0; q < 2 * ph + pw; ++q)
      base += (int64_t)parity_class(q >> 1, k, pad).nr * parity_class(q & 1, k, pad).nr;
    const ParityClass ch = parity_class(ph, k, pad), cw = parity_class(pw, k, pad);
    const int ii = (r - ch.rf) / 2, jj = (s - cw.rf) / 2;
    wT[base * Cin * Cout + (((int64_t)ci * ch.nr + (ch.nr - 1 - ii)) * cw.nr + (cw.nr - 1 - jj)) * Cout + co] = v;
  }
}

// ---- 7x7 stride-2 pad-3 stem as a 4x4 stride-1 convolution over 2x2 pixel blocks -----------------
// With 3 input channels the stem wastes most of a 32-row MFMA tile in backward-data and needs a per-vector
// tap decode in forward.  Storing the network input as 2x2 pixel blocks of 4 channels (3 used; 8 bytes per
// pixel, 32 per block),
//   x2[n][i][j][(ph*2+pw)*4 + c] = x[n][2i+ph][2j+pw][c]      (H, W even),
// turns it into a dense layer with 16 input channels:
//   forward:       y[ho][wo][co]  = sum_{a,b<4} sum_v  x2[ho-2+a][wo-2+b][v] * Vf[co][a][b][v]
//                  Vf[co][a][b][(ph,pw,c)] = W[co][2a+ph-1][2b+pw-1][c]
//   backward-data: dx2[i][j][v]   = sum_{a,b<4} sum_co dy[i-1+a][j-1+b][co] * Vb[v][a][b][co]
//                  Vb[(ph,pw,c)][a][b][co] = W[co][5+ph-2a][5+pw-2b][c]
// (filter taps outside 0..6 and channel 3 are zero: 49 of the 64 window/parity pairs are used), one launch
// each, all four pixel parities of the input gradient at once.  The four blocks of a window row are
// contiguous in memory, so the forward pass reads them as ONE tap of 64 channels (IgemmArgs::xstride = 16):
// a 4 x 1 filter over 64-channel pixels that overlap their neighbours.
constexpr int kStemV = 16;     // values per 2x2 block: 4 positions x 4 channels
__global__ void stem_weight_transform_kernel(const float* __restrict__ master, bf16_t* __restrict__ vf, bf16_t* __restrict__ vb,
                                             int Cout, int cin_real) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Cout * 16 * kStemV) return;
  {   // vf[co][a][b][v]
    const int v = i & 15, b = (i >> 4) & 3, a = (i >> 6) & 3, co = i >> 8;
    const int ph = v >> 3, pw = (v >> 2) & 1, c = v & 3;
    const int r = 2 * a + ph - 1, s = 2 * b + pw - 1;
    const bool ok = c < cin_real && r >= 0 && r < 7 && s >= 0 && s < 7;
    vf[i] = ok ? f2bf(master[((co * 7 + r) * 7 + s) * cin_real + c]) : (bf16_t)0;
  }
  {   // vb[v][a][b][co]
    const int co = i % Cout; int t = i / Cout;
    const int b = t & 3, a = (t >> 2) & 3, v = t >> 4;
    const int ph = v >> 3, pw = (v >> 2) & 1, c = v & 3;
    const int r = 5 + ph - 2 * a, s = 5 + pw - 2 * b;
    const bool ok = c < cin_real && r >= 0 && r < 7 && s >= 0 && s < 7;
    vb[i] = ok ? f2bf(master[((co * 7 + r) * 7 + s) * cin_real + c]) : (bf16_t)0;
  }
}

// dW[co][r][s][c] = dVf[co][a][b][(ph,pw,c)] with r = 2a+ph-1, s = 2b+pw-1
__global__ void stem_wgrad_gather_kernel(const float* __restrict__ dv, float* __restrict__ dw, int Cout, int cin_real, uint32_t* __restrict__ absmax) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t m = 0;
  if (i < Cout * 49 * cin_real) {
    const int c = i % cin_real; int t = i / cin_real;
    const int s = t % 7; t /= 7;
    const int r = t % 7; const int co = t / 7;
    const int ph = (r + 1) & 1, a = (r + 1) >> 1, pw = (s + 1) & 1, b = (s + 1) >> 1;
    const float v = dv[((co * 4 + a) * 4 + b) * kStemV + (ph * 2 + pw) * 4 + c];
    dw[i] = v;
    m = abs_bits(v);
  }
  if (absmax) {   // (all 64 lanes of every wavefront reach this point)
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
    if ((threadIdx.x & 63) == 0) absmax_publish(absmax_way(absmax, blockIdx.x), m);
  }
}

// ---- backward-weight ----------------------------------------------------------------------------
struct WgradArgs {
  const bf16_t* x;      // [B][H][W][Cin]
  const bf16_t* dy;     // [M][Cout], M = B*Ho*Wo
  float* ws;            // [splits][Cout][Ktot]
  int B, H, W, Cin, Ho, Wo, Cout, k, stride, pad;
  int M, Ktot, pix_per_split;
  int splits, gx, gy;    // gx x gy output tiles, each summed over `splits` pixel ranges
  int chunk;             // pixels per chain of fp32 MFMA sums (a multiple of the 64-pixel tile)
};

// ---- backward-weight through the LDS transpose reads of gfx950 -----------------------------------------------
// The contraction runs over pixels, but both operands are stored with channels contiguous.  Instead of transposing
// 8x8 blocks in registers, this kernel lands the tiles in LDS as they are in memory --
// dY [64 pixels][TC channels] and the shifted X [64 pixels][TJ columns], by the direct-to-LDS loads of the forward
// kernel -- and reads MFMA fragments with ds_read_b64_tr_b16: inside every group of 16 lanes, lane i receives
// element i%4 of the 8-byte chunks named by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12 (checked on the device).  With
// source lane j pointing at pixel pb + j/4, channels cb + 4*(j%4) .. +3, lane i ends up with four consecutive pixels
// of channel cb + i: two such reads are the eight k values of a 32x32x16 operand.
// LDS rows are 32-byte-segment swizzled by pixel so that the 4 pixels x 2 segments a half-wave touches cover all
// banks; the swizzle is applied on the source side of the direct loads (16-byte chunks keep their pair).
typedef short v4s16 __attribute__((ext_vector_type(4)));
union FragTr { v4s16 h[2]; bf16x8 v; };

template <int ROWB> __device__ __forceinline__ int tr_seg_flip(int pixel) {
  return ROWB == 256 ? 2 * (pixel & 3) : 2 * ((pixel >> 1) & 1);     // 256-byte rows: 8 segments; 128-byte rows: 4
}

//
// Two workgroups per CU, one round of them: the pixel range is split only as far as that takes, because every split
// costs a partial tile written and read again (64 KB; with four times the splits that traffic was a third to a half of
// the whole).  The chain of fp32 sums stays as short as with many splits: every `chunk` pixels the accumulators are
// added to a second set and start from zero -- the registers for it are there at two workgroups per CU.  All tiles of
// a pixel range run on one XCD (its L2 then holds both operands), every XCD an eighth of the work.
// Measured, kernel + reduction, us (2048 workgroups, flat loads -> this): 3x3, 391 images 128 -> 128 at 16x16
// 101 -> 44, 256 -> 256 at 8x8 74 -> 44; 256 images 64 -> 64 at 56x56 176 -> 92, 256 -> 256 at 14x14 110 -> 72 (830 TFLOP/s);
// 1x1 1024 -> 256 at 14x14 84 -> 43; 640 -> 640 at 8x8, 128 images 179 -> 78.  Error against 64 bits no larger (1.4e-7 / 1.6e-7).
template <int TC, int TJ>
__global__ __launch_bounds__(kThreads, 2) void wgrad_kernel(WgradArgs a) {
  constexpr int BP = 64;                           // pixels per LDS tile
  constexpr int RA = TC * 2, RBJ = TJ * 2;         // bytes per pixel row of the two tiles
  constexpr int CA = RA / 16, CJ = RBJ / 16;       // 16-byte chunks per row
  constexpr int NA = TC / 32, NB = TJ / 32;        // direct loads per thread and tile (1 KB per wave instruction)
  constexpr int WC = TC / 2, WJ = TJ / 2;
  constexpr int NI = WC / 32, NJ = WJ / 32;
  static_assert((RA == 128 || RA == 256) && RBJ == 256, "row swizzles are written for 128- and 256-byte rows");
  constexpr int STAGE = BP * (RA + RBJ);
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * STAGE];

  const int tiles = a.gx * a.gy, work = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  const int split = work / tiles, tile = work - split * tiles;
  if (split >= a.splits) return;
  const int c0 = (tile % a.gx) * TC, j0 = (tile / a.gx) * TJ;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave & 1, wj = wave >> 1;
  const int p_begin = split * a.pix_per_split;
  const int p_end = min(a.M, p_begin + a.pix_per_split);
  const int HW = a.Ho * a.Wo;

  // ---- what this thread's direct loads fetch: wave instruction q = i*4 + wave fills 1 KB = 64/CA (64/CJ) pixel rows.  The
  // swizzle depends on the low bits of the pixel only, so a thread's channel chunk -- for X its filter tap -- is the
  // same in all of its loads.  dY rows past the split lie beyond the descriptor's range; an X vector advances by
  // additions (64 pixels further = step_n images, step_q rows and step_r columns) and carries kOob where it lies outside the image.
  const BufRsrc abuf = buffer_of(a.dy + (int64_t)p_begin * a.Cout, (int64_t)(p_end - p_begin) * a.Cout);
  const BufRsrc bbuf = buffer_of(a.x, (int64_t)a.B * a.H * a.W * a.Cin);
  const int a_pr = wave * (64 / CA) + lane / CA, a_pc = lane % CA;
  const int a_lc = ((((a_pc >> 1) ^ tr_seg_flip<RA>(a_pr)) << 1) | (a_pc & 1));     // logical chunk behind physical chunk a_pc
  const bool a_ok = c0 + a_lc * 8 < a.Cout;
  uint32_t a_off = (uint32_t)(a_pr * a.Cout + c0 + a_lc * 8) * 2u;
  const uint32_t a_load_step = (uint32_t)(4 * (64 / CA)) * a.Cout * 2u, a_tile_step = (uint32_t)BP * a.Cout * 2u;
  const int b_pr = wave * (64 / CJ) + lane / CJ, b_pc = lane % CJ;
  const int b_lc = ((((b_pc >> 1) ^ tr_seg_flip<RBJ>(b_pr)) << 1) | (b_pc & 1));
  const int j = j0 + b_lc * 8;
  const bool b_ok = j < a.Ktot;
  const int tap = (b_ok ? j : 0) / a.Cin, b_ci = (b_ok ? j : 0) - tap * a.Cin, tap_r = tap / a.k;
  const int b_r = tap_r - a.pad, b_s = tap - tap_r * a.k - a.pad;
  const int sh = a.stride - 1;                                    // strides 1 and 2
  const int step_n = BP / HW, step_q = (BP - step_n * HW) / a.Wo, step_r = BP - step_n * HW - step_q * a.Wo;
  const uint32_t px = (uint32_t)a.Cin * 2u, d_col = (uint32_t)a.stride * px, d_row = (uint32_t)a.stride * a.W * px;
  const uint32_t image = (uint32_t)a.H * a.W * px, d_tile = step_n * image + step_q * d_row + step_r * d_col;
  const uint32_t d_wrap = d_row - a.Wo * d_col, d_image = image - a.Ho * d_row;
  int b_ho[NB], b_wo[NB]; uint32_t b_off[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int p = p_begin + b_pr + i * 4 * (64 / CJ);
    const int n = p / HW, rem = p - n * HW;
    b_ho[i] = rem / a.Wo; b_wo[i] = rem - b_ho[i] * a.Wo;
    b_off[i] = ((uint32_t)(n * a.H + b_ho[i] * a.stride + b_r) * a.W + b_wo[i] * a.stride + b_s) * px + b_ci * 2;
  }
  auto fetch = [&](int p0, unsigned char* stage) {
    unsigned char* const wave_a = stage + wave * 1024;
    unsigned char* const wave_b = wave_a + BP * RA;
#pragma unroll
    for (int i = 0; i < NA; ++i) load_to_lds(abuf, wave_a + i * 4096, a_ok ? a_off + i * a_load_step : kOob, 0);
    a_off += a_tile_step;
    const int left = b_ok ? p_end - p0 - b_pr : 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const uint32_t hi = (uint32_t)((b_ho[i] << sh) + b_r), wi = (uint32_t)((b_wo[i] << sh) + b_s);
      const bool ok = (i * 4 * (64 / CJ) < left) & (hi < (uint32_t)a.H) & (wi < (uint32_t)a.W);
      load_to_lds(bbuf, wave_b + i * 4096, ok ? b_off[i] : kOob, 0);
    }
    // the same lane's pixels in the next tile: at most one row wrap and one image wrap.  (Images smaller than a tile: a loop
    // over them cost up to four rounds per load, 1x1 256 -> 512 / 2 into 4x4, 512 images 21.8 us, without 20.1.)
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const bool wrap = b_wo[i] + step_r >= a.Wo;
      b_wo[i] += wrap ? step_r - a.Wo : step_r; b_ho[i] += wrap ? step_q + 1 : step_q; b_off[i] += wrap ? d_tile + d_wrap : d_tile;
      const bool next = b_ho[i] >= a.Ho;
      b_ho[i] -= next ? a.Ho : 0; b_off[i] += next ? d_image : 0u;
    }
  };
  // ---- fragment addresses: lane = 16 g + j names pixel 8 (g/2) + j/4 (+ 4 for the second read, + 16 per k-step) and
  // the 8-byte chunk of channels 16 (g%2) + 4 (j%4) of its 32-channel block
  const int g = lane >> 4, jl = lane & 15;
  const int fpix = 8 * (g >> 1) + (jl >> 2);
  int fa_off[NI], fb_off[NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int byte = (wc * WC + i * 32 + 16 * (g & 1) + 4 * (jl & 3)) * 2;
    fa_off[i] = fpix * RA + ((((byte >> 5) ^ tr_seg_flip<RA>(fpix)) << 5) | (byte & 31));
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int byte = (wj * WJ + j * 32 + 16 * (g & 1) + 4 * (jl & 3)) * 2;
    fb_off[j] = BP * RA + fpix * RBJ + ((((byte >> 5) ^ tr_seg_flip<RBJ>(fpix)) << 5) | (byte & 31));
  }

  f32x16 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  f32x16 sum[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) sum[i][j] = acc[i][j];
  int chunk_end = p_begin + a.chunk;

  fetch(p_begin, lds);
  int stage = 0;
  for (int p0 = p_begin; p0 < p_end; p0 += BP) {
    // this tile has landed, and behind the barrier every wave is done with the other stage
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    // all fragments of the tile first, then the next tile's loads (the compiler lets no transpose read pass a direct load
    // in flight), which land under the MFMAs
    const unsigned char* cur = lds + stage * STAGE;
    FragTr fa[BP / 16][NI], fb[BP / 16][NJ];
#pragma unroll
    for (int kk = 0; kk < BP / 16; ++kk) {
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          fa[kk][i].h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s16*)(cur + fa_off[i] + (kk * 16 + 4 * h) * RA));
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          fb[kk][j].h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s16*)(cur + fb_off[j] + (kk * 16 + 4 * h) * RBJ));
    }
    __builtin_amdgcn_sched_barrier(0);
    if (p0 + BP < p_end) fetch(p0 + BP, lds + (stage ^ 1) * STAGE);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < BP / 16; ++kk)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk][i].v, fb[kk][j].v, acc[i][j], 0, 0, 0);
    stage ^= 1;
    if (p0 + BP >= chunk_end || p0 + BP >= p_end) {
      chunk_end += a.chunk;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) { sum[i][j][e] += acc[i][j][e]; acc[i][j][e] = 0.f; }
    }
  }
  // ---- partial tile -> workspace[split][co][j]   (lane: column j = l%32, rows co = 8g+4h+e)
  float* dst = a.ws + (int64_t)split * a.Cout * a.Ktot;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int col = j0 + wj * WJ + j * 32 + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int co = c0 + wc * WC + i * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (co < a.Cout && col < a.Ktot) dst[(int64_t)co * a.Ktot + col] = sum[i][j][e];
      }
    }
}

// Sums the `splits` partial tiles in a fixed order: a workgroup owns 32 consecutive elements (one cache line per
// split); thread group g = tid / 32 adds splits g, g+8, ... (eight loads in flight), then the eight group sums
// are added in order.
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const float* __restrict__ ws, int splits, int64_t per_split, int Cin, int cin_real,
                                                           float scale, float* __restrict__ dw, uint32_t* __restrict__ absmax) {
  __shared__ float sh[8][32];
  const int lane = threadIdx.x & 31, grp = threadIdx.x >> 5;
  uint32_t* const slot = absmax ? absmax_way(absmax, blockIdx.x) : nullptr;
  const uint32_t seen = (slot && threadIdx.x == 0) ? absmax_peek(slot) : 0u;   // in flight with the loads below
  const int64_t i = (int64_t)blockIdx.x * 32 + lane;
  const int64_t ic = i < per_split ? i : per_split - 1;
  float s = 0.f;
  for (int k0 = grp; k0 < splits; k0 += 64) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + 8 * u;
      v[u] = ws[(int64_t)(k < splits ? k : splits - 1) * per_split + ic];
      if (k >= splits) v[u] = 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  sh[grp][lane] = s;
  __syncthreads();
  if (grp != 0) return;
  // (the 32 lanes of group 0 stay together to the end: their maximum is combined by lane exchanges)
  const int ci = (int)(ic % Cin);
  const bool live = i < per_split && ci < cin_real;
  s = 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g) s += sh[g][lane];
  const float v = s * scale;
  if (live) dw[(i / Cin) * cin_real + ci] = v;
  if (absmax) {
    uint32_t m = live ? abs_bits(v) : 0u;
#pragma unroll
    for (int d = 16; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
    if (lane == 0) absmax_raise(slot, seen, m);
  }
}

// The same for few splits: a thread owns four consecutive elements (one 16-byte load per split) and adds the splits
// s, s+4, ... into four sums.  Above kFewSplits the loads of one thread are too long a chain.
constexpr int kFewSplits = 16;
__global__ __launch_bounds__(256) void wgrad_reduce_few_kernel(const float* __restrict__ ws, int splits, int64_t per_split, int Cin, int cin_real,
                                                               float scale, float* __restrict__ dw, uint32_t* __restrict__ absmax) {
  uint32_t* const slot = absmax ? absmax_way(absmax, blockIdx.x) : nullptr;
  const uint32_t seen = (slot && (threadIdx.x & 63) == 0) ? absmax_peek(slot) : 0u;   // in flight with the loads below
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;                    // (per_split is a multiple of 8)
  uint32_t m = 0;
  if (i < per_split) {
    float4 s[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k0 = 0; k0 < splits; k0 += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k0 + u < splits) {
          const float4 v = *reinterpret_cast<const float4*>(ws + (int64_t)(k0 + u) * per_split + i);
          s[u].x += v.x; s[u].y += v.y; s[u].z += v.z; s[u].w += v.w;
        }
    }
    const float r[4] = {((s[0].x + s[1].x) + (s[2].x + s[3].x)) * scale, ((s[0].y + s[1].y) + (s[2].y + s[3].y)) * scale,
                        ((s[0].z + s[1].z) + (s[2].z + s[3].z)) * scale, ((s[0].w + s[1].w) + (s[2].w + s[3].w)) * scale};
    const int64_t row = i / Cin; const int ci = (int)(i - row * Cin);                 // (Cin is a multiple of 8: one row)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (ci + u < cin_real) { dw[row * cin_real + ci + u] = r[u]; m = max(m, abs_bits(r[u])); }
  }
  if (absmax) {   // (all 64 lanes of every wavefront reach this point)
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d));
    if ((threadIdx.x & 63) == 0) absmax_raise(slot, seen, m);
  }
}

struct WgradPlan { int splits, max_splits, pix_per_split, gx, gy, chunk; bool narrow; };   // max_splits: before rounding, grows with the batch

WgradPlan plan_wgrad(const ConvGeom& g) {
  WgradPlan p;
  const int M = g.B * g.Ho * g.Wo, Ktot = g.k * g.k * g.Cin;
  p.narrow = g.Cout <= 64;
  const int TC = p.narrow ? 64 : 128;
  p.gx = (g.Cout + TC - 1) / TC;
  p.gy = (Ktot + 127) / 128;
  const int tiles = p.gx * p.gy;
  const int max_by_pixels = (M + 255) / 256;
  // pixels per chain of fp32 sums: what about 2048 pieces of work would have
  int pieces = (2048 + tiles - 1) / tiles;
  if (pieces > max_by_pixels) pieces = max_by_pixels;
  if (pieces > 512) pieces = 512;
  p.chunk = ((M + pieces - 1) / pieces + 63) / 64 * 64;
  // splits: one round of workgroups, each at least five tiles long (four tiles: 18 of 558 measured shapes 4 to 19 % slower, 14x14
  // 1024 -> 256, 21 images 20.5 us, with four 24.5).  Two workgroups per CU; three of the narrow tiles of a filter window (64 -> 64
  // at 56x56, 256 images 92 us, two 95; but at 32x32, 391 images 57.9, two 57.1, and 40x40, 50 images 23.6, two 22.9; the 1x1
  // layers are bound by HBM and the partial tiles count: 95.7, three 100.7).  Where five tiles each leave less than that
  // round, some CUs hold one workgroup and some two: one for each then, longer, with fewer partial tiles (128 -> 256 / 2 into
  // 8x8, 100 images 360 workgroups 27.5 us, 252 23.4; 1x1 320 -> 640 / 2 into 8x8 24.6, 22.9; none of the 558 slower).
  const int cus = compute_units();
  int splits = (p.narrow && g.k > 1 ? 3 : 2) * cus / tiles;
  if (splits > (M + 319) / 320) {
    splits = (M + 319) / 320;
    if (splits * tiles <= 2 * cus && splits > cus / tiles && cus >= tiles) splits = cus / tiles;
  }
  if (splits < 1) splits = 1;
  const int span = (int)((int64_t)M * g.Cout >> 29) + 1;         // a split's dY stays below 2 GiB: 32-bit offsets past its end
  if (splits < span) splits = span;
  p.max_splits = splits;
  int pps = (M + splits - 1) / splits;
  pps = (pps + 63) / 64 * 64;
  p.pix_per_split = pps;
  p.splits = (M + pps - 1) / pps;
  return p;
}

}  // namespace

size_t conv_mfma_wgrad_workspace(const ConvGeom& g) {
  const WgradPlan p = plan_wgrad(g);
  return (size_t)p.max_splits * g.Cout * g.k * g.k * g.Cin * sizeof(float);
}

static void set_stats(IgemmArgs& a, const ConvStats* s, int slab0) {
  a.stat_mode = 0; a.stat_slab0 = slab0; a.stat_partial = nullptr;
  a.stat_x = nullptr; a.stat_mask = nullptr; a.stat_mean = nullptr; a.stat_rstd = nullptr;
  a.stat_x2 = nullptr; a.stat_mean2 = nullptr; a.stat_rstd2 = nullptr;
  if (!s || !s->mode) return;
  a.stat_mode = s->mode; a.stat_partial = s->partial;
  if (s->mode >= 2) { a.stat_x = s->bn_x; a.stat_mask = s->bn_mask; a.stat_mean = s->bn_mean; a.stat_rstd = s->bn_rstd; }
  if (s->mode == 3) { a.stat_x2 = s->bn_x2; a.stat_mean2 = s->bn_mean2; a.stat_rstd2 = s->bn_rstd2; }
}

int64_t conv_mfma_launch_count() { return g_launches.load(std::memory_order_relaxed); }

constexpr int kPixelTile = 128;   // smallest TP of the configurations run_igemm selects (pixel_tile gives the one of a launch)

int conv_stat_slabs(int64_t rows, int stride) {
  // stride 2 backward-data numbers its slabs by parity class: at most 3 extra partial tiles
  return (int)((rows + kPixelTile - 1) / kPixelTile) + (stride == 2 ? 4 : 0);
}

dat_status conv_mfma_forward(const bf16_t* x, const bf16_t* w, const bf16_t* res, bf16_t* y, const ConvGeom& g, ConvStats* stats, hipStream_t st) {
  IgemmArgs a;
  a.xstride = 0;
  a.xf_x = nullptr; a.xf_mask = nullptr; a.xf_tab = nullptr;
  a.in = x; a.wt = w; a.res = res; a.res_mask = nullptr; a.res_even_only = 0; a.out = y;
  a.B = g.B; a.Hin = g.H; a.Win = g.W; a.Cin = g.Cin; a.Hout = g.Ho; a.Wout = g.Wo; a.Cout = g.Cout;
  a.KH = g.k; a.KW = g.k; a.ostride = g.stride; a.pad_h = a.pad_w = g.pad;
  a.outH = g.Ho; a.outW = g.Wo; a.ostep = 1; a.oh0 = a.ow0 = 0;
  a.M = g.B * g.Ho * g.Wo; a.Ktot = g.k * g.k * g.Cin; a.nct = a.npt = 0;
  set_stats(a, stats, 0);
  const Switches sw = read_switches();
  const RingPick ring = pick_ring(a, sw);
  if (stats) stats->nslabs = (a.M + pixel_tile(ring) - 1) / pixel_tile(ring);
  return run_igemm(a, sw, ring, st);
}

bool conv_mfma_sparse_writer_ok(const ConvGeom& g) { return g.k == 1 && g.stride == 2 && g.pad == 0; }

bool conv_mfma_bn_operand_ok(const ConvGeom& g) {
  // The convolution's output channels are the contraction of its backward-data pass, its input channels the
  // rows of the result.  Every channel tile of the result transforms the operand again, so this pays only when
  // one tile covers all of them (measured: break-even at two tiles, a loss beyond) and the contraction is at
  // least two k-tiles long.
  return g.k == 1 && g.stride == 1 && g.pad == 0 && g.Cin % 8 == 0 && g.Cin > 32 && g.Cin <= 128 && g.Cout >= 2 * g.Cin &&
         g.Cout % (g.Cin <= 64 ? 64 : 32) == 0 && (size_t)g.Cout * kBnTabFloatsPerChannel * sizeof(float) <= 32768;
}

dat_status conv_mfma_backward_data(const bf16_t* dy, const bf16_t* wT, bf16_t* dx, const ConvGeom& g, bool accumulate, ConvStats* stats, hipStream_t st,
                                   const bf16_t* masked_res, const uint8_t* res_mask, const BnOperand* bn, int sparse) {
  if (accumulate && masked_res) return DAT_ERR_ARG;
  if (sparse == 1 && (!conv_mfma_sparse_writer_ok(g) || accumulate || masked_res || bn || (stats && stats->mode))) return DAT_ERR_ARG;
  if (sparse == 2 && !accumulate) return DAT_ERR_ARG;
  if (bn && !conv_mfma_bn_operand_ok(g)) return DAT_ERR_UNSUPPORTED;
  IgemmArgs a;
  a.xstride = 0;
  a.xf_x = nullptr; a.xf_mask = nullptr; a.xf_tab = nullptr;
  if (bn) { a.xf_x = bn->x; a.xf_mask = bn->mask; a.xf_tab = bn->tab; }
  a.in = dy; a.res = accumulate ? dx : masked_res; a.res_mask = masked_res ? res_mask : nullptr; a.out = dx;
  a.res_even_only = (sparse == 2 && g.stride == 1) ? 1 : 0;
  a.B = g.B; a.Hin = g.Ho; a.Win = g.Wo; a.Cin = g.Cout; a.Cout = g.Cin;
  a.ostride = 1; a.outH = g.H; a.outW = g.W; a.nct = a.npt = 0;
  if (g.stride == 1) {
    a.wt = wT; a.Hout = g.H; a.Wout = g.W; a.KH = a.KW = g.k; a.pad_h = a.pad_w = g.k - 1 - g.pad;
    a.ostep = 1; a.oh0 = a.ow0 = 0;
    a.M = g.B * g.H * g.W; a.Ktot = g.k * g.k * g.Cout;
    set_stats(a, stats, 0);
    const Switches sw = read_switches();
    const RingPick ring = pick_ring(a, sw);
    if (stats) stats->nslabs = (a.M + pixel_tile(ring) - 1) / pixel_tile(ring);
    return run_igemm(a, sw, ring, st);
  }
  if (g.stride != 2) return DAT_ERR_UNSUPPORTED;
  a.ostep = 2;
  set_stats(a, stats, 0);
  const bf16_t* const stored = a.res;
  const Switches sw = read_switches();
  IgemmClass cls[4];
  int n = 0, slab0 = 0;
  int64_t base = 0;
  for (int q = 0; q < 4; ++q) {
    const int ph = q >> 1, pw = q & 1;
    const ParityClass ch = parity_class(ph, g.k, g.pad), cw = parity_class(pw, g.k, g.pad);
    IgemmClass c;
    c.wt = wT + base * g.Cin * g.Cout;
    c.Hout = (g.H - ph + 1) / 2; c.Wout = (g.W - pw + 1) / 2;
    c.KH = ch.nr; c.KW = cw.nr; c.pad_h = ch.pad; c.pad_w = cw.pad;
    c.oh0 = ph; c.ow0 = pw;
    c.M = g.B * c.Hout * c.Wout; c.Ktot = ch.nr * cw.nr * g.Cout;
    c.with_res = !(sparse == 2 && q != 0);            // the stored gradient exists at even rows and columns only
    c.stat_slab0 = slab0; c.npt = c.begin = 0;
    const bool taps = c.Ktot != 0;
    if (!taps) c.KH = c.KW = 1;         // class without taps: only writes zeros (or keeps the stored gradient)
    if (sparse == 1 && !taps) continue;               // left unwritten: the accumulating pass that follows skips them
    if (c.M > 0) cls[n++] = c;
    slab0 += (c.M + kPixelTile - 1) / kPixelTile;
    base += (int64_t)ch.nr * cw.nr;
  }
  auto take = [&](const IgemmClass& c) {
    a.wt = c.wt; a.Hout = c.Hout; a.Wout = c.Wout; a.KH = c.KH; a.KW = c.KW; a.pad_h = c.pad_h; a.pad_w = c.pad_w;
    a.oh0 = c.oh0; a.ow0 = c.ow0; a.M = c.M; a.Ktot = c.Ktot; a.stat_slab0 = c.stat_slab0;
    a.res = c.with_res ? stored : nullptr;
  };
  if (n > 1) {
    // one launch: at 13 images of 32x32 four launches of a few workgroups each take about 8 us apiece, and in the larger
    // layers every class had a last wave of its own (attacks, ms, four launches -> one: pre-activation ResNet-18, 13 images
    // 9.23 -> 8.51; CIFAR ResNet-18, 512 images 28.01 -> 27.55; WRN-34-10, 256 images 95.1 -> 94.6; ResNet-50, 85 images
    // 28.34 -> 28.08)
    IgemmClasses cl{};
    cl.n = n;
    for (int i = 0; i < n; ++i) cl.c[i] = cls[i];
    for (int i = 1; i < n; ++i)          // most taps first
      for (int j = i; j > 0 && cl.c[j].Ktot > cl.c[j - 1].Ktot; --j) { const IgemmClass t = cl.c[j]; cl.c[j] = cl.c[j - 1]; cl.c[j - 1] = t; }
    take(cl.c[0]);
    a.res = stored;
    bool done;
    const dat_status s = run_igemm_classes(a, sw, cl, st, &done);
    if (done) { if (stats) stats->nslabs = slab0; return s; }
  }
  for (int i = 0; i < n; ++i) {
    take(cls[i]);
    const dat_status s = run_igemm(a, sw, pick_ring(a, sw), st);
    if (s != DAT_OK) return s;
  }
  if (stats) stats->nslabs = slab0;
  return DAT_OK;
}

// ---- stem on 2x2 pixel blocks ---------------------------------------------------------------------
bool conv_mfma_stem_blocked_ok(const ConvGeom& g, int cin_real) {
  return g.k == 7 && g.stride == 2 && g.pad == 3 && g.Cin == 8 && cin_real <= 4 && g.H % 2 == 0 && g.W % 2 == 0 && g.Cout % 8 == 0 && g.Cout <= 64;
}

ConvGeom conv_mfma_stem_blocked_geom(const ConvGeom& g) {
  ConvGeom q = g;
  q.H = g.H / 2; q.W = g.W / 2; q.Cin = kStemV; q.k = 4; q.stride = 1; q.pad = 2;   // Ho, Wo, Cout unchanged
  return q;
}

dat_status launch_stem_weight_transform(const float* master, bf16_t* vf, bf16_t* vb, int Cout, int cin_real, hipStream_t st) {
  const int n = Cout * 16 * kStemV;
  hipLaunchKernelGGL(stem_weight_transform_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, master, vf, vb, Cout, cin_real);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

dat_status conv_mfma_stem_forward(const bf16_t* x2, const bf16_t* vf, bf16_t* y, const ConvGeom& g, ConvStats* stats, hipStream_t st) {
  IgemmArgs a;
  a.xstride = 0;
  a.xf_x = nullptr; a.xf_mask = nullptr; a.xf_tab = nullptr;
  a.in = x2; a.wt = vf; a.res = nullptr; a.res_mask = nullptr; a.res_even_only = 0; a.out = y;
  // a window row of four blocks is one contiguous 64-value vector: 4 x 1 taps of 64 "channels", pixels kStemV apart
  a.B = g.B; a.Hin = g.H / 2; a.Win = g.W / 2; a.Cin = 4 * kStemV; a.xstride = kStemV; a.Hout = g.Ho; a.Wout = g.Wo; a.Cout = g.Cout;
  a.KH = 4; a.KW = 1; a.ostride = 1; a.pad_h = a.pad_w = 2;
  a.outH = g.Ho; a.outW = g.Wo; a.ostep = 1; a.oh0 = a.ow0 = 0;
  a.M = g.B * g.Ho * g.Wo; a.Ktot = 16 * kStemV; a.nct = a.npt = 0;
  set_stats(a, stats, 0);
  if (stats) stats->nslabs = (a.M + kPixelTile - 1) / kPixelTile;
  return run_igemm(a, read_switches(), kRNone, st);      // (run_igemm takes a row read as one tap first)
}

dat_status conv_mfma_stem_backward_data(const bf16_t* dy, const bf16_t* vb, bf16_t* dx2, const ConvGeom& g, bool accumulate, hipStream_t st) {
  IgemmArgs a;
  a.xstride = 0;
  a.xf_x = nullptr; a.xf_mask = nullptr; a.xf_tab = nullptr;
  a.in = dy; a.wt = vb; a.res = accumulate ? dx2 : nullptr; a.res_mask = nullptr; a.res_even_only = 0; a.out = dx2;
  a.B = g.B; a.Hin = g.Ho; a.Win = g.Wo; a.Cin = g.Cout; a.Hout = g.H / 2; a.Wout = g.W / 2; a.Cout = kStemV;
  a.KH = a.KW = 4; a.ostride = 1; a.pad_h = a.pad_w = 1;
  a.outH = a.Hout; a.outW = a.Wout; a.ostep = 1; a.oh0 = a.ow0 = 0;
  a.M = g.B * a.Hout * a.Wout; a.Ktot = 16 * g.Cout; a.nct = a.npt = 0;
  set_stats(a, nullptr, 0);
  const Switches sw = read_switches();
  return run_igemm(a, sw, pick_ring(a, sw), st);
}

dat_status conv_mfma_backward_weight(const bf16_t* x, const bf16_t* dy, float* dw, int cin_real, const ConvGeom& g, float scale,
                                     void* ws, hipStream_t st, uint32_t* absmax) {
  if (g.Cin % 8 != 0 || g.Cout % 8 != 0) return DAT_ERR_UNSUPPORTED;
  const WgradPlan p = plan_wgrad(g);
  WgradArgs a;
  a.x = x; a.dy = dy; a.ws = (float*)ws;
  a.B = g.B; a.H = g.H; a.W = g.W; a.Cin = g.Cin; a.Ho = g.Ho; a.Wo = g.Wo; a.Cout = g.Cout;
  a.k = g.k; a.stride = g.stride; a.pad = g.pad;
  a.M = g.B * g.Ho * g.Wo; a.Ktot = g.k * g.k * g.Cin; a.pix_per_split = p.pix_per_split;
  a.splits = p.splits; a.gx = p.gx; a.gy = p.gy; a.chunk = p.chunk;
  const int64_t work = (int64_t)p.gx * p.gy * p.splits;
  if (work + 7 >= (1ll << 31)) return DAT_ERR_UNSUPPORTED;
  const dim3 grid((unsigned)((work + 7) / 8 * 8));
  if (p.narrow) hipLaunchKernelGGL((wgrad_kernel<64, 128>), grid, dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL((wgrad_kernel<128, 128>), grid, dim3(kThreads), 0, st, a);
  DAT_LAUNCH_CHECK();
  const int64_t per_split = (int64_t)g.Cout * a.Ktot;
  if (p.splits <= kFewSplits)
    hipLaunchKernelGGL(wgrad_reduce_few_kernel, dim3((unsigned)((per_split + 1023) / 1024)), dim3(256), 0, st, (const float*)ws, p.splits,
                       per_split, g.Cin, cin_real, scale, dw, absmax);
  else
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)((per_split + 31) / 32)), dim3(256), 0, st, (const float*)ws, p.splits,
                       per_split, g.Cin, cin_real, scale, dw, absmax);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

dat_status launch_weight_transform(const float* master, bf16_t* w, bf16_t* wT, int Cout, int k, int cin_real, int Cin, int stride,
                                   int pad, hipStream_t st) {
  const int64_t n = (int64_t)Cout * k * k * Cin;
  hipLaunchKernelGGL(weight_transform_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, master, w, wT, Cout, k, cin_real, Cin, stride, pad);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

// dw [Cout][7][7][cin_real] through the blocked layer's gradient dv [Cout][4][4][16] (scratch, fp32).
dat_status conv_mfma_stem_backward_weight(const bf16_t* x2, const bf16_t* dy, float* dw, float* dv, int cin_real, const ConvGeom& g,
                                          float scale, void* ws, hipStream_t st, uint32_t* absmax) {
  const ConvGeom q = conv_mfma_stem_blocked_geom(g);
  const dat_status s = conv_mfma_backward_weight(x2, dy, dv, kStemV, q, scale, ws, st);
  if (s != DAT_OK) return s;
  const int n = g.Cout * 49 * cin_real;
  hipLaunchKernelGGL(stem_wgrad_gather_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const float*)dv, dw, g.Cout, cin_real, absmax);
  DAT_LAUNCH_CHECK();
  return DAT_OK;
}

}  // namespace dat

// ---- C entry points for per-shape tests and timing -----------------------------------------------
using namespace dat;

extern "C" dat_status dat_set_kernel_option(dat_kernel_option opt, int value) {
  switch (opt) {
    case DAT_KOPT_RING_KERNEL: g_ring_enabled.store(value != 0, std::memory_order_relaxed); return DAT_OK;
    case DAT_KOPT_TILE_160: g_tile160.store(value != 0, std::memory_order_relaxed); return DAT_OK;
    case DAT_KOPT_NARROW_UNDERFILLED: g_narrow_underfilled.store(value != 0, std::memory_order_relaxed); return DAT_OK;
  }
  return DAT_ERR_ARG;
}

static bool geom_from(int B, int H, int W, int Cin, int Cout, int k, int stride, int pad, ConvGeom* g) {
  if (B < 1 || H < 1 || W < 1 || Cin < 8 || Cout < 8 || Cin % 8 || Cout % 8 || k < 1 || pad < 0 || pad >= k) return false;
  if (stride != 1 && stride != 2) return false;
  g->B = B; g->H = H; g->W = W; g->Cin = Cin; g->Cout = Cout; g->k = k; g->stride = stride; g->pad = pad;
  g->Ho = (H + 2 * pad - k) / stride + 1; g->Wo = (W + 2 * pad - k) / stride + 1;
  if (g->Ho < 1 || g->Wo < 1) return false;
  if ((int64_t)B * H * W * Cin >= (1ll << 31) || (int64_t)B * g->Ho * g->Wo * Cout >= (1ll << 31)) return false;
  return true;
}

extern "C" dat_status dat_conv_plan(int pass, int stats, int B, int H, int W, int Cin, int Cout, int k, int stride, int pad, int32_t* info) {
  ConvGeom g;
  if (!info || pass < 0 || pass > 1 || stats < 0 || stats > 3 || (pass == 0 && stats > 1) || !geom_from(B, H, W, Cin, Cout, k, stride, pad, &g)) return DAT_ERR_ARG;
  ConvStats cs{};
  cs.mode = stats;
  LaunchRecord r{};
  t_record = &r;
  const dat_status s = pass == 0 ? conv_mfma_forward(nullptr, nullptr, nullptr, nullptr, g, &cs, nullptr)
                                 : conv_mfma_backward_data(nullptr, nullptr, nullptr, g, false, &cs, nullptr);
  t_record = nullptr;
  if (s != DAT_OK) return s;
  const int32_t v[10] = {r.launches, r.kernel, r.tile_c, r.tile_p, r.stages, r.k_tile, r.straddle, r.classes, (int32_t)r.slabs, cs.nslabs};
  for (int i = 0; i < 10; ++i) info[i] = v[i];
  return DAT_OK;
}

extern "C" dat_status dat_conv_forward(const uint16_t* x, const uint16_t* w, uint16_t* y, int B, int H, int W, int Cin,
                                       int Cout, int k, int stride, int pad, void* stream) {
  ConvGeom g;
  if (!x || !w || !y || !geom_from(B, H, W, Cin, Cout, k, stride, pad, &g)) return DAT_ERR_ARG;
  if (!aligned(x, 16) || !aligned(w, 16) || !aligned(y, 16)) return DAT_ERR_ARG;
  return conv_mfma_forward(x, w, nullptr, y, g, nullptr, (hipStream_t)stream);
}

extern "C" dat_status dat_conv_backward_data(const uint16_t* dy, const uint16_t* w, uint16_t* dx, int B, int H, int W,
                                             int Cin, int Cout, int k, int stride, int pad, void* stream) {
  ConvGeom g;
  if (!dy || !w || !dx || !geom_from(B, H, W, Cin, Cout, k, stride, pad, &g)) return DAT_ERR_ARG;
  if (!aligned(dy, 16) || !aligned(w, 16) || !aligned(dx, 16)) return DAT_ERR_ARG;
  // build the flipped transpose of w on the fly (test/timing path; the model caches it)
  hipStream_t st = (hipStream_t)stream;
  const size_t n = (size_t)Cout * k * k * Cin;
  float* wf = nullptr; bf16_t* w2 = nullptr; bf16_t* wT = nullptr;
  if (hipMalloc((void**)&wf, n * 4) != hipSuccess || hipMalloc((void**)&w2, n * 2) != hipSuccess ||
      hipMalloc((void**)&wT, n * 2) != hipSuccess) {
    (void)hipGetLastError();
    if (wf) (void)hipFree(wf);
    if (w2) (void)hipFree(w2);
    return DAT_ERR_NOMEM;
  }
  dat_status s = DAT_OK;
  hipLaunchKernelGGL(widen_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, wf, (int64_t)n);
  if (hipGetLastError() != hipSuccess) s = DAT_ERR_HIP;
  if (s == DAT_OK) s = launch_weight_transform(wf, w2, wT, Cout, k, Cin, Cin, stride, pad, st);
  if (s == DAT_OK) s = conv_mfma_backward_data(dy, wT, dx, g, false, nullptr, st);
  (void)hipStreamSynchronize(st);
  (void)hipFree(wf); (void)hipFree(w2); (void)hipFree(wT);
  return s;
}

extern "C" dat_status dat_conv_backward_weight(const uint16_t* x, const uint16_t* dy, float* dw, int B, int H, int W,
                                               int Cin, int Cout, int k, int stride, int pad, void* stream) {
  ConvGeom g;
  if (!x || !dy || !dw || !geom_from(B, H, W, Cin, Cout, k, stride, pad, &g)) return DAT_ERR_ARG;
  if (!aligned(x, 16) || !aligned(dy, 16) || !aligned(dw, 16)) return DAT_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  void* ws = nullptr;
  if (hipMalloc(&ws, conv_mfma_wgrad_workspace(g)) != hipSuccess) { (void)hipGetLastError(); return DAT_ERR_NOMEM; }
  dat_status s = conv_mfma_backward_weight(x, dy, dw, Cin, g, 1.0f, ws, st);
  (void)hipStreamSynchronize(st);
  (void)hipFree(ws);
  return s;
}

// ---- backward-weight without any allocation ------------------------------------------------------
// The split partial tiles of wgrad_kernel go to a buffer that is part of the library's device image instead
// of a workspace allocated per call: for callers that may not allocate (stream capture, serving loops).
// Each GPU holds its own copy of the array at its own address; in host code the array's name is only a handle
// for hipGetSymbolAddress, so the address is looked up once per device and that pointer is what the kernels get.
#define DAT_STATIC_SCRATCH_BYTES (32u << 20)
static __device__ __align__(256) unsigned char scratch[DAT_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on the first call per device).
dat_status static_scratch(void** out) {
  int dev = -1;
  DAT_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail_with(DAT_ERR_UNSUPPORTED, "device ordinal beyond the static scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    DAT_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail_with(DAT_ERR_HIP, "hipGetSymbolAddress returned a null address for the static scratch");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return DAT_OK;
}
}  // namespace

extern "C" size_t dat_conv_backward_weight_static_limit(void) { return (size_t)DAT_STATIC_SCRATCH_BYTES; }

extern "C" dat_status dat_conv_backward_weight_static(const uint16_t* x, const uint16_t* dy, float* dw, int B, int H, int W,
                                                      int Cin, int Cout, int k, int stride, int pad, void* stream) {
  ConvGeom g;
  if (!x || !dy || !dw || !geom_from(B, H, W, Cin, Cout, k, stride, pad, &g)) return DAT_ERR_ARG;
  if (!aligned(x, 16) || !aligned(dy, 16) || !aligned(dw, 16)) return DAT_ERR_ARG;
  // (the limit counts one partial sum per chain, as if each were stored: the shapes this entry point takes do not depend on how
  // many chains a workgroup adds up before it stores, nor on the number of compute units)
  const WgradPlan p = plan_wgrad(g);
  const size_t tile_bytes = (size_t)Cout * k * k * Cin * sizeof(float), chains = ((size_t)B * g.Ho * g.Wo + p.chunk - 1) / p.chunk;
  if (chains * tile_bytes > (size_t)DAT_STATIC_SCRATCH_BYTES || conv_mfma_wgrad_workspace(g) > (size_t)DAT_STATIC_SCRATCH_BYTES)
    return fail_with(DAT_ERR_UNSUPPORTED, "dat_conv_backward_weight_static: one partial sum for each chain of this shape exceeds the 32 MiB static "
                                          "scratch (use dat_conv_backward_weight)");
  void* ws = nullptr;
  const dat_status s = static_scratch(&ws);
  if (s != DAT_OK) return s;
  // every partial tile the reduction reads is written by this call's first launch: nothing to clear
  return conv_mfma_backward_weight(x, dy, dw, Cin, g, 1.0f, ws, (hipStream_t)stream);
}
