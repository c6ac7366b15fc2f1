// Observation encoder on the GPU: a ResNet-18-topology image network with
// GroupNorm and global average pooling (the pretrained policy's encoder,
// which the method leaves unchanged, Sec. 3.1 and Sec. 3.4).
//
// Activations are NHWC fp32 in HBM.  With bf16 operands, GroupNorm groups of
// 16 channels, widths that are multiples of 64 and every map after the stem's
// pooling 2 to 24 or so pixels wide (an arrangement of kFused for each layer,
// see plan_fused; frames from about 33x33 to 100x100 with four stages), every
// layer after the stem is one kernel that keeps whole images on a workgroup
// (conv_gn_kernel).  With at most 4 image channels, frames at least 12 pixels
// wide and a stem of a multiple of 64 channels that fits LDS, so are the stem
// and its pooling (stem_kernel).  512 frames of 84x84: 20 kernels, 750 us with
// other inputs for each call; the general path 41 kernels, 1490 us.
//
// The general path (fp32, all other shapes; see also plan_layer) is the rest
// of this comment.  Convolutions are implicit GEMMs on
// MFMA: M = output pixels, N = output channels, K = kh * kw * Cin in
// (kh, kw, Cin) order, which is the packed weight layout [Cout][Kp] (K
// padded to the K step).  The A tile is gathered from the input with the
// convolution's padding on the fly (no im2col buffer), converted to the
// operand type and double-buffered in LDS with the next step's global loads
// in flight during the current step's MFMAs, in 64 x 64 output tiles.  The
// gather keeps its K position (kernel tap and channel) from step to step
// instead of dividing, and every lane loads: positions outside the input
// (padding, rows beyond the output, K beyond the kernel) read a small block
// of zero bytes, so no branch surrounds the loads.
// Layers with few output tiles (small batches, late stages) split K over
// workgroups into partial outputs that the GroupNorm statistics pass sums
// in a fixed order.
//
// GroupNorm statistics are shifted sums (x - x0, x0 the group's first
// element), fp32 per thread and fp64 across threads.  Where there are many
// (image, channel chunk) workgroups or the map is small, one kernel per
// GroupNorm takes an image's groups whole (statistics, then apply);
// otherwise two passes: partial statistics over pixel chunks, then apply.
// The apply adds the residual and ReLU and, where the network pools next,
// does the pooling itself: 3x3/2 max pooling after the stem, global average
// pooling after the last block (the last block's output is never stored).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "evo_host.hpp"
#include "evo_kernels.hpp"

using namespace evo;

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kTargetWG = 512;      // split K below this many output tiles
constexpr int kMaxSplit = 16;
constexpr long long kWsFloats = 1024ll * 4096;  // split-K partials (>= splits * tiles * 64 * 64)
// GroupNorm workgroups aimed at when chunking an image's pixels (statistics
// and apply passes).  The K splits of the convolutions and the pixel chunks
// of the GroupNorm statistics are planned for the encoder's max_batch, not
// for the batch of a call: every call then sums an image's products and
// statistics in the same groupings, so an image's features do not depend on
// the batch size or on the other images.  A smaller batch runs the same
// per-image plan on fewer workgroups (an encoder meant for small batches is
// created with a small max_batch).  The apply pass is elementwise, so its
// chunking follows the call's batch.  (Fixed chunks of 64 or 128 pixels
// measured 3-8% slower.)
constexpr int kGnTarget = 1024;
// One GroupNorm kernel instead of two for maps of at most kFusedPixels
// pixels, and for maps of at most kFusedPixelsWide pixels where the
// max_batch plan has at least kFusedWG (image, channel chunk) workgroups;
// with fewer workgroups than kFusedWG it takes one group per workgroup.
// (Measured on 84x84 frames: 2 frames 0.290 -> 0.279 ms; one kernel for
// every map at 2 frames 0.50 ms; at 512 frames the stem's 1764-pixel maps
// took 165 us in one kernel against 126 us in two, the 441-pixel maps 10%
// less in one.)
constexpr int kFusedWG = 256;
constexpr int kFusedPixels = 128;
constexpr int kFusedPixelsWide = 1024;

template <class AT> struct ConvStep;
template <> struct ConvStep<__bf16> {
  static constexpr int KS = 64;  // K per stage: two 16x16x32 MFMAs per tile
};
template <> struct ConvStep<float> {
  static constexpr int KS = 32;  // K per stage: eight 16x16x4 MFMAs per tile
};

struct ConvArgs {
  const float* x;    // [N][H][W][Cin]
  const void* w;     // [Cout][Kp] operand type
  float* y;          // [N][Ho][Wo][Cout], or split z at y + z * split_stride
  const float* zeros;  // 64 zero bytes (16-byte aligned): the source of loads outside the input
  int H, W, Cin, Ho, Wo, Cout, kw, stride, pad, K, Kp;
  int M, mt, nt, splits, spp;  // pixels, tile counts, K splits, K steps per split
  long long split_stride;
};

// Maps a workgroup to a logical tile so that the workgroups of one XCD
// (blockIdx % 8) take a contiguous range of logical ids: neighbouring tiles
// that share input pixels or weights then meet in the same L2.
__device__ __forceinline__ int xcd_linear(int b, int total) {
  const int per = total >> 3, rem = total & 7, xcd = b & 7, slot = b >> 3;
  return xcd < rem ? xcd * (per + 1) + slot : rem * (per + 1) + (xcd - rem) * per + slot;
}

// Block tile BM x BN, 4 waves as 2 x 2, wave tile (BM/2) x (BN/2) of 16x16
// MFMA tiles.  Thread t stages chunk t % 4 (SEG = KS / 4 consecutive K) of
// rows t / 4 + p * 64 of the A (pixels) and B (output channels) tiles.
template <class AT, int BM, int BN>
__global__ void __launch_bounds__(kThreads) conv_kernel(const ConvArgs a) {
  constexpr int KS = ConvStep<AT>::KS, LDK = KS + 8, SEG = KS / 4, CPR = 4, RPP = kThreads / CPR;
  constexpr int PA = BM / RPP, PB = BN / RPP, MI = BM / 32, NJ = BN / 32;
  constexpr int BV = SEG * (int)sizeof(AT) / 16;  // 16-byte loads per B chunk
  static_assert(BM % RPP == 0 && BN % RPP == 0, "tile rows must be a multiple of the staging rows");
  __shared__ __attribute__((aligned(16))) AT As[2][BM * LDK];
  __shared__ __attribute__((aligned(16))) AT Bs[2][BN * LDK];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, wm = wv >> 1, wn = wv & 1;
  const int lr = lane & 15, lq = lane >> 4;

  const int id = xcd_linear(blockIdx.x, a.mt * a.nt * a.splits);
  const int nti = id % a.nt, rest = id / a.nt, mti = rest % a.mt, z = rest / a.mt;
  const int m0 = mti * BM, n0 = nti * BN;
  const int steps = a.Kp / KS;
  const int s_begin = z * a.spp, s_end = min(steps, s_begin + a.spp);

  const int chunk = tid % CPR, row0 = tid / CPR;
  // the A rows this thread stages: output pixel -> image base and window origin
  // (rlo, rhi: the part of a kernel row of kw * Cin contiguous K elements
  // that falls inside the image horizontally)
  // (wo0: element offset of the window origin within the image, negative
  // where the window starts in the padding; an image has fewer than 2^31
  // elements, checked at creation)
  const float* xb[PA];
  int ih0[PA], iw0[PA], wo0[PA], rlo[PA], rhi[PA];
  bool pv[PA];
#pragma unroll
  for (int p = 0; p < PA; ++p) {
    const int pm = m0 + row0 + p * RPP;
    pv[p] = pm < a.M;
    const int hw = a.Ho * a.Wo;
    const int pn = pv[p] ? pm / hw : 0;
    const int r = pv[p] ? pm - pn * hw : 0;
    const int oh = r / a.Wo, ow = r - oh * a.Wo;
    xb[p] = a.x + (size_t)pn * a.H * a.W * a.Cin;
    ih0[p] = oh * a.stride - a.pad;
    iw0[p] = ow * a.stride - a.pad;
    wo0[p] = (ih0[p] * a.W + iw0[p]) * a.Cin;
    rlo[p] = max(0, -iw0[p]) * a.Cin;
    rhi[p] = min(a.kw, a.W - iw0[p]) * a.Cin;
  }
  // weight rows beyond Cout read the zero bytes (their B step is SEG
  // operands, at most 64 bytes)
  const AT* wb[PB];
  bool bv[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    const int c = n0 + row0 + p * RPP;
    bv[p] = c < a.Cout;
    wb[p] = reinterpret_cast<const AT*>(a.w) + (size_t)(bv[p] ? c : 0) * a.Kp + chunk * SEG;
  }
  const bool vec = (a.Cin % SEG) == 0;  // a chunk then lies inside one input pixel

  // one K step of staged operands
  struct Regs {
    float a[PA][SEG];
    uint4 b[PB][BV];
  };

  // the K position of this thread's chunk, advanced by KS per step (loads
  // are requested for consecutive steps): vec: tap (ka, kb) and channel c;
  // otherwise kernel row ka0 and offset r0 within it
  int kc = 0, kka = 0, kkb = 0;
  const int rowlen = a.kw * a.Cin;
  {
    const int kk0 = s_begin * KS + chunk * SEG;
    if (vec) {
      const int pix = kk0 / a.Cin;
      kc = kk0 - pix * a.Cin;
      kka = pix / a.kw;
      kkb = pix - kka * a.kw;
    } else {
      kka = kk0 / rowlen;
      kc = kk0 - kka * rowlen;
    }
  }
  const auto advance = [&]() {
    kc += KS;
    if (vec) {
      while (kc >= a.Cin) {
        kc -= a.Cin;
        if (++kkb == a.kw) {
          kkb = 0;
          ++kka;
        }
      }
    } else {
      while (kc >= rowlen) {
        kc -= rowlen;
        ++kka;
      }
    }
  };
  auto load = [&](Regs& rg, int s) {
    const int kk = s * KS + chunk * SEG;
    if (vec) {
      // every lane loads: from the input inside the image, from the zero
      // bytes outside it (no branch around the loads; the tests are combined
      // with & so that they compile to compares and selects)
      const int ka = kka, kb = kkb, toff = (ka * a.W + kb) * a.Cin + kc;
#pragma unroll
      for (int p = 0; p < PA; ++p) {
        const int ih = ih0[p] + ka, iw = iw0[p] + kb;
        const bool in = pv[p] & (kk < a.K) & (ih >= 0) & (ih < a.H) & (iw >= 0) & (iw < a.W);
        const f32x4* src = reinterpret_cast<const f32x4*>(in ? xb[p] + (wo0[p] + toff) : a.zeros);
#pragma unroll
        for (int q = 0; q < SEG / 4; ++q) {
          const f32x4 t = src[q];
          rg.a[p][4 * q] = t[0];
          rg.a[p][4 * q + 1] = t[1];
          rg.a[p][4 * q + 2] = t[2];
          rg.a[p][4 * q + 3] = t[3];
        }
      }
    } else {
      // walk the chunk along kernel rows: K element (ka, r) sits at input
      // row ih0 + ka, offset iw0 * Cin + r of that row
      const int ka0 = kka, r0 = kc;
#pragma unroll
      for (int p = 0; p < PA; ++p) {
        int ka = ka0, r = r0;
#pragma unroll
        for (int q = 0; q < SEG; ++q) {
          const int ih = ih0[p] + ka;
          const bool in = pv[p] & (kk + q < a.K) & (ih >= 0) & (ih < a.H) & (r >= rlo[p]) & (r < rhi[p]);
          rg.a[p][q] = *(in ? xb[p] + ((ih * a.W + iw0[p]) * a.Cin + r) : a.zeros);
          if (++r == rowlen) {
            r = 0;
            ++ka;
          }
        }
      }
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const uint4* src = bv[p] ? reinterpret_cast<const uint4*>(wb[p] + (size_t)s * KS)
                               : reinterpret_cast<const uint4*>(a.zeros);
#pragma unroll
      for (int q = 0; q < BV; ++q) rg.b[p][q] = src[q];
    }
    advance();
  };
  auto store = [&](const Regs& rg, int buf) {
#pragma unroll
    for (int p = 0; p < PA; ++p) {
      AT* dst = As[buf] + (row0 + p * RPP) * LDK + chunk * SEG;
      if constexpr (sizeof(AT) == 2) {
#pragma unroll
        for (int h = 0; h < SEG / 8; ++h) {
          bf16x8_t t;
#pragma unroll
          for (int q = 0; q < 8; ++q) t[q] = (__bf16)rg.a[p][8 * h + q];
          *reinterpret_cast<bf16x8_t*>(dst + 8 * h) = t;
        }
      } else {
#pragma unroll
        for (int h = 0; h < SEG / 4; ++h)
          *reinterpret_cast<f32x4*>(dst + 4 * h) =
              f32x4{rg.a[p][4 * h], rg.a[p][4 * h + 1], rg.a[p][4 * h + 2], rg.a[p][4 * h + 3]};
      }
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      uint4* dst = reinterpret_cast<uint4*>(Bs[buf] + (row0 + p * RPP) * LDK + chunk * SEG);
#pragma unroll
      for (int q = 0; q < BV; ++q) dst[q] = rg.b[p][q];
    }
  };

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](int buf) {
    const AT* A = As[buf] + (wm * (BM / 2) + lr) * LDK;
    const AT* B = Bs[buf] + (wn * (BN / 2) + lr) * LDK;
    if constexpr (sizeof(AT) == 2) {
#pragma unroll
      for (int kk = 0; kk < KS / 32; ++kk) {
        bf16x8_t af[MI], bf[NJ];
#pragma unroll
        for (int i = 0; i < MI; ++i) af[i] = *reinterpret_cast<const bf16x8_t*>(A + i * 16 * LDK + kk * 32 + lq * 8);
#pragma unroll
        for (int j = 0; j < NJ; ++j) bf[j] = *reinterpret_cast<const bf16x8_t*>(B + j * 16 * LDK + kk * 32 + lq * 8);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bf[j], acc[i][j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int k4 = 0; k4 < KS / 4; ++k4) {
        float af[MI], bf[NJ];
#pragma unroll
        for (int i = 0; i < MI; ++i) af[i] = A[i * 16 * LDK + k4 * 4 + lq];
#pragma unroll
        for (int j = 0; j < NJ; ++j) bf[j] = B[j * 16 * LDK + k4 * 4 + lq];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bf[j], acc[i][j], 0, 0, 0);
      }
    }
  };

  // Step i computes from LDS buffer i % 2 while the loads of step i + 1 are
  // in flight; they go to the other buffer, which step i - 1 read before the
  // barrier that ended it.  (A second register set for two steps of slack
  // costs occupancy and measured slower.)
  const int n = s_end - s_begin;
  Regs r;
  if (n > 0) {
    load(r, s_begin);
    store(r, 0);
  }
  __syncthreads();
  for (int i = 0; i < n; ++i) {
    const bool more = i + 1 < n;
    if (more) load(r, s_begin + i + 1);
    compute(i & 1);
    if (more) store(r, (i & 1) ^ 1);
    __syncthreads();
  }
  // D: lane holds rows 4 * (lane / 16) + r of column lane % 16 of each tile
  float* y = a.y + (long long)z * a.split_stride;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int col = n0 + wn * (BN / 2) + j * 16 + lr;
      if (col >= a.Cout) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = m0 + wm * (BM / 2) + i * 16 + lq * 4 + r;
        if (row < a.M) y[(size_t)row * a.Cout + col] = acc[i][j][r];
      }
    }
}

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2 round4(f32x4 v) {  // four bf16, round to nearest even
  const bf16x2_t lo = {(__bf16)v[0], (__bf16)v[1]}, hi = {(__bf16)v[2], (__bf16)v[3]};
  return u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
}

enum { GN_PLAIN = 0, GN_MAXPOOL = 1, GN_AVGPOOL = 2 };

struct GnArgs {
  const float* ws;   // split-K partials (splits > 1): x = sum over z of ws[z * split_stride + i]
  int splits;
  long long split_stride;
  float* x;          // conv output [N][HW][C] (written by the statistics pass when splits > 1)
  const float* gamma;
  const float* beta;
  const float* res;  // residual [N][HW][C] or NULL
  float* y;          // PLAIN: [N][HW][C] (may be x); MAXPOOL: [N][Hp][Wp][C]; AVGPOOL: out + n * out_stride
  __bf16* yb;        // MAXPOOL: a rounded copy of y, or NULL
  double2* part;     // [N][groups][ps_stats] shifted (sum, sum of squares)
  float* shift;      // [N][groups] the shift x0 (read before the apply pass may overwrite x in place)
  int relu, mode, H, W, C, G, gpw, ps_stats, ps_apply, Hp, Wp, out_stride;
  float eps;
};

// Statistics pass: workgroup (image n, channel chunk of gpw groups, pixel
// chunk); thread t reads float4 column t % Q of pixel rows t / Q + i * RP.
// Sums are of (x - x0), x0 the group's first element, so that a mean far
// from zero does not cancel the variance.
__global__ void __launch_bounds__(kThreads) gn_stats_kernel(const GnArgs a) {
  const int HW = a.H * a.W, CW = a.G * a.gpw, Q = CW >> 2, RP = kThreads / Q;
  const int chunks = a.C / CW, groups = a.C / a.G;
  const int pi = blockIdx.x % a.ps_stats, rest = blockIdx.x / a.ps_stats;
  const int ch = rest % chunks, n = rest / chunks;
  const int tid = threadIdx.x, col = tid % Q, prow = tid / Q;
  const int c = ch * CW + col * 4, j = (col * 4) / a.G;
  const size_t base = (size_t)n * HW * a.C;
  const int pc = (HW + a.ps_stats - 1) / a.ps_stats, p0 = pi * pc, p1 = min(HW, p0 + pc);
  const bool split = a.splits > 1;

  float x0;
  {
    const size_t i0 = base + ch * CW + j * a.G;
    if (!split) {
      x0 = a.x[i0];
    } else {  // all partials requested before the first is added (same order of additions)
      float t[kMaxSplit];
#pragma unroll
      for (int z = 0; z < kMaxSplit; ++z) t[z] = z < a.splits ? a.ws[(long long)z * a.split_stride + i0] : 0.f;
      x0 = t[0];
#pragma unroll
      for (int z = 1; z < kMaxSplit; ++z)
        if (z < a.splits) x0 += t[z];
    }
  }
  float s = 0.f, q = 0.f;
  for (int p = p0 + prow; p < p1; p += RP) {
    const size_t i = base + (size_t)p * a.C + c;
    f32x4 v;
    if (!split) {
      v = *reinterpret_cast<const f32x4*>(a.x + i);
    } else {
      f32x4 t[kMaxSplit];
#pragma unroll
      for (int z = 0; z < kMaxSplit; ++z)
        t[z] = z < a.splits ? *reinterpret_cast<const f32x4*>(a.ws + (long long)z * a.split_stride + i)
                            : f32x4{0.f, 0.f, 0.f, 0.f};
      v = t[0];
#pragma unroll
      for (int z = 1; z < kMaxSplit; ++z)
        if (z < a.splits) v += t[z];
      *reinterpret_cast<f32x4*>(a.x + i) = v;
    }
    const f32x4 d = v - x0;
    s += (d[0] + d[1]) + (d[2] + d[3]);
    q += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
  }
  __shared__ double sd[kThreads], qd[kThreads];
  sd[tid] = s;
  qd[tid] = q;
  __syncthreads();
  for (int h = RP >> 1; h > 0; h >>= 1) {
    if (prow < h) {
      sd[tid] += sd[tid + h * Q];
      qd[tid] += qd[tid + h * Q];
    }
    __syncthreads();
  }
  if (tid < a.gpw) {
    const int cols = a.G >> 2;
    double S = 0.0, Qs = 0.0;
    for (int k = 0; k < cols; ++k) {
      S += sd[tid * cols + k];
      Qs += qd[tid * cols + k];
    }
    a.part[((size_t)n * groups + ch * a.gpw + tid) * a.ps_stats + pi] = make_double2(S, Qs);
  }
  if (pi == 0 && col * 4 % a.G == 0 && prow == 0) a.shift[(size_t)n * groups + ch * a.gpw + j] = x0;
}

// Apply pass: mean and 1/sqrt(var + eps) from the partials, then
// f(v) = [relu]((v - mean) rstd gamma + beta [+ res]) per mode.
__global__ void __launch_bounds__(kThreads) gn_apply_kernel(const GnArgs a) {
  const int HW = a.H * a.W, CW = a.G * a.gpw, Q = CW >> 2, RP = kThreads / Q;
  const int chunks = a.C / CW, groups = a.C / a.G;
  const int pi = blockIdx.x % a.ps_apply, rest = blockIdx.x / a.ps_apply;
  const int ch = rest % chunks, n = rest / chunks;
  const int tid = threadIdx.x, col = tid % Q, prow = tid / Q;
  const int c = ch * CW + col * 4, j = (col * 4) / a.G;
  const size_t base = (size_t)n * HW * a.C;
  // merge the partials of each of the gpw groups (a fixed order per chunk
  // count): one thread per group when there are few, else L = kThreads / gpw
  // threads per group, thread l summing partials l, l + L, ..., then a tree
  // over l
  __shared__ float2 st[16];
  __shared__ double2 mrg[kThreads];
  const auto finish = [&](int jg, double S, double Qs) {
    const int g = ch * a.gpw + jg;
    const double cnt = (double)HW * a.G, m = S / cnt;
    const double var = std::max(Qs / cnt - m * m, 0.0);
    const float x0 = a.shift[(size_t)n * groups + g];
    st[jg] = make_float2((float)((double)x0 + m), (float)(1.0 / std::sqrt(var + (double)a.eps)));
  };
  if (a.ps_stats <= 8) {
    if (tid < a.gpw) {
      const double2* pp = a.part + ((size_t)n * groups + ch * a.gpw + tid) * a.ps_stats;
      double S = 0.0, Qs = 0.0;
      for (int k = 0; k < a.ps_stats; ++k) {
        S += pp[k].x;
        Qs += pp[k].y;
      }
      finish(tid, S, Qs);
    }
  } else {
    const int L = kThreads / a.gpw, jg = tid / L, l = tid - jg * L;
    const double2* pp = a.part + ((size_t)n * groups + ch * a.gpw + jg) * a.ps_stats;
    double S = 0.0, Qs = 0.0;
    for (int k = l; k < a.ps_stats; k += L) {
      S += pp[k].x;
      Qs += pp[k].y;
    }
    mrg[tid] = make_double2(S, Qs);
    __syncthreads();
    for (int h = L >> 1; h > 0; h >>= 1) {
      if (l < h) {
        mrg[tid].x += mrg[tid + h].x;
        mrg[tid].y += mrg[tid + h].y;
      }
      __syncthreads();
    }
    if (l == 0) finish(jg, mrg[tid].x, mrg[tid].y);
  }
  __syncthreads();
  const float2 ms = st[j];
  const f32x4 gm = *reinterpret_cast<const f32x4*>(a.gamma + c);
  const f32x4 bt = *reinterpret_cast<const f32x4*>(a.beta + c);
  auto f = [&](f32x4 v, size_t i) -> f32x4 {
    f32x4 r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = (v[k] - ms.x) * ms.y * gm[k] + bt[k];
    if (a.res) r += *reinterpret_cast<const f32x4*>(a.res + i);
    if (a.relu) {
#pragma unroll
      for (int k = 0; k < 4; ++k) r[k] = fmaxf(r[k], 0.f);
    }
    return r;
  };
  if (a.mode == GN_PLAIN) {
    const int pc = (HW + a.ps_apply - 1) / a.ps_apply, p0 = pi * pc, p1 = min(HW, p0 + pc);
    for (int p = p0 + prow; p < p1; p += RP) {
      const size_t i = base + (size_t)p * a.C + c;
      *reinterpret_cast<f32x4*>(a.y + i) = f(*reinterpret_cast<const f32x4*>(a.x + i), i);
    }
  } else if (a.mode == GN_MAXPOOL) {
    const int HWp = a.Hp * a.Wp, pc = (HWp + a.ps_apply - 1) / a.ps_apply, p0 = pi * pc, p1 = min(HWp, p0 + pc);
    for (int p = p0 + prow; p < p1; p += RP) {
      const int oh = p / a.Wp, ow = p - oh * a.Wp;
      f32x4 m = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      for (int u = 0; u < 3; ++u) {
        const int ih = oh * 2 - 1 + u;
        if (ih < 0 || ih >= a.H) continue;
        for (int v = 0; v < 3; ++v) {
          const int iw = ow * 2 - 1 + v;
          if (iw < 0 || iw >= a.W) continue;
          const size_t i = base + ((size_t)ih * a.W + iw) * a.C + c;
          const f32x4 r = f(*reinterpret_cast<const f32x4*>(a.x + i), i);
#pragma unroll
          for (int k = 0; k < 4; ++k) m[k] = fmaxf(m[k], r[k]);
        }
      }
      const size_t o = (size_t)n * HWp * a.C + (size_t)p * a.C + c;
      *reinterpret_cast<f32x4*>(a.y + o) = m;
      if (a.yb) *reinterpret_cast<u32x2*>(a.yb + o) = round4(m);
    }
  } else {
    // global average pooling (one pixel chunk): column sums over the rows
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int p = prow; p < HW; p += RP) {
      const size_t i = base + (size_t)p * a.C + c;
      acc += f(*reinterpret_cast<const f32x4*>(a.x + i), i);
    }
    __shared__ f32x4 red[kThreads];
    red[tid] = acc;
    __syncthreads();
    for (int h = RP >> 1; h > 0; h >>= 1) {
      if (prow < h) red[tid] += red[tid + h * Q];
      __syncthreads();
    }
    if (prow == 0) {
      const f32x4 m = red[tid] / (float)HW;
      float* o = a.y + (size_t)n * a.out_stride + c;
      o[0] = m[0];
      o[1] = m[1];
      o[2] = m[2];
      o[3] = m[3];
    }
  }
}

// One kernel per GroupNorm: workgroup (image n, channel chunk of gpw
// groups) computes the statistics of its groups over the whole image, then
// applies them (the apply reads what the first sweep just touched, mostly
// from L2).  Thread t reads float4 column t % Q of pixel rows t / Q + i *
// RP, as the two-pass kernels do.
__global__ void __launch_bounds__(kThreads) gn_fused_kernel(const GnArgs a) {
  const int HW = a.H * a.W, CW = a.G * a.gpw, Q = CW >> 2, RP = kThreads / Q;
  const int chunks = a.C / CW;
  const int ch = blockIdx.x % chunks, n = blockIdx.x / chunks;
  const int tid = threadIdx.x, col = tid % Q, prow = tid / Q;
  const int c = ch * CW + col * 4, j = (col * 4) / a.G;
  const size_t base = (size_t)n * HW * a.C;
  const bool split = a.splits > 1;
  __shared__ float sx0[16];
  __shared__ float2 st[16];
  __shared__ double sd[kThreads], qd[kThreads];
  // the conv output at i: the sum of the split partials in split order (all
  // requested before the first is added), or x itself
  const auto value = [&](size_t i) -> f32x4 {
    if (!split) return *reinterpret_cast<const f32x4*>(a.x + i);
    f32x4 t[kMaxSplit];
#pragma unroll
    for (int z = 0; z < kMaxSplit; ++z)
      t[z] = z < a.splits ? *reinterpret_cast<const f32x4*>(a.ws + (long long)z * a.split_stride + i)
                          : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 v = t[0];
#pragma unroll
    for (int z = 1; z < kMaxSplit; ++z)
      if (z < a.splits) v += t[z];
    return v;
  };
  // shift: the group's first element (pixel 0, first channel of the group;
  // a multiple of four channels, so the float4 load is aligned)
  const float x0 = value(base + ch * CW + j * a.G)[0];
  float s = 0.f, q = 0.f;
  const auto add = [&](f32x4 v, size_t i) {
    if (split) *reinterpret_cast<f32x4*>(a.x + i) = v;
    const f32x4 d = v - x0;
    s += (d[0] + d[1]) + (d[2] + d[3]);
    q += (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
  };
  {
    constexpr int U = 4;  // pixel rows requested together
    int p = prow;
    for (; p + (U - 1) * RP < HW; p += U * RP) {
      f32x4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = value(base + (size_t)(p + u * RP) * a.C + c);
#pragma unroll
      for (int u = 0; u < U; ++u) add(v[u], base + (size_t)(p + u * RP) * a.C + c);
    }
    for (; p < HW; p += RP) add(value(base + (size_t)p * a.C + c), base + (size_t)p * a.C + c);
  }
  sd[tid] = s;
  qd[tid] = q;
  if (prow == 0 && col * 4 % a.G == 0) sx0[j] = x0;
  __syncthreads();
  for (int h = RP >> 1; h > 0; h >>= 1) {
    if (prow < h) {
      sd[tid] += sd[tid + h * Q];
      qd[tid] += qd[tid + h * Q];
    }
    __syncthreads();
  }
  if (tid < a.gpw) {
    const int cols = a.G >> 2;
    double S = 0.0, Qs = 0.0;
    for (int k = 0; k < cols; ++k) {
      S += sd[tid * cols + k];
      Qs += qd[tid * cols + k];
    }
    const double cnt = (double)HW * a.G, m = S / cnt;
    const double var = std::max(Qs / cnt - m * m, 0.0);
    st[tid] = make_float2((float)((double)sx0[tid] + m), (float)(1.0 / std::sqrt(var + (double)a.eps)));
  }
  __syncthreads();  // also orders the split sums stored above before the reads below
  const float2 ms = st[j];
  const f32x4 gm = *reinterpret_cast<const f32x4*>(a.gamma + c);
  const f32x4 bt = *reinterpret_cast<const f32x4*>(a.beta + c);
  auto f = [&](f32x4 v, size_t i) -> f32x4 {
    f32x4 r;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = (v[k] - ms.x) * ms.y * gm[k] + bt[k];
    if (a.res) r += *reinterpret_cast<const f32x4*>(a.res + i);
    if (a.relu) {
#pragma unroll
      for (int k = 0; k < 4; ++k) r[k] = fmaxf(r[k], 0.f);
    }
    return r;
  };
  if (a.mode == GN_PLAIN) {
    for (int p = prow; p < HW; p += RP) {
      const size_t i = base + (size_t)p * a.C + c;
      *reinterpret_cast<f32x4*>(a.y + i) = f(*reinterpret_cast<const f32x4*>(a.x + i), i);
    }
  } else if (a.mode == GN_MAXPOOL) {
    const int HWp = a.Hp * a.Wp;
    for (int p = prow; p < HWp; p += RP) {
      const int oh = p / a.Wp, ow = p - oh * a.Wp;
      f32x4 m = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      for (int u = 0; u < 3; ++u) {
        const int ih = oh * 2 - 1 + u;
        if (ih < 0 || ih >= a.H) continue;
        for (int v = 0; v < 3; ++v) {
          const int iw = ow * 2 - 1 + v;
          if (iw < 0 || iw >= a.W) continue;
          const size_t i = base + ((size_t)ih * a.W + iw) * a.C + c;
          const f32x4 r = f(*reinterpret_cast<const f32x4*>(a.x + i), i);
#pragma unroll
          for (int k = 0; k < 4; ++k) m[k] = fmaxf(m[k], r[k]);
        }
      }
      const size_t o = (size_t)n * HWp * a.C + (size_t)p * a.C + c;
      *reinterpret_cast<f32x4*>(a.y + o) = m;
      if (a.yb) *reinterpret_cast<u32x2*>(a.yb + o) = round4(m);
    }
  } else {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int p = prow; p < HW; p += RP) {
      const size_t i = base + (size_t)p * a.C + c;
      acc += f(*reinterpret_cast<const f32x4*>(a.x + i), i);
    }
    __shared__ f32x4 red[kThreads];
    red[tid] = acc;
    __syncthreads();
    for (int h = RP >> 1; h > 0; h >>= 1) {
      if (prow < h) red[tid] += red[tid + h * Q];
      __syncthreads();
    }
    if (prow == 0) {
      const f32x4 m = red[tid] / (float)HW;
      float* o = a.y + (size_t)n * a.out_stride + c;
      o[0] = m[0];
      o[1] = m[1];
      o[2] = m[2];
      o[3] = m[3];
    }
  }
}

// ---------------------------------------------------------------- fused layers
// Convolution + GroupNorm + shortcut + ReLU (+ global average pooling) of
// whole images in one kernel (bf16 operands, groups of 16 channels, 3x3 or
// 1x1, channel counts multiples of 64, maps that fit a workgroup).
//
// A workgroup takes `ipw` whole images and 16 * NBW * WN output channels, so
// that every GroupNorm group it produces is complete and the conv output
// never travels through memory.  Its input pixels, 64 channels at a time,
// sit in LDS as zero-bordered images (a row of W + 1 pixels: the zero column
// ends one row and begins the next), so the nine taps of a 3x3 kernel read
// the same LDS bytes at nine offsets instead of being gathered nine times.
// The stride of a pixel is 144 bytes (128 + 16), which spreads 16 consecutive
// pixels over all LDS banks.  Weights come straight from L2 as packed MFMA
// fragments, D k-steps ahead in registers.  Products are transposed (weights
// first), so a lane holds four channels of one pixel: a 16-channel group is
// one accumulator block, and its sums are in-lane adds and two lane swaps.
//
// Waves: WM along the pixels, WN along the channels, WK along K (each its
// share of the 64-channel chunks; partial sums meet in LDS).  What bounds a
// large layer: matrix cores (16 cycles a 16x16x32 MFMA) against 1 KiB of LDS
// per pixel block and 1 KiB of L2 per channel block and k-step; a wave tile
// of 7 x 4 or 8 x 4 blocks needs about half of either.  A small batch takes
// 16 channels a workgroup, for more workgroups and a shorter weight stream.
// An image's results do not depend on its place in a tile, the other images
// or the arrangement, as long as WK is the same (and MBW and WM, where the
// statistics are summed in registers): rows of a product are independent, an
// element's products are summed in the order of K within a share, and the
// statistics in an order that the map's size or the waves' rows decide.  So a
// call of few images takes an arrangement of its own (see plan_layer) and
// gives the same bits.
constexpr int kPix = 144;  // LDS bytes of a pixel's 64 channels

struct FusedArgs {
  const __bf16* x;      // [N][H][W][Cin]
  const uint4* w;       // fragments [Cin / 64][taps][2][Cout / 16][64 lanes]
  const float* gamma;
  const float* beta;
  const float* res;     // shortcut [N][Ho][Wo][Cout] or NULL
  float* yf;            // fp32 output or NULL
  __bf16* yb;           // bf16 output (rounded) or NULL
  float* feat;          // mean over the pixels, row n at feat + n * out_stride, or NULL
  int out_stride, relu;
  int N, H, W, Ho, Wo, Cin, Cout, stride;
  int ipw, PW, PP, nit;  // images per workgroup, LDS row and image pixels, chunks per K share
  uint32_t div_px, div_pw, div_hw, div_wo, div_ipw;  // ceil(2^32 / d) of PP, PW, Ho * Wo, Wo, ipw (0: ipw is 1)
  int mt, nt, a_bytes;
  int in_regs;  // GroupNorm statistics in registers (FusedPlan::in_regs)
  int tpl;      // else log2 of the threads that sum the rows of one (group, image)
  float eps;
};

__device__ __forceinline__ int fast_div(int n, uint32_t m) { return (int)__umulhi((uint32_t)n, m); }

__device__ __forceinline__ float row16_sum(float v) {  // over the lanes that share lane / 16
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true));
  return v;
}
__device__ __forceinline__ float quad_sum(float v) {  // over the lanes that share lane % 16
  u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// sum over each 1 << lg consecutive lanes, in all of them (register moves:
// a tree through LDS shuffles cost 0.4 us a sum)
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v) {
  const u32x2 x = __builtin_bit_cast(u32x2, v);
  const u32x2 y = {(unsigned)__builtin_amdgcn_mov_dpp((int)x[0], CTRL, 0xF, 0xF, true),
                   (unsigned)__builtin_amdgcn_mov_dpp((int)x[1], CTRL, 0xF, 0xF, true)};
  return v + __builtin_bit_cast(double, y);
}
__device__ __forceinline__ double lanes_sum(double v, int lg) {
  if (lg > 0) v = add_dpp<0xB1>(v);   // neighbours
  if (lg > 1) v = add_dpp<0x4E>(v);   // pairs
  if (lg > 2) v = add_dpp<0x141>(v);  // quads
  if (lg > 3) v = add_dpp<0x140>(v);  // halves of a row of 16
  if (lg > 4) {
    const u32x2 x = __builtin_bit_cast(u32x2, v);
    const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(x[0], x[0], false, false));
    const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(x[1], x[1], false, false));
    v = __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
  }
  if (lg > 5) {
    const u32x2 x = __builtin_bit_cast(u32x2, v);
    const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(x[0], x[0], false, false));
    const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(x[1], x[1], false, false));
    v = __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
  }
  return v;
}

// (LDS: the A region, which the row sums [channel blocks][rows] of the
// statistics take over; then their mean and 1 / deviation [channel blocks]
// [ipw], or summed in registers the waves' sums, twice.)
template <int MBW, int NBW, int WM, int WN, int WK, int TAPS>
__global__ void __launch_bounds__(WM * WN * WK * 64, MBW * NBW > 32 ? 1 : 2) conv_gn_kernel(const FusedArgs a) {
  constexpr int NT = WM * WN * WK * 64, NB = NBW * WN, S = TAPS * 2;
  constexpr int D = TAPS == 1 ? 2 : NBW == 4 ? 3 : NBW == 2 ? 6 : 9;  // k-steps of weights in flight
  static_assert(S % D == 0, "ring");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lc = lane & 15, lq = lane >> 4;
  const int kg = wave / (WM * WN), wm = wave % (WM * WN) / WN, wn = wave % WN;
  const int id = xcd_linear(blockIdx.x, a.mt * a.nt), nti = id % a.nt, img0 = id / a.nt * a.ipw;
  const int HW = a.Ho * a.Wo, rows = a.ipw * HW, nbt = a.Cout / 16, nb0 = nti * NB + wn * NBW;

  // ---- weights: the wave's k-steps are consecutive in memory
  const int steps = a.nit * S, ks0 = kg * steps;
  const auto wrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(a.w), (short)0, a.Cin / 64 * S * nbt * 1024, 0x00020000);
  const auto wload = [&](int j, int n) {
    return __builtin_bit_cast(
        uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16, ((ks0 + min(j, steps - 1)) * nbt + nb0 + n) * 1024, 0));
  };
  uint4 ring[D][NBW];
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int n = 0; n < NBW; ++n) ring[d][n] = wload(d, n);

  // LDS byte of tap (0, 0), channel octet lq, of this lane's output pixels
  int abase[MBW];
#pragma unroll
  for (int m = 0; m < MBW; ++m) {
    const int r = (wm * MBW + m) * 16 + lc;
    int px = 0;
    if (r < rows) {
      const int im = fast_div(r, a.div_hw), q = r - im * HW;
      if (TAPS == 1) {
        px = r;
      } else {
        const int oy = fast_div(q, a.div_wo), ox = q - oy * a.Wo;
        px = im * a.PP + oy * a.stride * a.PW + ox * a.stride;
      }
    }
    abase[m] = (kg * a.ipw * a.PP + px) * kPix + lq * 16;
  }

  f32x4 acc[MBW][NBW];
#pragma unroll
  for (int m = 0; m < MBW; ++m)
#pragma unroll
    for (int n = 0; n < NBW; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int it = 0; it < a.nit; ++it) {
    // stage 64 channels of every K share's images (1x1: of the pixels used),
    // U 16-byte loads a thread in flight
    const int units = WK * a.ipw * a.PP * 8;
    constexpr int U = 8;
    for (int u0 = tid; u0 < units; u0 += U * NT) {
      uint4 v[U];
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int u = u0 + q * NT, oct = u & 7, slot = u >> 3, gi = fast_div(slot, a.div_px), px = slot - gi * a.PP;
        const int g = a.div_ipw ? fast_div(gi, a.div_ipw) : gi, im = gi - g * a.ipw, img = img0 + im;
        int iy, ix;
        if (TAPS == 1) {
          const int oy = fast_div(px, a.div_wo);
          iy = oy * a.stride;
          ix = (px - oy * a.Wo) * a.stride;
        } else {
          const int py = fast_div(px, a.div_pw);
          iy = py - 1;
          ix = px - py * a.PW - 1;
        }
        v[q] = make_uint4(0u, 0u, 0u, 0u);
        if (u < units && img < a.N && iy >= 0 && iy < a.H && ix >= 0)
          v[q] = *reinterpret_cast<const uint4*>(a.x + (((size_t)img * a.H + iy) * a.W + ix) * a.Cin + (g * a.nit + it) * 64 + oct * 8);
      }
#pragma unroll
      for (int q = 0; q < U; ++q) {
        const int u = u0 + q * NT;
        if (u < units) *reinterpret_cast<uint4*>(lds + (u >> 3) * kPix + (u & 7) * 16) = v[q];
      }
    }
    __syncthreads();
    uint4 af[2][MBW];
    const auto aload = [&](int s, uint4 (&f)[MBW]) {
      const int tap = s >> 1, off = (TAPS == 1 ? 0 : (tap / 3 * a.PW + tap % 3) * kPix) + (s & 1) * 64;
#pragma unroll
      for (int m = 0; m < MBW; ++m) f[m] = *reinterpret_cast<const uint4*>(lds + abase[m] + off);
    };
    aload(0, af[0]);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (s + 1 < S) aload(s + 1, af[(s + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < MBW; ++m)
#pragma unroll
        for (int n = 0; n < NBW; ++n)
          acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ring[s % D][n]),
                                                              __builtin_bit_cast(bf16x8_t, af[s & 1][m]), acc[m][n], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int n = 0; n < NBW; ++n) ring[s % D][n] = wload(it * S + s + D, n);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();  // the region is rewritten by the next chunk, or by what follows
  }

  // ---- K shares: row block m is summed, in share order, by share
  // m * WK / MBW, which also finishes it
  const auto mine = [&](int m) { return WK == 1 || m * WK / MBW == kg; };
  if constexpr (WK > 1) {
    f32x4* part = reinterpret_cast<f32x4*>(lds);
    // slot of share g's contribution to a block that another share owns
    const auto at = [&](int g, int m, int n) {
      const int x = g - (g > m * WK / MBW ? 1 : 0);
      return (((x * WM * WN + wm * WN + wn) * MBW + m) * NBW + n) * 64 + lane;
    };
#pragma unroll
    for (int m = 0; m < MBW; ++m)
      if (!mine(m)) {
#pragma unroll
        for (int n = 0; n < NBW; ++n) part[at(kg, m, n)] = acc[m][n];
      }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MBW; ++m)
      if (mine(m)) {
#pragma unroll
        for (int n = 0; n < NBW; ++n) {
          f32x4 t = kg == 0 ? acc[m][n] : part[at(0, m, n)];
#pragma unroll
          for (int g = 1; g < WK; ++g) t += g == kg ? acc[m][n] : part[at(g, m, n)];
          acc[m][n] = t;
        }
      }
    __syncthreads();
  }

  // ---- GroupNorm statistics of every image and group (mean, then the
  // squares around it).  In registers (one image a workgroup, also in the
  // max_batch arrangement): a lane's rows, the wave's lanes, then the waves in
  // order.  Else the channels of each row to LDS, 1 << tpl threads take every
  // (1 << tpl)-th row of an image, and a tree adds the threads.
  float* const smean = reinterpret_cast<float*>(lds + a.a_bytes);  // [NB][ipw]
  float* const srstd = smean + NB * a.ipw;
  const double inv_cnt = 1.0 / ((double)HW * 16.0);
  const auto row_of = [&](int m) { return (wm * MBW + m) * 16 + lc; };
  float mu[NBW], rs[NBW];  // one image; several: in LDS
  int im[MBW];
#pragma unroll
  for (int m = 0; m < MBW; ++m) im[m] = a.ipw > 1 ? fast_div(min(row_of(m), rows - 1), a.div_hw) : 0;
  if (a.in_regs) {
    float* const buf = smean;  // [2][NW][NB]
    constexpr int NW = WM * WK;
    const auto total = [&](float* buf, auto value, double (&out)[NBW]) {  // buf [NW][NB]
#pragma unroll
      for (int n = 0; n < NBW; ++n) {
        float t = 0.f;
#pragma unroll
        for (int m = 0; m < MBW; ++m)
          if (mine(m)) {
            const float v = value(m, n);
            t += row_of(m) < rows ? v : 0.f;
          }
        t = quad_sum(row16_sum(t));
        if (lane == 0) buf[(kg * WM + wm) * NB + wn * NBW + n] = t;
      }
      __syncthreads();
#pragma unroll
      for (int n = 0; n < NBW; ++n) {
        double t = 0.0;
#pragma unroll
        for (int x = 0; x < NW; ++x) t += (double)buf[x * NB + wn * NBW + n];
        out[n] = t;
      }
    };
    double t[NBW];
    total(buf, [&](int m, int n) { return (acc[m][n][0] + acc[m][n][1]) + (acc[m][n][2] + acc[m][n][3]); }, t);
#pragma unroll
    for (int n = 0; n < NBW; ++n) mu[n] = (float)(t[n] * inv_cnt);
    total(buf + NW * NB, [&](int m, int n) {
      const f32x4 d = acc[m][n] - mu[n];
      return (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
    }, t);
#pragma unroll
    for (int n = 0; n < NBW; ++n) rs[n] = (float)(1.0 / std::sqrt(t[n] * inv_cnt + (double)a.eps));
  } else {
    float* const rsum = reinterpret_cast<float*>(lds);  // [NB][rows], in the A region's place
    const int pairs = NB * a.ipw, tp = 1 << a.tpl;
    const auto total = [&](auto value, auto finish, float* st) {
#pragma unroll
      for (int m = 0; m < MBW; ++m)
        if (mine(m)) {
          float v[NBW];
#pragma unroll
          for (int n = 0; n < NBW; ++n) v[n] = quad_sum(value(m, n));
          if (lq == 0 && row_of(m) < rows) {
#pragma unroll
            for (int n = 0; n < NBW; ++n) rsum[(wn * NBW + n) * rows + row_of(m)] = v[n];
          }
        }
      __syncthreads();
      for (int p0 = 0; p0 < pairs; p0 += NT >> a.tpl) {
        const int p = p0 + (tid >> a.tpl), l = tid & (tp - 1), nb = a.div_ipw ? fast_div(p, a.div_ipw) : p;
        double sum = 0.0;
        if (p < pairs) {
          const float* src = rsum + nb * rows + (p - nb * a.ipw) * HW;
          for (int r = l; r < HW; r += 8 * tp) {  // eight reads in flight
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = src[min(r + k * tp, HW - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k) sum += r + k * tp < HW ? (double)v[k] : 0.0;
          }
        }
        sum = lanes_sum(sum, a.tpl);
        if (p < pairs && l == 0) st[p] = finish(sum);
      }
      __syncthreads();
    };
    total([&](int m, int n) { return (acc[m][n][0] + acc[m][n][1]) + (acc[m][n][2] + acc[m][n][3]); },
          [&](double t) { return (float)(t * inv_cnt); }, smean);
    total([&](int m, int n) {
      const f32x4 d = acc[m][n] - smean[(wn * NBW + n) * a.ipw + im[m]];
      return (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
    }, [&](double t) { return (float)(1.0 / std::sqrt(t * inv_cnt + (double)a.eps)); }, srstd);
  }

  // ---- normalise, add the shortcut, ReLU, store
  float* const fin = reinterpret_cast<float*>(lds);  // [rows][16 NB] (average pooling)
  {
    f32x4 gm[NBW], bt[NBW];
#pragma unroll
    for (int n = 0; n < NBW; ++n) {
      const int ch = (nb0 + n) * 16 + lq * 4;
      gm[n] = *reinterpret_cast<const f32x4*>(a.gamma + ch);
      bt[n] = *reinterpret_cast<const f32x4*>(a.beta + ch);
    }
    const auto live = [&](int m) { return row_of(m) < rows && img0 + im[m] < a.N; };
    const auto at = [&](int m) { return ((size_t)img0 * HW + row_of(m)) * a.Cout + nb0 * 16 + lq * 4; };
    // the shortcut's rows one block ahead (an output may overwrite it in place,
    // each element after its own read)
    f32x4 res[2][NBW];
    const auto rload = [&](int m, f32x4 (&v)[NBW]) {
#pragma unroll
      for (int n = 0; n < NBW; ++n) {
        v[n] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (a.res && mine(m) && live(m)) v[n] = *reinterpret_cast<const f32x4*>(a.res + at(m) + n * 16);
      }
    };
    rload(0, res[0]);
#pragma unroll
    for (int m = 0; m < MBW; ++m) {
      if (m + 1 < MBW) rload(m + 1, res[(m + 1) & 1]);
      if (!mine(m) || !live(m)) continue;
      const size_t o = at(m);
#pragma unroll
      for (int n = 0; n < NBW; ++n) {
        const int q = (wn * NBW + n) * a.ipw + im[m];
        const float mn = a.in_regs ? mu[n] : smean[q], rd = a.in_regs ? rs[n] : srstd[q];
        f32x4 v = (acc[m][n] - mn) * rd * gm[n] + bt[n];
        if (a.res) v += res[m & 1][n];
        if (a.relu) {
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
        }
        if (a.yf) *reinterpret_cast<f32x4*>(a.yf + o + n * 16) = v;
        if (a.yb) *reinterpret_cast<u32x2*>(a.yb + o + n * 16) = round4(v);
        if (a.feat) *reinterpret_cast<f32x4*>(fin + (size_t)row_of(m) * (16 * NB) + (wn * NBW + n) * 16 + lq * 4) = v;
      }
    }
  }
  if (a.feat) {
    __syncthreads();
    for (int i = tid; i < a.ipw * 16 * NB; i += NT) {
      const int g = i / (16 * NB), c = i % (16 * NB);
      if (img0 + g >= a.N) break;
      float s = 0.f;
      for (int r = 0; r < HW; ++r) s += fin[(size_t)(g * HW + r) * (16 * NB) + c];
      a.feat[(size_t)(img0 + g) * a.out_stride + nti * (16 * NB) + c] = s / (float)HW;
    }
  }
}

// weights [Cout][k][k][Cin] fp32 -> bf16 fragments of conv_gn_kernel
__global__ void pack_fused_kernel(const float* __restrict__ w, int Cout, int Cin, int taps, uint4* dst) {
  const long long total = (long long)Cin / 32 * taps * (Cout / 16) * 64;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const int lane = (int)(i % 64);
    const long long f = i / 64;
    const int nb = (int)(f % (Cout / 16)), s = (int)(f / (Cout / 16));
    const int h = s & 1, tap = (s >> 1) % taps, chunk = (s >> 1) / taps;
    const int o = nb * 16 + (lane & 15), c = chunk * 64 + h * 32 + (lane >> 4) * 8;
    bf16x8_t v;
    for (int e = 0; e < 8; ++e) v[e] = (__bf16)w[((size_t)o * taps + tap) * Cin + c + e];
    dst[i] = __builtin_bit_cast(uint4, v);
  }
}

// compiled wave arrangements (MBW, NBW, WM, WN, WK).  The last seven are taken
// only by small calls of encoders whose layer runs a wide one with the same
// rows (free to choose, more waves of fewer rows are faster: 2 frames of
// 84x84, first stage, 9.5 us a layer with (4, 1, 8, 1, 1) against 12.0 with
// (7, 1, 4, 1, 1)).
#define EVO_FUSED(X)                                                                              \
  X(7, 4, 4, 1, 1) X(9, 4, 4, 1, 1) X(4, 4, 2, 2, 1) X(8, 4, 1, 2, 2) X(9, 4, 1, 2, 2)            \
  X(5, 4, 1, 2, 2) X(5, 4, 1, 1, 4) X(4, 1, 8, 1, 1) X(5, 1, 8, 1, 1) X(2, 1, 4, 1, 2)            \
  X(3, 1, 4, 1, 2) X(2, 1, 4, 1, 1) X(3, 1, 4, 1, 1) X(3, 1, 1, 1, 4) X(3, 1, 1, 1, 2)            \
  X(1, 1, 1, 1, 8) X(1, 1, 1, 1, 4) X(3, 2, 1, 2, 4) X(3, 2, 1, 2, 2) X(5, 2, 1, 2, 2)            \
  X(7, 1, 4, 1, 1) X(9, 1, 4, 1, 1) X(4, 1, 2, 1, 1) X(8, 1, 1, 1, 2) X(9, 1, 1, 1, 2)            \
  X(5, 1, 1, 1, 2) X(5, 1, 1, 1, 4)
constexpr int kSmallCalls = 7;

struct FusedCfg {
  int mbw, nbw, wm, wn, wk;
};
constexpr FusedCfg kFused[] = {
#define X(a, b, c, d, e) {a, b, c, d, e},
    EVO_FUSED(X)
#undef X
};
constexpr size_t kLdsBytes = 160 * 1024;

// ---------------------------------------------------------------- fused stem
// 7x7 stride-2 convolution (at most 4 image channels), GroupNorm (groups of
// 16), ReLU and 3x3 stride-2 max pooling of one image's 16 * NB channels in
// one kernel: the conv output (231 MB for 512 frames of 84x84, read three
// times when it went through memory) is formed twice from the image in LDS
// instead, once for the statistics and once, four rows at a time, to be
// normalised and pooled.
//
// The image sits in LDS in bf16 with 4 channels a pixel (8 bytes) and its
// zero border, so a kernel row of 7 pixels plus one of weight zero is one
// K step of 32, and an operand fragment is an aligned 16-byte read at pixel
// 2 ow + 2 (lane / 16) of the row.  The 7 x NB weight fragments stay in
// registers.  512 frames of 84x84: three kernels 282 us, this one 107 us.
constexpr int kStemWaves = 8, kStripRows = 5;
constexpr int kStemWide = 128;  // images from which a workgroup takes all 64 channels

struct StemArgs {
  const float* x;    // [N][H][W][Cin]
  const uint4* w;    // fragments [7][C / 16][64 lanes]
  const float* gamma;
  const float* beta;
  float* yf;         // [N][Hp][Wp][C]
  __bf16* yb;        // the same rounded
  int H, W, Cin, Ho, Wo, Hp, Wp, C, PW, PR, nt;  // PW, PR: pixels a row and rows of the bordered image
  uint32_t div_pw, div_wo, div_wp;
  int strip_off, red_off;  // LDS bytes
  float eps;
};

template <int NB>
__global__ void __launch_bounds__(kStemWaves * 64) stem_kernel(const StemArgs a) {
  constexpr int NT = kStemWaves * 64, LD = 16 * NB + 4;  // strip floats a pixel (padded: no bank conflicts)
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  float* const strip = reinterpret_cast<float*>(lds + a.strip_off);      // [kStripRows][Wo][LD]
  double2* const red = reinterpret_cast<double2*>(lds + a.red_off);      // [waves][NB]
  const int tid = threadIdx.x, lane = tid & 63, lc = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int img = blockIdx.x / a.nt, nb0 = blockIdx.x % a.nt * NB, nbt = a.C / 16;

  uint4 wf[7][NB];
#pragma unroll
  for (int k = 0; k < 7; ++k)
#pragma unroll
    for (int n = 0; n < NB; ++n) wf[k][n] = a.w[(size_t)(k * nbt + nb0 + n) * 64 + lane];

  const float* src = a.x + (size_t)img * a.H * a.W * a.Cin;
  constexpr int U = 6;  // pixels in flight a thread
  for (int p0 = tid; p0 < a.PR * a.PW; p0 += U * NT) {
    f32x4 v[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int p = p0 + q * NT, py = fast_div(p, a.div_pw), iy = py - 3, ix = p - py * a.PW - 3;
      v[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (p < a.PR * a.PW && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (c < a.Cin) v[q][c] = src[(iy * a.W + ix) * a.Cin + c];
      }
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (p0 + q * NT < a.PR * a.PW) *reinterpret_cast<u32x2*>(lds + (p0 + q * NT) * 8) = round4(v[q]);
  }
  __syncthreads();

  // conv outputs of pixels px0 + lc (clamped to the last), channels 4 lq .. + 3 of each block
  const int HW = a.Ho * a.Wo;
  const auto conv = [&](int px0, f32x4 (&y)[NB]) {
    const int r = min(px0 + lc, HW - 1), oh = fast_div(r, a.div_wo), ow = r - oh * a.Wo;
    const unsigned char* at = lds + (2 * oh * a.PW + 2 * ow) * 8 + lq * 16;
    uint4 f[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) f[k] = *reinterpret_cast<const uint4*>(at + k * a.PW * 8);
#pragma unroll
    for (int n = 0; n < NB; ++n) y[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 7; ++k)
#pragma unroll
      for (int n = 0; n < NB; ++n)
        y[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[k][n]), __builtin_bit_cast(bf16x8_t, f[k]),
                                                      y[n], 0, 0, 0);
  };

  // ---- statistics: sums of (x - x0), x0 the group's first element, fp32 in
  // a lane, fp64 across the waves in order
  f32x4 y[NB];
  float x0[NB], s[NB], q[NB];
  conv(0, y);
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    x0[n] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(y[n][0])));
    s[n] = q[n] = 0.f;
  }
  for (int b = w * 16; b < HW; b += kStemWaves * 16) {
    conv(b, y);
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const f32x4 d = y[n] - x0[n];
      const float ds = (d[0] + d[1]) + (d[2] + d[3]), dq = (d[0] * d[0] + d[1] * d[1]) + (d[2] * d[2] + d[3] * d[3]);
      s[n] += b + lc < HW ? ds : 0.f;
      q[n] += b + lc < HW ? dq : 0.f;
    }
  }
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const float ts = quad_sum(row16_sum(s[n])), tq = quad_sum(row16_sum(q[n]));
    if (lane == 0) red[w * NB + n] = make_double2((double)ts, (double)tq);
  }
  __syncthreads();
  float mean[NB], rstd[NB];
  f32x4 gm[NB], bt[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    double S = 0.0, Q = 0.0;
#pragma unroll
    for (int x = 0; x < kStemWaves; ++x) {
      S += red[x * NB + n].x;
      Q += red[x * NB + n].y;
    }
    const double cnt = (double)HW * 16.0, m = S / cnt, var = std::max(Q / cnt - m * m, 0.0);
    mean[n] = (float)((double)x0[n] + m);
    rstd[n] = (float)(1.0 / std::sqrt(var + (double)a.eps));
    gm[n] = *reinterpret_cast<const f32x4*>(a.gamma + (nb0 + n) * 16 + lq * 4);
    bt[n] = *reinterpret_cast<const f32x4*>(a.beta + (nb0 + n) * 16 + lq * 4);
  }

  // ---- four conv rows at a time, kept in a ring of five: normalise, ReLU,
  // then the two pooled rows they complete (pooled row p covers conv rows
  // 2 p - 1 .. 2 p + 1)
  for (int c0 = 0; c0 < a.Ho; c0 += 4) {
    const int c1 = min(a.Ho, c0 + 4), end = c1 * a.Wo;
    for (int b = c0 * a.Wo + w * 16; b < end; b += kStemWaves * 16) {
      conv(b, y);
      const int r = b + lc, oh = fast_div(r, a.div_wo), ow = r - oh * a.Wo;
      if (r < end) {
        float* dst = strip + (oh % kStripRows * a.Wo + ow) * LD + lq * 4;
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          f32x4 v = (y[n] - mean[n]) * rstd[n] * gm[n] + bt[n];
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
          *reinterpret_cast<f32x4*>(dst + n * 16) = v;
        }
      }
    }
    __syncthreads();
    const int p0 = c0 / 2, p1 = c1 == a.Ho ? a.Hp : c1 / 2;
    for (int i = tid; i < (p1 - p0) * a.Wp * 4 * NB; i += NT) {
      const int c4 = i % (4 * NB), px = i / (4 * NB), pr = fast_div(px, a.div_wp), pw = px - pr * a.Wp, ph = p0 + pr;
      f32x4 m = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
      for (int u = -1; u <= 1; ++u)
#pragma unroll
        for (int v = -1; v <= 1; ++v) {
          const int ih = 2 * ph + u, iw = 2 * pw + v;
          if (ih < 0 || ih >= a.Ho || iw < 0 || iw >= a.Wo) continue;
          const f32x4 t = *reinterpret_cast<const f32x4*>(strip + (ih % kStripRows * a.Wo + iw) * LD + c4 * 4);
#pragma unroll
          for (int k = 0; k < 4; ++k) m[k] = fmaxf(m[k], t[k]);
        }
      const size_t o = (((size_t)img * a.Hp + ph) * a.Wp + pw) * a.C + nb0 * 16 + c4 * 4;
      *reinterpret_cast<f32x4*>(a.yf + o) = m;
      *reinterpret_cast<u32x2*>(a.yb + o) = round4(m);
    }
    __syncthreads();
  }
}

// stem weights [C][7][7][Cin] fp32 -> bf16 fragments of stem_kernel
__global__ void pack_stem_kernel(const float* __restrict__ w, int C, int Cin, uint4* dst) {
  const int total = 7 * (C / 16) * 64;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int lane = i % 64, nb = i / 64 % (C / 16), ky = i / 64 / (C / 16), o = nb * 16 + (lane & 15);
    bf16x8_t v;
    for (int e = 0; e < 8; ++e) {
      const int kx = 2 * (lane >> 4) + e / 4, c = e % 4;
      v[e] = (__bf16)(kx < 7 && c < Cin ? w[((size_t)(o * 7 + ky) * 7 + kx) * Cin + c] : 0.f);
    }
    dst[i] = __builtin_bit_cast(uint4, v);
  }
}

// weights [Cout][K] fp32 -> [Cout][Kp] operand type, zero padded
__global__ void pack_conv_kernel(const float* __restrict__ w, int Cout, int K, int Kp, int bf, void* dst) {
  const long long total = (long long)Cout * Kp;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)gridDim.x * 256) {
    const int k = (int)(i % Kp), o = (int)(i / Kp);
    const float v = k < K ? w[(size_t)o * K + k] : 0.f;
    if (bf) reinterpret_cast<__bf16*>(dst)[i] = (__bf16)v;
    else reinterpret_cast<float*>(dst)[i] = v;
  }
}

unsigned grid_for(long long total) { return (unsigned)std::min<long long>((total + 255) / 256, 16384); }

// A fused layer's launch.
struct FusedPlan {
  int cfg = -1, ipw = 0, PW = 0, PP = 0, nit = 0, a_bytes = 0, lds = 0;
  bool in_regs = false;
};
// Plans are made at creation, one for every power of two of images a call may
// have (the last one for max_batch): plan plan_class(n) serves n images.
int plan_class(int n) {
  int c = 0;
  while ((1 << c) < n) ++c;
  return c;
}

struct ConvLayer {
  int cin, cout, k, stride, pad, K, Kp;
  void* w = nullptr;             // packed operand weights
  std::vector<FusedPlan> fp;     // [plan_class(max_batch) + 1]
  const float* gamma = nullptr;  // GroupNorm affine (device, inside the raw copy)
  const float* beta = nullptr;
};

}  // namespace

struct evo_encoder {
  evo_encoder_desc desc{};
  int device = 0;
  int bf = 1;
  bool fused = false;            // the layers after the stem run as conv_gn_kernel
  int stem_nb = 0;               // 16-channel blocks a workgroup of stem_kernel takes in large calls (0: the stem runs unfused)
  float* d_raw = nullptr;        // fp32 parameter copy (GroupNorm affine, packing source)
  std::vector<ConvLayer> convs;  // stem, then per block a, b[, d]
  float* buf[4] = {nullptr, nullptr, nullptr, nullptr};
  size_t buf_floats = 0;
  float* zeros = nullptr;        // 256 zero bytes: the convolutions' loads outside their inputs
  float* ws = nullptr;           // split-K partials, kWsFloats
  double2* part = nullptr;       // GroupNorm partial statistics
  size_t part_cap = 0;
  float* shift = nullptr;        // GroupNorm shifts [image][group]
  size_t shift_cap = 0;
  uint64_t flops_per_image = 0;
  hipEvent_t ev_done = nullptr;  // recorded after the last encode's launches
  bool launched = false;
};

namespace {

int enc_check(const evo_encoder_desc* d) {
  if (!d) return fail(EVO_E_INVALID, "desc is NULL");
  if (d->height < 8 || d->width < 8 || d->height > 4096 || d->width > 4096)
    return fail(EVO_E_INVALID, "image size %d x %d outside [8, 4096]", d->height, d->width);
  if (d->in_ch < 1 || d->in_ch > 64) return fail(EVO_E_INVALID, "in_ch %d outside [1, 64]", d->in_ch);
  if (d->n_stages < 1 || d->n_stages > 4) return fail(EVO_E_INVALID, "n_stages %d outside [1, 4]", d->n_stages);
  if (d->gn_group < 1 || d->stem_ch < 1 || d->stem_ch % d->gn_group)
    return fail(EVO_E_INVALID, "stem_ch %d must be a positive multiple of gn_group %d", d->stem_ch, d->gn_group);
  if (d->stem_ch % 8) return fail(EVO_E_UNSUPPORTED, "stem_ch must be a multiple of 8");
  for (int s = 0; s < d->n_stages; ++s) {
    if (d->widths[s] < 8 || d->widths[s] % 8 || d->widths[s] % d->gn_group || d->widths[s] > 4096)
      return fail(EVO_E_INVALID, "width %d of stage %d must be a multiple of 8 and of gn_group, at most 4096",
                  d->widths[s], s);
    if (d->blocks[s] < 1 || d->blocks[s] > 16) return fail(EVO_E_INVALID, "blocks[%d] = %d", s, d->blocks[s]);
  }
  if (d->gn_group != 4 && d->gn_group != 8 && d->gn_group != 16 && d->gn_group != 32 && d->gn_group != 64)
    return fail(EVO_E_UNSUPPORTED, "gn_group must be 4, 8, 16, 32 or 64");
  if (d->dtype != EVO_FP32 && d->dtype != EVO_BF16) return fail(EVO_E_INVALID, "bad dtype");
  if (d->max_batch < 1 || d->max_batch > (1 << 16)) return fail(EVO_E_INVALID, "max_batch %d", d->max_batch);
  // pixel indices of a batch (stem output and below) are 32-bit
  if ((int64_t)d->max_batch * d->height * d->width >= (int64_t(1) << 31))
    return fail(EVO_E_UNSUPPORTED, "max_batch * height * width must stay below 2^31");
  return EVO_OK;
}

// every convolution of the network in execution order (stem; per block a, b, [d])
std::vector<ConvLayer> enc_layers(const evo_encoder_desc* d) {
  std::vector<ConvLayer> v;
  v.push_back({d->in_ch, d->stem_ch, 7, 2, 3, 0, 0});
  int cin = d->stem_ch;
  for (int s = 0; s < d->n_stages; ++s)
    for (int b = 0; b < d->blocks[s]; ++b) {
      const int c = d->widths[s], stride = (s > 0 && b == 0) ? 2 : 1;
      v.push_back({cin, c, 3, stride, 1, 0, 0});
      v.push_back({c, c, 3, 1, 1, 0, 0});
      if (stride != 1 || cin != c) v.push_back({cin, c, 1, stride, 0, 0, 0});
      cin = c;
    }
  return v;
}

inline int out_size(int h, int k, int s, int p) { return (h + 2 * p - k) / s + 1; }
inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

// Launch shape of one convolution: 64 x 64 tiles (four workgroups fit a CU;
// 128 x 128 and 128 x 64 tiles, two per CU, measured 8% slower over the
// 512-frame encode), K split where there are few tiles.
constexpr int kBM = 64, kBN = 64;
struct ConvPlan {
  int mt, nt, splits, spp;
};

ConvPlan plan_conv(int M, int Cout, int steps) {
  ConvPlan pl{};
  pl.mt = cdiv(M, kBM);
  pl.nt = cdiv(Cout, kBN);
  const int tiles = pl.mt * pl.nt;
  int splits = 1;
  if (tiles < kTargetWG) splits = std::min({cdiv(kTargetWG, tiles), std::max(1, steps / 2), kMaxSplit});
  pl.spp = cdiv(steps, splits);
  pl.splits = cdiv(steps, pl.spp);  // every split has at least one step
  return pl;
}

// Cheapest wave arrangement of a fused layer for n images of H x W, with the
// order of sums of `like` if given.  Cycles of a workgroup: matrix cores or its
// LDS reads, shared by the workgroups that run on a CU at once; plus staging
// and about 5000 for its start and statistics.  (The weight stream from L2 is
// not counted.)
bool plan_fused(int n, const ConvLayer& L, int H, int W, bool pool, int n_cu, const FusedPlan* like, FusedPlan* out) {
  const int Ho = out_size(H, L.k, L.stride, L.pad), Wo = out_size(W, L.k, L.stride, L.pad), HW = Ho * Wo;
  if ((L.k != 3 && L.k != 1) || L.cin % 64 || L.cout % 64 || Wo < 2 || HW < 2) return false;
  const int nch = L.cin / 64, S = L.k * L.k * 2;
  const int PW = L.k == 1 ? Wo : W + 1, PP = L.k == 1 ? HW : (H + 2) * PW + 1;
  double best = 0.0;
  out->cfg = -1;
  for (int c = 0; c < (int)(sizeof(kFused) / sizeof(kFused[0])) - (like ? 0 : kSmallCalls); ++c) {
    const FusedCfg& f = kFused[c];
    const int nb = f.nbw * f.wn, cap = 16 * f.mbw * f.wm, waves = f.wm * f.wn * f.wk;
    if (L.cout % (16 * nb) || nch % f.wk || cap < HW) continue;
    if (like && f.wk != kFused[like->cfg].wk) continue;
    if (like && like->in_regs && (f.mbw != kFused[like->cfg].mbw || f.wm != kFused[like->cfg].wm)) continue;
    for (int ipw = 1; ipw <= (like && like->in_regs ? 1 : std::min(cap / HW, n)); ++ipw) {
      const int rows = ipw * HW;
      const long long stage = (long long)f.wk * ipw * PP * kPix;
      const long long part = (long long)(f.wk - 1) * f.wm * f.wn * f.mbw * f.nbw * 1024;
      const bool in_regs = like ? like->in_regs : ipw == 1;
      const long long stats = in_regs ? 0 : (long long)rows * nb * 4;
      const long long a_bytes = (std::max({stage, part, pool ? (long long)rows * 16 * nb * 4 : 0ll, stats}) + 15) / 16 * 16;
      const long long lds = a_bytes + 2ll * nb * (in_regs ? f.wm * f.wk : ipw) * 4;
      if (lds > (long long)kLdsBytes) continue;
      const int nit = nch / f.wk;
      const long long wgs = (long long)cdiv(n, ipw) * (L.cout / (16 * nb));
      const long long occ = std::max(1ll, std::min((long long)kLdsBytes / lds, 8ll / waves));
      const double on = (double)std::min<long long>(occ, (wgs + n_cu - 1) / n_cu);  // workgroups that share a CU
      const double steps = (double)nit * S, one = f.mbw * f.nbw * 16.0 * steps;      // one wave's MFMAs
      const double mf = std::max(one * waves * on / 4.0, one);
      const double ld = waves * steps * f.mbw * 8.0 * on, st = stage / 32.0 * nit * on;
      const double cost = (double)((wgs + n_cu * occ - 1) / (n_cu * occ)) * (std::max(mf, ld) + st + 5000.0);
      if (out->cfg < 0 || cost < best) {
        best = cost;
        *out = FusedPlan{c, ipw, PW, PP, nit, (int)a_bytes, (int)lds, in_regs};
      }
    }
  }
  return out->cfg >= 0;
}

// The plans of a layer: the best arrangement for max_batch, which decides the
// order of every sum (see conv_gn_kernel), and for every smaller class of
// calls the best one with that order.
bool plan_layer(int max_batch, ConvLayer& L, int H, int W, bool pool, int n_cu) {
  const int last = plan_class(max_batch);
  L.fp.assign(last + 1, FusedPlan());
  // A map too large for arrangements with K shares, five or more 64-channel
  // chunks one after another and too few images to fill the device: the
  // general path's K splits are faster (96x96 frames, widths 320 and 640 or
  // 512 to 2048: 210 and 192 us against 269 and 264 for one frame, 233 and 237
  // against 271 and 268 for two; from 16 frames with widths 512 to 2048 667
  // against 599)
  const int Ho = out_size(H, L.k, L.stride, L.pad), Wo = out_size(W, L.k, L.stride, L.pad);
  if (Ho * Wo > 144 && L.cin >= 320 && L.k == 3 && max_batch < 4) return false;
  if (!plan_fused(max_batch, L, H, W, pool, n_cu, nullptr, &L.fp[last])) return false;
  for (int c = 0; c < last; ++c)
    if (!plan_fused(1 << c, L, H, W, pool, n_cu, &L.fp[last], &L.fp[c])) return false;
  return true;
}

const void* fused_kernel(int cfg, int k) {
  int i = 0;
#define X(a, b, c, d, e)                                                                            \
  if (cfg == i++)                                                                                   \
    return k == 1 ? reinterpret_cast<const void*>(&conv_gn_kernel<a, b, c, d, e, 1>)                \
                  : reinterpret_cast<const void*>(&conv_gn_kernel<a, b, c, d, e, 9>);
  EVO_FUSED(X)
#undef X
  return nullptr;
}

// One fused layer on N images of H x W (`*Ho` x `*Wo` out).
hipError_t launch_fused(const ConvLayer& L, const __bf16* x, int N, int H, int W, int* Ho, int* Wo, const float* res,
                        int relu, float* yf, __bf16* yb, float* feat, int out_stride, hipStream_t st) {
  const FusedPlan& p = L.fp[plan_class(N)];
  const FusedCfg& f = kFused[p.cfg];
  const auto magic = [](int d) { return (uint32_t)(((uint64_t(1) << 32) + d - 1) / d); };
  FusedArgs a;
  a.x = x;
  a.w = reinterpret_cast<const uint4*>(L.w);
  a.gamma = L.gamma;
  a.beta = L.beta;
  a.res = res;
  a.yf = yf;
  a.yb = yb;
  a.feat = feat;
  a.out_stride = out_stride;
  a.relu = relu;
  a.N = N;
  a.H = H;
  a.W = W;
  a.Ho = *Ho = out_size(H, L.k, L.stride, L.pad);
  a.Wo = *Wo = out_size(W, L.k, L.stride, L.pad);
  a.Cin = L.cin;
  a.Cout = L.cout;
  a.stride = L.stride;
  a.ipw = p.ipw;
  a.PW = p.PW;
  a.PP = p.PP;
  a.nit = p.nit;
  a.div_px = magic(p.PP);
  a.div_pw = magic(p.PW);
  a.div_hw = magic(a.Ho * a.Wo);
  a.div_wo = magic(a.Wo);
  a.div_ipw = p.ipw > 1 ? magic(p.ipw) : 0u;
  a.mt = cdiv(N, p.ipw);
  a.nt = L.cout / (16 * f.nbw * f.wn);
  a.a_bytes = p.a_bytes;
  a.in_regs = p.in_regs;
  a.tpl = 0;  // about eight rows a thread
  while (a.tpl < 6 && (8 << a.tpl) < a.Ho * a.Wo) ++a.tpl;
  a.eps = 1e-5f;
  void* args[] = {&a};
  return hipLaunchKernel(fused_kernel(p.cfg, L.k), dim3((unsigned)(a.mt * a.nt)), dim3(f.wm * f.wn * f.wk * 64), args,
                         (size_t)p.lds, st);
}

int stem_pitch(int W) { return (W + 8) / 2 * 2; }
int stem_lds(const evo_encoder_desc& d, int nb, int* strip_off, int* red_off) {
  const int Ho = out_size(d.height, 7, 2, 3), Wo = out_size(d.width, 7, 2, 3);
  const long long img = ((long long)(2 * (Ho - 1) + 7) * stem_pitch(d.width) * 8 + 15) / 16 * 16;
  const long long strip = (long long)kStripRows * Wo * (16 * nb + 4) * 4;
  const long long all = img + strip + kStemWaves * nb * 16;
  if (all > (long long)kLdsBytes) return 0;
  *strip_off = (int)img;
  *red_off = (int)(img + strip);
  return (int)all;
}
const void* stem_fn(int nb) {
  return nb == 4 ? reinterpret_cast<const void*>(&stem_kernel<4>) : reinterpret_cast<const void*>(&stem_kernel<1>);
}

hipError_t launch_stem(const evo_encoder* e, const ConvLayer& L, const float* images, int N, float* yf, __bf16* yb,
                       hipStream_t st) {
  const evo_encoder_desc& d = e->desc;
  const auto magic = [](int v) { return (uint32_t)(((uint64_t(1) << 32) + v - 1) / v); };
  StemArgs a;
  // all channels a workgroup where the images alone fill the device, else one
  // group (more workgroups, each with the whole image; the same bits)
  const int nb = N >= kStemWide ? e->stem_nb : 1;
  const int lds = stem_lds(d, nb, &a.strip_off, &a.red_off);
  a.x = images;
  a.w = reinterpret_cast<const uint4*>(L.w);
  a.gamma = L.gamma;
  a.beta = L.beta;
  a.yf = yf;
  a.yb = yb;
  a.H = d.height;
  a.W = d.width;
  a.Cin = d.in_ch;
  a.Ho = out_size(d.height, 7, 2, 3);
  a.Wo = out_size(d.width, 7, 2, 3);
  a.Hp = out_size(a.Ho, 3, 2, 1);
  a.Wp = out_size(a.Wo, 3, 2, 1);
  a.C = L.cout;
  a.PW = stem_pitch(d.width);
  a.PR = 2 * (a.Ho - 1) + 7;
  a.nt = L.cout / (16 * nb);
  a.div_pw = magic(a.PW);
  a.div_wo = magic(a.Wo);
  a.div_wp = magic(a.Wp);
  a.eps = 1e-5f;
  void* args[] = {&a};
  return hipLaunchKernel(stem_fn(nb), dim3((unsigned)(N * a.nt)), dim3(kStemWaves * 64), args, (size_t)lds, st);
}

// Which layers run fused, and their plans.  Every layer after the stem, or
// none (see conv_gn_kernel): bf16 operands, groups of 16 channels, and an
// arrangement for every layer.  The stem too where the image fits LDS.
// (84x84 frames, fused and general path: 2 frames 171 and 259 us, 100 frames
// 392 and 511, 512 frames 695 and 1500; on an encoder for 512 frames 2 frames
// 226 and 560 us, 64 frames 269 and 627.)
void plan_encoder(evo_encoder* e, int n_cu) {
  const evo_encoder_desc& d = e->desc;
  e->fused = e->bf && d.gn_group == 16;
  int h = out_size(out_size(d.height, 7, 2, 3), 3, 2, 1), w = out_size(out_size(d.width, 7, 2, 3), 3, 2, 1);
  size_t i = 1;
  int cin = d.stem_ch;
  for (int s = 0; s < d.n_stages && e->fused; ++s)
    for (int b = 0; b < d.blocks[s] && e->fused; ++b) {
      ConvLayer& La = e->convs[i++];
      ConvLayer& Lb = e->convs[i++];
      const int ho = out_size(h, 3, La.stride, 1), wo = out_size(w, 3, La.stride, 1);
      const bool last = s == d.n_stages - 1 && b == d.blocks[s] - 1;
      e->fused = plan_layer(d.max_batch, La, h, w, false, n_cu) && plan_layer(d.max_batch, Lb, ho, wo, last, n_cu) &&
                 ((La.stride == 1 && cin == Lb.cout) || plan_layer(d.max_batch, e->convs[i++], h, w, false, n_cu));
      h = ho;
      w = wo;
      cin = Lb.cout;
    }
  if (e->fused && d.in_ch <= 4 && d.width >= 12 && d.stem_ch % 64 == 0) {
    int so, ro;
    const int nb = d.max_batch >= kStemWide ? 4 : 1;
    if (stem_lds(d, nb, &so, &ro)) e->stem_nb = nb;
  }
}

// The conv result lands in `y` (one split) or as partials in the encoder's
// workspace; `*gn` gets the source fields of the GroupNorm that follows.
hipError_t launch_conv(const evo_encoder* e, const ConvLayer& L, const float* x, int N, int H, int W, float* y,
                       int* Ho, int* Wo, GnArgs* gn, hipStream_t st) {
  ConvArgs a;
  a.x = x;
  a.w = L.w;
  a.H = H;
  a.W = W;
  a.Cin = L.cin;
  a.Ho = *Ho = out_size(H, L.k, L.stride, L.pad);
  a.Wo = *Wo = out_size(W, L.k, L.stride, L.pad);
  a.Cout = L.cout;
  a.kw = L.k;
  a.stride = L.stride;
  a.pad = L.pad;
  a.K = L.K;
  a.Kp = L.Kp;
  a.M = N * a.Ho * a.Wo;
  const int KS = e->bf ? ConvStep<__bf16>::KS : ConvStep<float>::KS;
  // K splits of the max_batch plan; tiles for this call's pixels
  ConvPlan pl = plan_conv(e->desc.max_batch * a.Ho * a.Wo, L.cout, L.Kp / KS);
  pl.mt = cdiv(a.M, kBM);
  a.mt = pl.mt;
  a.nt = pl.nt;
  a.splits = pl.splits;
  a.spp = pl.spp;
  a.split_stride = (long long)a.M * L.cout;
  // splits * tiles * 64 * 64 bounds the partials, below the workspace by construction
  if (pl.splits > 1 && (long long)pl.splits * a.split_stride > kWsFloats) return hipErrorInvalidValue;
  a.y = pl.splits > 1 ? e->ws : y;
  a.zeros = e->zeros;
  gn->ws = e->ws;
  gn->splits = pl.splits;
  gn->split_stride = a.split_stride;
  gn->x = y;
  const unsigned grid = (unsigned)((long long)pl.mt * pl.nt * pl.splits);
  if (e->bf) hipLaunchKernelGGL((conv_kernel<__bf16, kBM, kBN>), dim3(grid), dim3(kThreads), 0, st, a);
  else hipLaunchKernelGGL((conv_kernel<float, kBM, kBN>), dim3(grid), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

// One GroupNorm pass (gn_fused_kernel) or two (statistics over pixel
// chunks, then apply).  Chosen from the encoder's max_batch and the map
// size, never from a call's batch, so an image's statistics are summed in
// the same order at every batch size.
bool fused_gn(const evo_encoder* e, int HW, int chunks) {
  return HW <= kFusedPixels || ((long long)e->desc.max_batch * chunks >= kFusedWG && HW <= kFusedPixelsWide);
}

// GroupNorm of layer L's conv output (g.ws / splits / x set by launch_conv).
hipError_t launch_gn(const evo_encoder* e, const ConvLayer& L, GnArgs g, int N, int H, int W, const float* res,
                     int relu, int mode, float* y, int out_stride, hipStream_t st) {
  const int C = L.cout, G = e->desc.gn_group, groups = C / G;
  int gpw = 1;  // groups per workgroup: up to 64 channels, a power of two dividing the group count
  while (gpw * 2 * G <= 64 && groups % (gpw * 2) == 0) gpw *= 2;
  int chunks = groups / gpw;
  const int HW = H * W;
  const bool fused = fused_gn(e, HW, chunks);
  if (fused && (long long)e->desc.max_batch * chunks < kFusedWG) {
    gpw = 1;  // few images: one group per workgroup, for more workgroups
    chunks = groups;
  }
  const int base = N * chunks;
  // statistics chunks of the max_batch plan (see kGnTarget)
  const int ps = std::max(1, std::min(cdiv(kGnTarget, e->desc.max_batch * chunks), cdiv(HW, 16)));
  if ((size_t)N * groups * ps > e->part_cap) return hipErrorInvalidValue;  // sized at creation
  g.gamma = L.gamma;
  g.beta = L.beta;
  g.res = res;
  g.y = y;
  g.part = e->part;
  g.shift = e->shift;
  g.relu = relu;
  g.mode = mode;
  g.H = H;
  g.W = W;
  g.C = C;
  g.G = G;
  g.gpw = gpw;
  g.ps_stats = ps;
  g.Hp = mode == GN_MAXPOOL ? out_size(H, 3, 2, 1) : 0;
  g.Wp = mode == GN_MAXPOOL ? out_size(W, 3, 2, 1) : 0;
  g.out_stride = out_stride;
  g.eps = 1e-5f;
  const int out_px = mode == GN_MAXPOOL ? g.Hp * g.Wp : HW;
  g.ps_apply = mode == GN_AVGPOOL ? 1 : std::max(1, std::min(cdiv(kGnTarget, base), cdiv(out_px, 16)));
  if (fused) {
    hipLaunchKernelGGL(gn_fused_kernel, dim3((unsigned)base), dim3(kThreads), 0, st, g);
  } else {
    hipLaunchKernelGGL(gn_stats_kernel, dim3((unsigned)(base * ps)), dim3(kThreads), 0, st, g);
    hipLaunchKernelGGL(gn_apply_kernel, dim3((unsigned)(base * g.ps_apply)), dim3(kThreads), 0, st, g);
  }
  return hipGetLastError();
}

}  // namespace

extern "C" {

int64_t evo_encoder_weight_count(const evo_encoder_desc* desc) {
  clear_error();
  int rc = enc_check(desc);
  if (rc) return rc;
  int64_t n = 0;
  for (const ConvLayer& L : enc_layers(desc)) n += (int64_t)L.cout * L.k * L.k * L.cin + 2 * L.cout;
  return n;
}

int evo_create_encoder(const evo_encoder_desc* desc, const float* host_weights, size_t n_floats,
                       evo_encoder** out) {
  clear_error();
  int rc = enc_check(desc);
  if (rc) return rc;
  if (!host_weights || !out) return fail(EVO_E_INVALID, "NULL pointer");
  const int64_t need = evo_encoder_weight_count(desc);
  if ((int64_t)n_floats != need)
    return fail(EVO_E_INVALID, "n_floats is %zu, this encoder needs %lld", n_floats, (long long)need);
  evo_encoder* e = new (std::nothrow) evo_encoder();
  if (!e) return fail(EVO_E_NOMEM, "host allocation failed");
  const auto body = [&]() -> int {
    e->desc = *desc;
    e->bf = desc->dtype == EVO_BF16;
    if (hipGetDevice(&e->device) != hipSuccess) return fail(EVO_E_HIP, "no current HIP device");
#define ENC_TRY(expr)                                                                          \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess)                                                                      \
      return fail(e_ == hipErrorOutOfMemory ? EVO_E_NOMEM : EVO_E_HIP, "%s failed: %s", #expr, \
                  hipGetErrorString(e_));                                                      \
  } while (0)
    // activation sizes and FLOPs: walk the network once
    size_t maxact = 0, maxpart = 0;  // per image: activation floats, GroupNorm partials
    int maxgroups = 0;
    uint64_t flops = 0;
    {
      int h = out_size(desc->height, 7, 2, 3), w = out_size(desc->width, 7, 2, 3);
      maxact = std::max(maxact, (size_t)h * w * desc->stem_ch);
      maxgroups = desc->stem_ch / desc->gn_group;
      maxpart = (size_t)maxgroups * cdiv((long long)h * w, 16);
      flops += 2ull * h * w * desc->stem_ch * 49 * desc->in_ch;
      h = out_size(h, 3, 2, 1);
      w = out_size(w, 3, 2, 1);
      int cin = desc->stem_ch;
      for (int s = 0; s < desc->n_stages; ++s)
        for (int b = 0; b < desc->blocks[s]; ++b) {
          const int c = desc->widths[s], stride = (s > 0 && b == 0) ? 2 : 1;
          const int ho = out_size(h, 3, stride, 1), wo = out_size(w, 3, stride, 1);
          if (ho < 1 || wo < 1) return fail(EVO_E_INVALID, "the image is too small for the network");
          maxact = std::max(maxact, (size_t)ho * wo * c);
          maxgroups = std::max(maxgroups, c / desc->gn_group);
          maxpart = std::max(maxpart, (size_t)(c / desc->gn_group) * cdiv((long long)ho * wo, 16));
          flops += 2ull * ho * wo * c * 9 * cin + 2ull * ho * wo * c * 9 * c;
          if (stride != 1 || cin != c) flops += 2ull * ho * wo * c * cin;
          h = ho;
          w = wo;
          cin = c;
        }
    }
    if (maxact * desc->max_batch >= (size_t(1) << 31))
      return fail(EVO_E_UNSUPPORTED, "activations of max_batch images exceed 2^31 floats");
    e->flops_per_image = flops;
    e->buf_floats = maxact * desc->max_batch;
    e->part_cap = (size_t)desc->max_batch * maxpart;
    e->shift_cap = (size_t)desc->max_batch * maxgroups;
    ENC_TRY(hipMalloc(&e->d_raw, n_floats * sizeof(float)));
    ENC_TRY(hipMemcpy(e->d_raw, host_weights, n_floats * sizeof(float), hipMemcpyHostToDevice));
    e->convs = enc_layers(desc);
    int n_cu = 256;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, e->device) == hipSuccess) n_cu = prop.multiProcessorCount;
    plan_encoder(e, n_cu);
    const int KS = e->bf ? ConvStep<__bf16>::KS : ConvStep<float>::KS;
    size_t off = 0;
    for (ConvLayer& L : e->convs) {
      L.K = L.k * L.k * L.cin;
      L.Kp = (L.K + KS - 1) / KS * KS;
      // (the fused stem's 7 fragments of 32 a channel block exceed Kp for few image channels)
      ENC_TRY(hipMalloc(&L.w, (size_t)L.cout * (e->stem_nb && L.k == 7 ? std::max(L.Kp, 7 * 32) : L.Kp) * (e->bf ? 2 : 4)));
      if (e->fused && L.k != 7) {
        hipLaunchKernelGGL(pack_fused_kernel, dim3(grid_for((long long)L.cout * L.K / 8)), dim3(256), 0, 0, e->d_raw + off,
                           L.cout, L.cin, L.k * L.k, reinterpret_cast<uint4*>(L.w));
        for (const FusedPlan& p : L.fp)
          ENC_TRY(hipFuncSetAttribute(fused_kernel(p.cfg, L.k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes));
      } else if (e->stem_nb && L.k == 7) {
        hipLaunchKernelGGL(pack_stem_kernel, dim3(grid_for(7ll * L.cout * 4)), dim3(256), 0, 0, e->d_raw + off, L.cout, L.cin,
                           reinterpret_cast<uint4*>(L.w));
        for (int nb : {1, e->stem_nb})
          ENC_TRY(hipFuncSetAttribute(stem_fn(nb), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes));
      } else
        hipLaunchKernelGGL(pack_conv_kernel, dim3(grid_for((long long)L.cout * L.Kp)), dim3(256), 0, 0,
                         e->d_raw + off, L.cout, L.K, L.Kp, e->bf, L.w);
      ENC_TRY(hipGetLastError());
      off += (size_t)L.cout * L.K;
      L.gamma = e->d_raw + off;
      L.beta = e->d_raw + off + L.cout;
      off += 2 * (size_t)L.cout;
    }
    for (int i = 0; i < 4; ++i) ENC_TRY(hipMalloc(&e->buf[i], e->buf_floats * sizeof(float)));
    if (!e->fused || !e->stem_nb) {  // some layer runs on the general path
      ENC_TRY(hipMalloc(&e->ws, (size_t)kWsFloats * sizeof(float)));
      ENC_TRY(hipMalloc(&e->zeros, 256));
      ENC_TRY(hipMemset(e->zeros, 0, 256));
      ENC_TRY(hipMalloc(&e->part, e->part_cap * sizeof(double2)));
      ENC_TRY(hipMalloc(&e->shift, e->shift_cap * sizeof(float)));
    }
    ENC_TRY(hipEventCreateWithFlags(&e->ev_done, hipEventDisableTiming));
    ENC_TRY(hipDeviceSynchronize());
#undef ENC_TRY
    *out = e;
    return (int)EVO_OK;
  };
  rc = guarded(body);
  if (rc) evo_destroy_encoder(e);
  return rc;
}

int evo_debug_encoder_plan(const evo_encoder_desc* desc, int32_t batch, int32_t n_cu, int32_t* out, int32_t n_out) {
  clear_error();
  int rc = enc_check(desc);
  if (rc) return rc;
  if (batch < 1 || batch > desc->max_batch || n_cu < 1 || !out) return fail(EVO_E_INVALID, "bad argument");
  return guarded([&]() -> int {
    evo_encoder e;
    e.desc = *desc;
    e.bf = desc->dtype == EVO_BF16;
    e.convs = enc_layers(desc);
    if (n_out < (int)(4 * e.convs.size())) return fail(EVO_E_INVALID, "n_out %d < %zu", n_out, 4 * e.convs.size());
    plan_encoder(&e, n_cu);
    for (size_t i = 0; i < e.convs.size(); ++i) {
      int32_t* o = out + 4 * i;
      const ConvLayer& L = e.convs[i];
      std::fill(o, o + 4, 0);
      if (i == 0 && e.stem_nb) {
        const int nb = batch >= kStemWide ? e.stem_nb : 1;
        o[0] = batch * (L.cout / (16 * nb)), o[1] = 1, o[2] = nb, o[3] = 1;
      } else if (i > 0 && e.fused) {
        const FusedPlan& p = L.fp[plan_class(batch)];
        const FusedCfg& f = kFused[p.cfg];
        o[1] = p.ipw, o[2] = f.nbw * f.wn, o[3] = f.wk;
        o[0] = cdiv(batch, p.ipw) * (L.cout / (16 * o[2]));
      }
    }
    return (int)e.convs.size();
  });
}

int evo_encode(evo_encoder* e, int32_t batch, const float* images, float* features_out, int32_t out_stride,
               void* hip_stream) {
  clear_error();
  if (!e) return fail(EVO_E_INVALID, "encoder is NULL");
  const evo_encoder_desc& d = e->desc;
  if (batch < 1 || batch > d.max_batch) return fail(EVO_E_INVALID, "batch %d outside [1, %d]", batch, d.max_batch);
  if (!images || !features_out) return fail(EVO_E_INVALID, "NULL device pointer");
  // the convolutions read whole input pixels with 16-byte loads where the channel count allows
  if (reinterpret_cast<uintptr_t>(images) % 16)
    return fail(EVO_E_INVALID, "images must be 16-byte aligned");
  const int C_out = d.widths[d.n_stages - 1];
  if (out_stride < C_out) return fail(EVO_E_INVALID, "out_stride %d < feature size %d", out_stride, C_out);
  DeviceGuard guard(e->device);
  hipStream_t st = (hipStream_t)hip_stream;
  float *X = e->buf[0], *Y = e->buf[1], *Z = e->buf[2], *R = e->buf[3];
  int H = d.height, W = d.width, Ho, Wo;
  size_t li = 0;
  GnArgs g{};
#define ENC_HIP(expr)                                                                            \
  do {                                                                                           \
    hipError_t e_ = (expr);                                                                      \
    if (e_ != hipSuccess) return fail(EVO_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)
  // stem: conv 7x7/2, then GroupNorm + ReLU + max pool 3x3/2 in one apply pass
  {
    const ConvLayer& L = e->convs[li++];
    if (e->stem_nb) {
      Ho = out_size(H, 7, 2, 3);
      Wo = out_size(W, 7, 2, 3);
      ENC_HIP(launch_stem(e, L, images, batch, X, reinterpret_cast<__bf16*>(Z), st));
    } else {
      ENC_HIP(launch_conv(e, L, images, batch, H, W, Y, &Ho, &Wo, &g, st));
      g.yb = e->fused ? reinterpret_cast<__bf16*>(Z) : nullptr;
      ENC_HIP(launch_gn(e, L, g, batch, Ho, Wo, nullptr, 1, GN_MAXPOOL, X, 0, st));
    }
    H = out_size(Ho, 3, 2, 1);
    W = out_size(Wo, 3, 2, 1);
  }
  int cin = d.stem_ch;
  if (e->fused) {
    // block input: fp32 in X (where an identity shortcut reads it) and
    // rounded in xb; the inner activation only rounded, in yb; a projected
    // shortcut in fp32 in Y.  A block's output may take its input's place:
    // every element is read by the thread that writes it.
    __bf16 *xb = reinterpret_cast<__bf16*>(Z), *yb = reinterpret_cast<__bf16*>(R);
    for (int s = 0; s < d.n_stages; ++s)
      for (int b = 0; b < d.blocks[s]; ++b) {
        const int c = d.widths[s];
        const bool last = s == d.n_stages - 1 && b == d.blocks[s] - 1;
        const ConvLayer& La = e->convs[li++];
        const ConvLayer& Lb = e->convs[li++];
        const bool proj = La.stride != 1 || cin != c;
        int H2, W2, H3, W3;
        ENC_HIP(launch_fused(La, xb, batch, H, W, &H2, &W2, nullptr, 1, nullptr, yb, nullptr, 0, st));
        const float* shortcut = X;
        if (proj) {
          int Hd, Wd;
          ENC_HIP(launch_fused(e->convs[li++], xb, batch, H, W, &Hd, &Wd, nullptr, 0, Y, nullptr, nullptr, 0, st));
          shortcut = Y;
        }
        const bool next_identity = !last && b + 1 < d.blocks[s];  // (a stage's first block projects its shortcut)
        ENC_HIP(launch_fused(Lb, yb, batch, H2, W2, &H3, &W3, shortcut, 1, next_identity ? X : nullptr,
                             last ? nullptr : xb, last ? features_out : nullptr, out_stride, st));
        H = H3;
        W = W3;
        cin = c;
      }
    ENC_HIP(hipEventRecord(e->ev_done, st));
    e->launched = true;
    return EVO_OK;
  }
  for (int s = 0; s < d.n_stages; ++s)
    for (int b = 0; b < d.blocks[s]; ++b) {
      const int c = d.widths[s];
      const bool last = s == d.n_stages - 1 && b == d.blocks[s] - 1;
      const ConvLayer& La = e->convs[li++];
      const ConvLayer& Lb = e->convs[li++];
      const bool proj = La.stride != 1 || cin != c;
      int H2, W2, H3, W3;
      ENC_HIP(launch_conv(e, La, X, batch, H, W, Y, &H2, &W2, &g, st));
      ENC_HIP(launch_gn(e, La, g, batch, H2, W2, nullptr, 1, GN_PLAIN, Y, 0, st));
      const float* shortcut = X;
      if (proj) {  // before conv b: each conv's partials are consumed before the next conv runs
        const ConvLayer& Ld = e->convs[li++];
        int Hd, Wd;
        ENC_HIP(launch_conv(e, Ld, X, batch, H, W, R, &Hd, &Wd, &g, st));
        ENC_HIP(launch_gn(e, Ld, g, batch, Hd, Wd, nullptr, 0, GN_PLAIN, R, 0, st));
        shortcut = R;
      }
      ENC_HIP(launch_conv(e, Lb, Y, batch, H2, W2, Z, &H3, &W3, &g, st));
      // block output = ReLU(GN(conv b) + shortcut): into Y, or averaged into the features
      if (last) ENC_HIP(launch_gn(e, Lb, g, batch, H3, W3, shortcut, 1, GN_AVGPOOL, features_out, out_stride, st));
      else ENC_HIP(launch_gn(e, Lb, g, batch, H3, W3, shortcut, 1, GN_PLAIN, Y, 0, st));
      std::swap(X, Y);
      H = H3;
      W = W3;
      cin = c;
    }
  ENC_HIP(hipEventRecord(e->ev_done, st));
  e->launched = true;
#undef ENC_HIP
  return EVO_OK;
}

int evo_encoder_flops(const evo_encoder* e, int32_t batch, uint64_t* flops_out) {
  clear_error();
  if (!e || !flops_out) return fail(EVO_E_INVALID, "NULL pointer");
  *flops_out = e->flops_per_image * (uint64_t)std::max(batch, 0);
  return EVO_OK;
}

void evo_destroy_encoder(evo_encoder* e) {
  if (!e) return;
  DeviceGuard guard(e->device);
  // the encoder's own launches end before its buffers are freed (no
  // device-wide wait: other work on the device is not this encoder's)
  if (e->launched && e->ev_done) (void)hipEventSynchronize(e->ev_done);
  for (ConvLayer& L : e->convs) (void)hipFree(L.w);
  for (int i = 0; i < 4; ++i) (void)hipFree(e->buf[i]);
  (void)hipFree(e->ws);
  (void)hipFree(e->zeros);
  (void)hipFree(e->part);
  (void)hipFree(e->shift);
  (void)hipFree(e->d_raw);
  if (e->ev_done) (void)hipEventDestroy(e->ev_done);
  delete e;
}

}  // extern "C"
