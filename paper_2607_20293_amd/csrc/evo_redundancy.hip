// Redundancy-aware initialisation of the schedule search (Sec. 3.3): the
// dissimilarity score of Eq. 6 from activations recorded by the uncached
// policy.  For every query r and unit b the step x step Gram matrix of the
// unit's activation vectors is formed on fp32 MFMA and reduced to the mean
// cosine dissimilarity of each step against the other steps; a last kernel
// averages the queries in order.  Every sum has a fixed order.
//
// What bounds it: the activations are read once (315 MB for 8 Push-T
// queries, 66 us at the 4.8 TB/s of a large copy) and the lower triangle of
// step tiles is 11 GFLOP of fp32 MFMA (73 us at 154 TFLOP/s), so loads and
// MFMAs have to run side by side on every CU.
//  * A Gram tile's two operands have the same lane layout, so a wave loads
//    each 16-step tile of a 32-element chunk once, straight from memory to
//    registers (a row's 128-byte line in two 16-byte loads a lane), and
//    multiplies all pairs of tiles from them: 7 tiles feed 28 x 8 MFMAs, no
//    LDS on the way, the next chunk in flight meanwhile.
//  * The elements are split over the four waves of a workgroup and over KS
//    workgroups (gram_splits), whose partial matrices a second kernel sums;
//    with KS = 1 the workgroup finishes alone.
// Measured (Push-T, 8 queries, 100 steps; the whole call): 470 us with one
// workgroup per (query, unit), LDS staging and all 49 tiles, 120 us now
// (2.6 TB/s of activations).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "evo_kernels.hpp"

namespace evo {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kNW = 4;            // waves per workgroup
constexpr int kKC = 32;           // activation elements per chunk
constexpr int kMaxMT = kGramMaxSteps / 16;
constexpr int pairs_of(int mt) { return mt * (mt + 1) / 2; }

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// element (r, c), r / 16 >= c / 16, of a triangle of 16x16 accumulator tiles
// [pair][lane][4] (lane: column c % 16, rows 4 (lane / 16) .. + 3)
__device__ __forceinline__ int tri_index(int r, int c) {
  const int i = r >> 4, j = c >> 4, m = r & 15, n = c & 15;
  return ((i * (i + 1) / 2 + j) * 64 + n + 16 * (m >> 2)) * 4 + (m & 3);
}

// part[t] = 1/(T-1) sum_{t' != t} (1 - cos(a_t, a_t')) from the Gram triangle
// in LDS (a zero vector's cosine taken as 0); two lanes a row, each half of
// the columns in order.  256 threads.
__device__ __forceinline__ void finish_scores(const float* g, float* nrm, int T, float* part) {
  const int tid = threadIdx.x;
  if (tid < T) nrm[tid] = g[tri_index(tid, tid)];
  __syncthreads();
  const int r = tid >> 1, half = (T + 1) / 2, c0 = (tid & 1) * half, c1 = min(T, c0 + half);
  float s = 0.f;
  if (r < T)
    for (int c = c0; c < c1; ++c)
      if (c != r) {
        const float n2 = nrm[r] * nrm[c];
        const float v = (r >> 4) >= (c >> 4) ? g[tri_index(r, c)] : g[tri_index(c, r)];
        s += 1.f - (n2 > 0.f ? v / sqrtf(n2) : 0.f);
      }
  s += __shfl_xor(s, 1);
  if (r < T && (tid & 1) == 0) part[r] = s / (float)(T - 1);
}

// Workgroup (r, b, ks): the Gram triangle over its share of the V elements,
// written to ws [r, b][ks][pairs][256], or with one share per (r, b) finished
// here.  Steps beyond T repeat the last one and are never read back.
template <int MT>
__global__ void __launch_bounds__(kNW * 64) gram_kernel(const float* __restrict__ acts, int T, int V, int KS,
                                                        float* __restrict__ ws, float* __restrict__ part) {
  constexpr int NP = pairs_of(MT);
  __shared__ __attribute__((aligned(16))) float tri[2][NP * 256];
  __shared__ float nrm[kGramMaxSteps];
  const int rb = blockIdx.x / KS, ks = blockIdx.x % KS;
  const int tid = threadIdx.x, lane = tid & 63, lc = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nch = V / kKC, nw = KS * kNW, wi = ks * kNW + w;
  const int cb = (int)((long long)nch * wi / nw), ce = (int)((long long)nch * (wi + 1) / nw);
  // (T <= 128 steps of V floats: a unit's activations stay below 2^31 bytes,
  // checked by the host)
  const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(acts) + (size_t)rb * T * V, (short)0, T * V * 4,
                                                    0x00020000);
  int off[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) off[i] = (min(i * 16 + lc, T - 1) * V + lq * 8) * 4;
  f32x4 acc[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  // lane group lq takes elements 8 lq .. + 7 of the chunk, one per MFMA (an
  // order of the elements that both operands share)
  const auto load = [&](f32x4 (&x)[MT][2], int c) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        x[i][h] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off[i], c * (kKC * 4) + h * 16, 0));
  };
  const auto multiply = [&](const f32x4 (&x)[MT][2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j <= i; ++j)
            acc[i * (i + 1) / 2 + j] = mfma4(x[i][h][e], x[j][h][e], acc[i * (i + 1) / 2 + j]);
  };
  if (cb < ce) {
    f32x4 x0[MT][2], x1[MT][2];
    load(x0, cb);
    // (a chunk past the wave's share is requested in bounds and not used)
    for (int c = cb; c < ce; c += 2) {
      load(x1, min(c + 1, ce - 1));
      __builtin_amdgcn_sched_barrier(0);
      multiply(x0);
      __builtin_amdgcn_sched_barrier(0);
      load(x0, min(c + 2, ce - 1));
      __builtin_amdgcn_sched_barrier(0);
      if (c + 1 < ce) multiply(x1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // ((w0 + w2) + (w1 + w3)) through LDS
  const auto put = [&](float* dst) {
#pragma unroll
    for (int q = 0; q < NP; ++q) *reinterpret_cast<f32x4*>(dst + (q * 64 + lane) * 4) = acc[q];
  };
  const auto add = [&](const float* src) {
#pragma unroll
    for (int q = 0; q < NP; ++q) acc[q] += *reinterpret_cast<const f32x4*>(src + (q * 64 + lane) * 4);
  };
  if (w >= 2) put(tri[w - 2]);
  __syncthreads();
  if (w < 2) add(tri[w]);
  if (w == 1) put(tri[1]);
  __syncthreads();
  if (w == 0) {
    add(tri[1]);
    if (KS > 1) put(ws + (size_t)blockIdx.x * (NP * 256));
    else put(tri[0]);
  }
  if (KS > 1) return;
  __syncthreads();
  finish_scores(tri[0], nrm, T, part + (size_t)rb * T);
}

// Sums the KS partial triangles of (r, b) in order and finishes it.
__global__ void __launch_bounds__(kNW * 64) gram_finish_kernel(const float* __restrict__ ws, int T, int KS, int NP,
                                                               float* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float tri[pairs_of(kMaxMT) * 256];
  __shared__ float nrm[kGramMaxSteps];
  const f32x4* src = reinterpret_cast<const f32x4*>(ws) + (size_t)blockIdx.x * KS * NP * 64;
  for (int i = threadIdx.x; i < NP * 64; i += kNW * 64) {
    f32x4 s = src[i];
    for (int k = 1; k < KS; ++k) s += src[(size_t)k * NP * 64 + i];
    reinterpret_cast<f32x4*>(tri)[i] = s;
  }
  __syncthreads();
  finish_scores(tri, nrm, T, part + (size_t)blockIdx.x * T);
}

__global__ void mean_kernel(const float* __restrict__ part, int R, int n, float* __restrict__ d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
  for (int r = 0; r < R; ++r) s += part[(size_t)r * n + i];
  d[i] = s / (float)R;
}

// Workgroups per (query, unit).  A workgroup costs its chunks' MFMAs (pairs x
// 8 x 32 cycles each) plus about 6000 cycles to start and to hand its
// triangle over; the CUs run ceil(units x KS / n_cu) of them one after
// another.  The cheapest KS, the smallest of equals, within a partial
// workspace of kMaxParts triangles.
constexpr int kMaxParts = 1024;
int gram_splits(int n, int mt, int V, int n_cu) {
  const int nch = V / kKC;
  long long best = -1;
  int ks = 1;
  for (int k = 1; k <= 64 && (k == 1 || (n * (long long)k <= kMaxParts && 4 * k * 2 <= nch)); ++k) {
    const long long rounds = ((long long)n * k + n_cu - 1) / n_cu, chunks = (nch + 4 * k - 1) / (4 * k);
    const long long cost = rounds * (chunks * pairs_of(mt) * 256 + 6000) + (k > 1 ? 6000 : 0);
    if (best < 0 || cost < best) {
      best = cost;
      ks = k;
    }
  }
  return ks;
}

}  // namespace

size_t redundancy_workspace_floats(int max_queries, int U, int T, long long V, int n_cu) {
  if (T < 2 || T > kGramMaxSteps) return 0;
  const int mt = (T + 15) / 16;
  size_t need = 0;
  for (int R = 1; R <= max_queries && (long long)R * U <= kMaxParts; ++R) {
    const int ks = gram_splits(R * U, mt, (int)V, n_cu);
    if (ks > 1) need = std::max(need, (size_t)R * U * ks * pairs_of(mt) * 256);
  }
  return need;
}

hipError_t launch_redundancy(const float* acts, int R, int U, int T, long long V, int n_cu, float* ws, float* part,
                             float* d, hipStream_t stream) {
  if (R < 1 || U < 1 || T < 2 || T > kGramMaxSteps || V < kKC || V % kKC || (long long)T * V * 4 >= (1ll << 31))
    return hipErrorInvalidValue;
  const int mt = (T + 15) / 16, ks = gram_splits(R * U, mt, (int)V, n_cu);
  const dim3 grid((unsigned)(R * U * ks)), block(kNW * 64);
  switch (mt) {
#define EVO_GRAM(M)                                                                            \
  case M:                                                                                      \
    hipLaunchKernelGGL(gram_kernel<M>, grid, block, 0, stream, acts, T, (int)V, ks, ws, part); \
    break;
    EVO_GRAM(1) EVO_GRAM(2) EVO_GRAM(3) EVO_GRAM(4) EVO_GRAM(5) EVO_GRAM(6) EVO_GRAM(7) EVO_GRAM(8)
#undef EVO_GRAM
  }
  if (ks > 1)
    hipLaunchKernelGGL(gram_finish_kernel, dim3(R * U), block, 0, stream, ws, T, ks, pairs_of(mt), part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int n = U * T;
  hipLaunchKernelGGL(mean_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, part, R, n, d);
  return hipGetLastError();
}

}  // namespace evo
