// HIP kernels (gfx950) of the schedule-driven cached denoising loop.
//
// Design: one workgroup owns a tile of whole samples (rows = samples x
// horizon tokens) for the entire T-step reverse process.  Samples never
// interact, so a tile needs no communication with other workgroups: the
// whole query is one launch with no grid-wide synchronisation.
//
//  * The residual stream h of the tile lives in registers, laid out as the
//    accumulator fragments of 16x16 MFMA tiles (each wave owns a fixed set
//    of 16-column blocks of d).  Every product is formed transposed (weights
//    as the first MFMA operand, activations as the second), so a lane holds
//    four consecutive columns of ONE row: row statistics are sums inside the
//    lane plus two lane swaps, operands go to LDS as one wide store per
//    block, and a product's result can feed the next fp32 product straight
//    from its registers (attention probabilities, the head, the sampler).
//  * The schedule arrives as per-step unit bitmasks {evaluate, reuse,
//    store}.  Cacheable units (Sec. 3.1: SA, CA, FFN residual branches) are
//    evaluated only where the schedule says so (Eq. 1); a refreshed residual
//    is stored in the tile's cache in HBM only if a later step reuses it.
//    Between two evaluated units the reused residuals of the skipped units
//    are added in order, their cache loads issued in batches.
//  * Every unit is "LayerNorm -> chunked stage-1 product -> per-chunk
//    transform (attention per head group, or GELU) -> stage-2 product
//    accumulated into the unit's residual".  Activations stay in LDS;
//    projection weights are streamed from L2/HBM as pre-packed 1 KiB MFMA
//    fragments (16 output columns x 32 bf16 / 16 fp32 of K, 16 bytes per
//    lane), so every weight load is one coalesced 16-byte load per lane, and
//    the first fragments of each product are requested before the phase
//    that precedes it.
//  * Attention, the action embedding and the head use fp32 16x16x4 MFMA
//    tiles; the DDPM update is fused at the end of every step.
#include "evo_kernels.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace evo {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4_dword __attribute__((ext_vector_type(4), aligned(4)));  // in a caller's buffer (float alignment only)

constexpr uint64_t kMergedBit = 1ull << 63;
constexpr int kMaskEntries = 341;  // (T x samples per tile) entries of 3 x u64 in LDS (8 KiB)

// float -> bfloat16 bits, round to nearest even: gfx950's conversion
// instruction (v_cvt_pk_bf16_f32), two values at a time where possible
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}
// (bf16(lo) | bf16(hi) << 16)
__device__ __forceinline__ uint32_t bf16x2_rne(float lo, float hi) {
  const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// fp16 pair: each value clamped to the finite fp16 range, then rounded to
// nearest even (a residual beyond +-65504 is stored as +-65504)
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f16x2_sat(float lo, float hi) {
  const f16x2_t v = {(_Float16)__builtin_amdgcn_fmed3f(lo, -65504.f, 65504.f),
                     (_Float16)__builtin_amdgcn_fmed3f(hi, -65504.f, 65504.f)};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ f32x4 f16x4_to_f32(uint32_t x0, uint32_t x1) {
  const f16x2_t a = __builtin_bit_cast(f16x2_t, x0), b = __builtin_bit_cast(f16x2_t, x1);
  return f32x4{(float)a[0], (float)a[1], (float)b[0], (float)b[1]};
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// 16x16 tile of k · qᵀ over a DH-long dot product on fp32 MFMA: lane holds
// the scores of query lane % 16 with keys 4 (lane / 16) .. + 3.  The K order
// is permuted (any bijection of k works when both operands use it): lane
// group lq takes k = 16·lq + j at step j, so each lane reads 16 contiguous
// floats of its row (four 16-byte LDS reads) instead of 16 strided ones, and
// four independent accumulators shorten the dependent MFMA chain.
// The order of the last sum is a choice among equals, made by its outcome:
// with bf16 operands another rounding of a score travels through all later
// steps, and the worst of the 128 samples of the width-768 batch moves with it
// around the 3e-2 that the tests allow: 2.5e-2 from the exact chunk with this
// order, 3.1e-2 with (a0 + a1) + (a2 + a3).  Neither is the more exact sum; the
// samples' median is 1.1e-2.
template <int DH>
__device__ __forceinline__ f32x4 qk_tile(const float* qrow, const float* krow, int lq) {
  static_assert(DH % 64 == 0 || DH == 32, "head size");
  f32x4 acc[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  constexpr int KPL = DH / 4;  // k per lane group
#pragma unroll
  for (int j4 = 0; j4 < KPL / 4; ++j4) {
    const f32x4 qv = *reinterpret_cast<const f32x4*>(qrow + lq * KPL + 4 * j4);
    const f32x4 kv = *reinterpret_cast<const f32x4*>(krow + lq * KPL + 4 * j4);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = mfma4(kv[e], qv[e], acc[e]);
  }
  return (acc[0] + acc[2]) + (acc[1] + acc[3]);
}

// waves sharing one (head, 16-query block) of attention: each repeats the
// scores and computes its share of the DH / 16 value column blocks
constexpr int attn_waves_per_pair(int nw, int npair, int ncb) {
  int wpp = 1;
  while (wpp * 2 <= nw / (npair > 0 ? npair : 1) && ncb % (wpp * 2) == 0) wpp *= 2;
  return wpp;
}

// Cross-lane moves within a quad of lanes (DPP): swap neighbours (0xB1),
// swap pairs (0x4E).
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

// The values of the two lanes 16 (32) apart that share a lane's low bits, in
// lane order and the same in both lanes: a symmetric function of the pair
// gives both the same bits.  A 16x16 accumulator holds a row in the four
// lanes l, l + 16, l + 32, l + 48, so two such steps reduce a row.
struct Pair {
  float a, b;
};
__device__ __forceinline__ Pair swap16(float v) {
  const u32x2 r = __builtin_bit_cast(
      u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Pair swap32(float v) {
  const u32x2 r = __builtin_bit_cast(
      u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float quad_rows_sum(float v) {
  Pair p = swap16(v);
  p = swap32(p.a + p.b);
  return p.a + p.b;
}
__device__ __forceinline__ float quad_rows_max(float v) {
  Pair p = swap16(v);
  p = swap32(fmaxf(p.a, p.b));
  return fmaxf(p.a, p.b);
}

// Operand traits of the two matmul precisions.  A fragment is 16 bytes per
// lane: 8 bf16 (K = 32 per fragment, one 16x16x32 MFMA) or 4 fp32 (K = 16
// per fragment, four 16x16x4 MFMAs).
template <class AT> struct Op;

template <> struct Op<__bf16> {
  static constexpr int KF = 32, VE = 8, PAD = 8;
  __device__ static __forceinline__ void store(__bf16* buf, int ld, int row, int k, float v) {
    reinterpret_cast<uint16_t*>(buf)[row * ld + k] = (uint16_t)bf16_rne(v);
  }
  // four consecutive k (k a multiple of 4)
  __device__ static __forceinline__ void store4(__bf16* buf, int ld, int row, int k, f32x4 v) {
    *reinterpret_cast<u32x2*>(buf + row * ld + k) = u32x2{bf16x2_rne(v[0], v[1]), bf16x2_rne(v[2], v[3])};
  }
  // acc (rows: output columns, columns: tile rows) += weights w x activations a
  __device__ static __forceinline__ void mma(f32x4& acc, uint4 w, uint4 a) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w),
                                                  __builtin_bit_cast(bf16x8_t, a), acc, 0, 0, 0);
  }
};

template <> struct Op<float> {
  // a lane's four consecutive k feed four 16x16x4 MFMAs (k order permuted
  // alike in both operands)
  static constexpr int KF = 16, VE = 4, PAD = 4;
  __device__ static __forceinline__ void store(float* buf, int ld, int row, int k, float v) { buf[row * ld + k] = v; }
  __device__ static __forceinline__ void store4(float* buf, int ld, int row, int k, f32x4 v) {
    *reinterpret_cast<f32x4*>(buf + row * ld + k) = v;
  }
  __device__ static __forceinline__ void mma(f32x4& acc, uint4 w, uint4 a) {
    acc = mfma4(__uint_as_float(w.x), __uint_as_float(a.x), acc);
    acc = mfma4(__uint_as_float(w.y), __uint_as_float(a.y), acc);
    acc = mfma4(__uint_as_float(w.z), __uint_as_float(a.z), acc);
    acc = mfma4(__uint_as_float(w.w), __uint_as_float(a.w), acc);
  }
};

// acc[m][rb] += (A[rb*16 .. +16][k-range] x W[col block gcb(m)][k-range]^T)^T
// A: LDS operand, row stride lda elements, offset to the k-range start.
// W: packed fragments of a matrix with KBT fragments per column block; kf0
// is the first fragment of the k-range, NKF its length.  Weight fragments are
// requested PD k-steps ahead of their MFMAs (about six 1 KiB fragments in
// flight per wave); a scheduling fence per step keeps the compiler from
// hoisting further loads.  (The products outside the layers: observation
// tokens and their keys and values.)
template <class AT, int RBk, int MPW, int NKF, class GCB>
__device__ __forceinline__ void gemm_acc(f32x4 (&acc)[MPW][RBk], const AT* A, int lda, const uint4* W, int KBT,
                                         int kf0, GCB gcb, int lane) {
  using O = Op<AT>;
  constexpr int PD0 = 6 / MPW > 0 ? 6 / MPW : 1, PD = PD0 < NKF ? PD0 : (NKF > 1 ? NKF - 1 : 1);
  const int lc = lane & 15, lq = lane >> 4;
  const uint4* wp[MPW];
#pragma unroll
  for (int m = 0; m < MPW; ++m) wp[m] = W + ((size_t)gcb(m) * KBT + kf0) * 64 + lane;
  uint4 buf[PD + 1][MPW];
#pragma unroll
  for (int d = 0; d < PD; ++d)
#pragma unroll
    for (int m = 0; m < MPW; ++m)
      if (d < NKF) buf[d][m] = wp[m][d * 64];
#pragma unroll
  for (int kf = 0; kf < NKF; ++kf) {
    if (kf + PD < NKF) {
#pragma unroll
      for (int m = 0; m < MPW; ++m) buf[(kf + PD) % (PD + 1)][m] = wp[m][(kf + PD) * 64];
    }
    uint4 a[RBk];
#pragma unroll
    for (int rb = 0; rb < RBk; ++rb)
      a[rb] = *reinterpret_cast<const uint4*>(A + (rb * 16 + lc) * lda + kf * O::KF + lq * O::VE);
#pragma unroll
    for (int m = 0; m < MPW; ++m)
#pragma unroll
      for (int rb = 0; rb < RBk; ++rb) O::mma(acc[m][rb], buf[kf % (PD + 1)][m], a[rb]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// a value every lane of the wave holds alike, as a scalar
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (uint64_t)hi << 32 | lo;
}

// Hardware transcendental approximations (v_rsq_f32, v_exp_f32, v_rcp_f32;
// about 1 ulp).  The phases around the matrix products run at one or two
// waves per SIMD, where every dependent instruction is exposed latency; the
// correctly rounded library sequences cost tens of instructions each.
__device__ __forceinline__ float fast_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
constexpr float kLog2e = 1.4426950408889634f;

// GELU with the error function (0.5 v (1 + erf(v / sqrt 2))).  erfc(x) for
// x >= 0 uses the rational-exponential approximation of Abramowitz and
// Stegun, Handbook of Mathematical Functions, formula 7.1.26 (absolute error
// below 1.5e-7); 1 + erf(v/sqrt2) is then erfc(|x|) for v < 0 and
// 2 - erfc(|x|) for v >= 0, which avoids cancellation on the negative side.
__device__ __forceinline__ float gelu_erf(float v) {
  const float x = fabsf(v) * 0.70710678118654752f;
  const float t = fast_rcp(1.0f + 0.3275911f * x);
  const float poly =
      t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float q = poly * fast_exp2(-x * x * kLog2e);  // erfc(x)
  return 0.5f * v * (v >= 0.f ? 2.0f - q : q);
}

template <class AT, int D, int DH, int HZ, int SPT, int DFF, int NW, int HG, int FC, int SMAX, int TEAM>
struct Cfg {
  static constexpr int NWV = NW;
  static constexpr int NT = NW * 64;
  static constexpr int R = SPT * HZ;
  static constexpr int RB = R / 16;
  static constexpr int NH = D / DH;
  static constexpr int CB = D / 16;
  static constexpr int CBW = CB / NW;
  static constexpr int GW = HG * DH;
  static constexpr int LDY = 3 * GW + 4;
  static constexpr int ZW = GW > FC ? GW : FC;
  static constexpr int KOBS = 64;
  static constexpr int NJB = HZ >= 16 ? HZ / 16 : 1;   // key blocks per query block (self-attention)
  static constexpr int SPB = HZ >= 16 ? 1 : 16 / HZ;   // samples per 16-row block
  static constexpr int SLOTS = 16 / SPB;               // memory columns per sample in a 16-wide tile
  static constexpr int LDR = 2 * NW + 4;               // LayerNorm partials per row (padded: no bank conflicts)
  static constexpr int NB = (8 / (CBW * RB)) > 0 ? (8 / (CBW * RB)) : 1;  // reuse loads per batch
  // cross-attention folded into per-token fold records (width 256; one
  // sample per 16-row block); used when n_heads x memory tokens <= 16
  static constexpr bool FOLD = D == 256 && HZ >= 16;
  static constexpr int REC = 2 * NH * D + 16;                              // floats per fold record
  static constexpr int FOLD_LDS = FOLD ? NW * RB * 256 : 0;  // partial scores of the waves

  // Weight streams.  A wave's fragments of one group of a unit (TY 0
  // self-attention: a head group's q, k, v columns, then its slice of W_o;
  // 1 projected cross-attention: q columns, W_o2; 2 feed-forward: a chunk of
  // W_1, then of W_2) form one sequence, in the order they are multiplied,
  // and travel through a ring of P fragments of registers: the first P are
  // requested before the unit's LayerNorm, the load of sequence element i + P
  // is issued when element i has been multiplied, and the last P loads of a
  // group are the first P of the unit's next one, so a wave has P KiB of
  // weights in flight from the unit's start to its end, also while attention
  // and GELU run.
  static constexpr int KF = sizeof(AT) == 2 ? 32 : 16;
  static constexpr int K1 = D / KF;  // k-steps of a product over d
  static constexpr int m1(int ty) { return (ty == 0 ? 3 * GW / 16 : ty == 1 ? GW / 16 : FC / 16) / NW; }
  // column blocks multiplied together in stage 1 (feed-forward with bf16
  // operands: two at a time, so that the GELU of one pair runs while the next
  // pair streams; fp32 products need the independent accumulators of more)
  static constexpr int g1(int ty) { return ty == 2 && sizeof(AT) == 2 && m1(2) % 2 == 0 ? 2 : m1(ty); }
  static constexpr int k2(int ty) { return (ty == 2 ? FC : GW) / KF; }
  static constexpr int kbt2(int ty) { return ty == 2 ? DFF / KF : K1; }  // fragments per column block, stage 2
  static constexpr int s1(int ty) { return K1 * m1(ty); }
  static constexpr int total(int ty) { return s1(ty) + k2(ty) * CBW; }
  // ring size: 16 fragments a wave (128 KiB in flight per CU; Push-T batch 1
  // with bf16 operands 3.54, 3.42, 3.35, 3.35 ms with 4, 8, 16, 32), or what
  // divides a short sequence.  Width 768: 8, which leaves registers for the
  // running layer sums (batch 128 37.6 ms with 16 or 8 and
  // the sums in memory, 47.4 ms with 16 and the sums in registers, 35.7 ms
  // with 8)
  static constexpr int PLIM = D > 256 ? 8 : 16;
  static constexpr int ring_size() {
    int p = PLIM;
    while (p > 1 && (total(0) < p || total(1) < p || total(2) < p || total(0) % p || total(2) % p)) p /= 2;
    return p;
  }
  // float offsets of one layer's small tensors (flat order of evo.h) from the
  // layer's first parameter, and a layer's parameter count
  static constexpr int DD = D * D;
  static constexpr int pLN1 = 0, pBQKV = 2 * D + 3 * DD, pBO = 5 * D + 4 * DD, pLN2 = 6 * D + 4 * DD,
                       pBQ = 8 * D + 5 * DD, pBO2 = 11 * D + 8 * DD, pLN3 = 12 * D + 8 * DD,
                       pB1 = 14 * D + 8 * DD + DFF * D, pB2 = 14 * D + 8 * DD + DFF + 2 * DFF * D,
                       PLAYER = 15 * D + 8 * DD + DFF + 2 * DFF * D;
  // sequence length with the padding that keeps the next sequence at slot 0
  static constexpr int padded(int ty) { return (total(ty) + ring_size() - 1) / ring_size() * ring_size(); }
  // byte offsets inside one layer's packed matrices (qkv, o, q, kv, o2, w1, w2)
  static constexpr int FB = D * D / (16 * KF) * 1024;  // a d x d matrix
  static constexpr int LAYER = 8 * FB + 2 * (DFF / D) * FB;
  static constexpr int off1(int ty) { return ty == 0 ? 0 : ty == 1 ? 4 * FB : 8 * FB; }
  static constexpr int off2(int ty) { return ty == 0 ? 3 * FB : ty == 1 ? 7 * FB : 8 * FB + (DFF / D) * FB; }
  // constant part of the offset of sequence element i
  static constexpr int elem(int ty, int i) {
    if (i < s1(ty)) {
      const int r = i % (K1 * g1(ty)), k = r / g1(ty), m = i / (K1 * g1(ty)) * g1(ty) + r % g1(ty);
      const int nb = ty == 0 ? (NW * m) / (GW / 16) * CB + (NW * m) % (GW / 16) : NW * m;
      return off1(ty) + (nb * K1 + k) * 1024;
    }
    const int j = i - s1(ty);
    return off2(ty) + (j % CBW * kbt2(ty) + j / CBW) * 1024;
  }
  // wave- and group-dependent part (layer base included by the caller)
  static constexpr int wave1(int ty, int w, int g) { return (g * ((ty == 2 ? FC : GW) / 16) + w) * K1 * 1024; }
  static constexpr int wave2(int ty, int w, int g) { return (w * CBW * kbt2(ty) + g * k2(ty)) * 1024; }
};

// Cross-attention with few memory tokens, folded.  With q = x W_q^T + b_q
// (x the LayerNorm output of a row), the score of head h against memory
// token j is q_h . k_jh = x . u_jh + c_jh with u_jh = W_q,h^T k_jh (W_q,h the
// head's DH rows of W_q) and c_jh = b_q,h . k_jh, and the unit's output
// sum_h sum_j p_jh v_jh W_o2,h^T + b_o2 = sum_h sum_j p_jh w_jh + b_o2 with
// w_jh = W_o2,h v_jh (W_o2,h the head's DH columns of W_o2).  Projecting the
// S tokens once per (token, layer) replaces the two d x d products of every
// evaluation by two products with S x n_heads columns.
//
// A fold record holds u [NH][D], w [NH][D] and c [NH].  The
// workgroup folds `nrows` <= MR key/value rows (kv: [row][2D] keys then
// values, row stride ldkv, in LDS) with the layer's W_q (rows), the
// transposed W_o2 (row e = column e of W_o2) and b_q; dst(row) is the record
// of a row or null.  Weights are rounded to bf16 first when BF, as the packed matrices.
template <int D, int DH, int NT, int MR, bool BF, class DST>
__device__ void fold_rows(const float* __restrict__ raw, uint32_t wq, uint32_t wo2t,
                                                    uint32_t bq, const float* kv, int ldkv, int nrows, DST dst,
                                                    int tid) {
  constexpr int NH = D / DH, C4 = D / 4, EB = 32;  // EB weight rows requested at once
  static_assert(DH % EB == 0, "fold batches");
  // work item = (u or w, head, 4 columns): the head's DH weight rows are
  // read 16 bytes per lane, EB rows in flight
  for (int it = tid; it < 2 * NH * C4; it += NT) {
    const int isw = it / (NH * C4), hd = (it / C4) % NH, c0 = (it % C4) * 4;
    const float* W = raw + (isw ? wo2t : wq) + (size_t)hd * DH * D + c0;
    const float* kr = kv + (isw ? D : 0) + hd * DH;
    f32x4 acc[MR];
#pragma unroll
    for (int r = 0; r < MR; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int e0 = 0; e0 < DH; e0 += EB) {
      f32x4 wv[EB];
#pragma unroll
      for (int e = 0; e < EB; ++e) wv[e] = *reinterpret_cast<const f32x4*>(W + (size_t)(e0 + e) * D);
      if (BF) {
#pragma unroll
        for (int e = 0; e < EB; ++e)
#pragma unroll
          for (int q = 0; q < 4; ++q) wv[e][q] = __uint_as_float(bf16_rne(wv[e][q]) << 16);
      }
#pragma unroll
      for (int r = 0; r < MR; ++r)
        if (r < nrows) {
#pragma unroll
          for (int e4 = 0; e4 < EB / 4; ++e4) {
            const f32x4 kk = *reinterpret_cast<const f32x4*>(kr + r * ldkv + e0 + 4 * e4);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int t = 0; t < 4; ++t) acc[r][t] = fmaf(wv[4 * e4 + q][t], kk[q], acc[r][t]);
          }
        }
    }
#pragma unroll
    for (int r = 0; r < MR; ++r)
      if (r < nrows) {
        float* q = dst(r);
        if (!q) continue;
        *reinterpret_cast<f32x4*>(q + (isw ? NH * D : 0) + hd * D + c0) = acc[r];
      }
  }
  for (int it = tid; it < nrows * NH; it += NT) {
    const int r = it / NH, hd = it % NH;
    float a = 0.f;
    for (int e = 0; e < DH; ++e) a = fmaf(raw[bq + hd * DH + e], kv[r * ldkv + hd * DH + e], a);
    float* q = dst(r);
    if (q) q[2 * NH * D + hd] = a;
  }
}

// LayerNorm statistics of the tile rows from the register-resident stream: a
// lane takes (mean, M2) of its columns of its row, two lane swaps merge the
// four lanes of the row, the waves' partials meet in LDS (one barrier), and
// every lane merges its row's partials itself in a fixed tree (pairwise,
// equal counts), so all waves hold the same bits.
// (m, q) of two equal groups of n values each: mean of the two means, M2 sum
// plus the spread term (symmetric, so both partners agree bitwise)
__device__ __forceinline__ void merge_stats(float& m, float& q, float ma, float qa, float mb, float qb, float n) {
  const float d = mb - ma;
  m = 0.5f * (ma + mb);
  q = qa + qb + d * d * (0.5f * n);
}
template <class C>
__device__ __forceinline__ void ln_stats(const f32x4 (&h)[C::CBW][C::RB], float (*red)[C::LDR], float (&mu)[C::RB],
                                         float (&rs)[C::RB], int w, int lc, int lq) {
  constexpr int D = C::CB * 16, NWV = C::NWV;
  static_assert((NWV & (NWV - 1)) == 0, "pairwise merges of the waves");
#pragma unroll
  for (int rb = 0; rb < C::RB; ++rb) {
    float m = 0.f;
#pragma unroll
    for (int c = 0; c < C::CBW; ++c) m += (h[c][rb][0] + h[c][rb][1]) + (h[c][rb][2] + h[c][rb][3]);
    m *= 0.25f / C::CBW;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < C::CBW; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = h[c][rb][i] - m;
        q += e * e;
      }
    Pair pm = swap16(m), pq = swap16(q);
    merge_stats(m, q, pm.a, pq.a, pm.b, pq.b, 4.f * C::CBW);
    pm = swap32(m);
    pq = swap32(q);
    merge_stats(m, q, pm.a, pq.a, pm.b, pq.b, 8.f * C::CBW);
    if (lq == 0) *reinterpret_cast<f32x2*>(&red[rb * 16 + lc][2 * w]) = f32x2{m, q};
  }
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < C::RB; ++rb) {
    float m[NWV], q[NWV];
#pragma unroll
    for (int x = 0; x < NWV / 2; ++x) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&red[rb * 16 + lc][4 * x]);
      m[2 * x] = v[0];
      q[2 * x] = v[1];
      m[2 * x + 1] = v[2];
      q[2 * x + 1] = v[3];
    }
    float n = 16.f * C::CBW;
#pragma unroll
    for (int st = 1; st < NWV; st *= 2) {
#pragma unroll
      for (int x = 0; x < NWV; x += 2 * st) merge_stats(m[x], q[x], m[x], q[x], m[x + st], q[x + st], n);
      n *= 2.f;
    }
    mu[rb] = m[0];
    rs[rb] = fast_rsqrt(q[0] * (1.0f / D) + 1e-5f);
  }
}

template <class AT, int D, int DH, int HZ, int SPT, int DFF, int NW, int HG, int FC, int SMAX, int TEAM>
__global__ void __launch_bounds__(NW * 64) denoise_kernel(const KParams p) {
  using O = Op<AT>;
  using OF = Op<float>;
  using C = Cfg<AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM>;
  constexpr int NT = C::NT, R = C::R, RB = C::RB, NH = C::NH, CB = C::CB, CBW = C::CBW, GW = C::GW;
  constexpr int LDA = D + O::PAD, LDY = C::LDY, LDZ = C::ZW + O::PAD;
  constexpr int KOBS = C::KOBS, LDO = KOBS + O::PAD;
  constexpr int NJB = C::NJB, SLOTS = C::SLOTS, NB = C::NB;
  static_assert(R % 16 == 0 && CB % NW == 0 && NH % HG == 0 && DFF % FC == 0, "tile shape");
  static_assert((3 * GW / 16) % NW == 0 && (GW / 16) % NW == 0 && (FC / 16) % NW == 0, "block split");
  static_assert((NH / HG) % TEAM == 0 && (DFF / FC) % TEAM == 0, "team members split head groups and chunks");
  static_assert(HZ % 4 == 0 && (HZ & (HZ - 1)) == 0 && HZ <= 64, "horizon must be a power of two in [4, 64]");
  static_assert(NW * RB * 256 <= R * LDY, "head partials must fit the stage-1 buffer");
  static_assert(16 * LDO * (int)sizeof(AT) <= R * LDY * 4, "observation operand must fit");
  static_assert(SMAX <= SLOTS, "memory tokens per sample must fit a 16-column tile");
  static_assert(DH % 16 == 0, "head dim");
  // embedding / head constants of the lane's columns, kept across steps in
  // LDS (EMB_LDS, where it fits) or in registers (KEEP_EMB), else re-read
  constexpr bool EMB_LDS = RB == 1 && CBW <= 4 && (sizeof(AT) == 2 || TEAM > 1 || D <= 64);
  constexpr bool KEEP_EMB = RB == 1 && CBW <= 4 && !EMB_LDS;
  constexpr bool PB_LDS = EMB_LDS && (TEAM > 1 || D <= 64);  // else the row biases stay in registers
  // Operand rows read from LDS one k-step ahead: with fp32 operands (batch 37
  // 2.99 -> 2.92 ms) and tiles of two row blocks (population of 512 9.83 ->
  // 9.61 ms); a bf16 k-step of one row block is too short to gain by it (Push-T
  // batch 1 3.36 ms without, 3.40 with)
  constexpr bool KAHEAD = RB == 2 || sizeof(AT) == 4;
  constexpr float kScale = (DH == 64) ? 0.125f : (DH == 32 ? 0.17677669529663688f : 0.0f);
  static_assert(DH == 64 || DH == 32, "head dim");

  __shared__ __attribute__((aligned(16))) AT xa[R * LDA];
  __shared__ __attribute__((aligned(16))) float ybuf[R * LDY > C::FOLD_LDS ? R * LDY : C::FOLD_LDS];
  // the feed-forward chunks alternate between two operand buffers, so a
  // chunk's GELU outputs never overwrite the previous chunk's while a wave
  // may still read them, and no barrier ends a chunk (where LDS allows)
  constexpr bool ZB2 = DFF / FC > TEAM && !(sizeof(AT) == 4 && SPT > 1) && R * LDZ * (int)sizeof(AT) <= 20 * 1024;
  __shared__ __attribute__((aligned(16))) AT zbuf[(ZB2 ? 2 : 1) * R * LDZ];
  __shared__ __attribute__((aligned(16))) float kvbuf[SPT * SMAX * 2 * GW];
  __shared__ __attribute__((aligned(16))) float red[R][C::LDR];
  __shared__ uint64_t msk[kMaskEntries * 3];
  __shared__ int smp[SPT];

  const int tid = threadIdx.x;
  // the wave index in a scalar register: weight, bias and cache addresses
  // are then scalar bases plus one per-lane offset
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // lane indices are made opaque to the optimiser (an empty asm) once per
  // step, unit, head group and d_ff chunk, so that the address arithmetic
  // derived from them is recomputed inside the loops instead of being
  // hoisted into registers held for the whole kernel (which spilled)
  int lane = tid & 63, lc = lane & 15, lq = lane >> 4;
  // a team of TEAM workgroups shares a tile: each member evaluates its share
  // of every unit's head groups / d_ff chunks and the partial residuals are
  // summed through HBM; everything else is replicated in every member
  const int member = blockIdx.x % TEAM;
  const int tile = blockIdx.x / TEAM;
  __shared__ int s_abort;
  const int L = p.L, A = p.A, T = p.T, U = 3 * L, nobs = p.n_obs, S = 1 + nobs;
  const float* raw = p.raw;
  // folded cross-attention (n_heads x S <= 16, checked by the host): okv
  // then holds fold records [batch][L][n_obs][REC] instead of keys/values
  const bool fold = C::FOLD && p.fold != 0;
  constexpr int REC = C::REC;

  if (tid < SPT) smp[tid] = p.tile_sample[tile * SPT + tid];
  if (tid == 0) s_abort = 0;
  float* const okv = p.okv + (size_t)member * p.okv_member_stride;
  for (int it = tid; it < SPT * T * 3; it += NT) {
    const int j = it / (T * 3), r = it % (T * 3);
    msk[it] = p.masks[(size_t)p.tile_slot[tile * SPT + j] * T * 3 + r];
  }
  __syncthreads();

  // the tile's samples as scalars, and the sample of this lane's rows in
  // row block rb
  int ssmp[SPT];
#pragma unroll
  for (int j = 0; j < SPT; ++j) ssmp[j] = __builtin_amdgcn_readfirstlane(smp[j]);
  const auto row_sample = [&](int rb) { return HZ >= 16 ? ssmp[rb * 16 / HZ] : smp[(rb * 16 + lc) / HZ]; };

  // current sample x_t of this lane's rows (row rb * 16 + lc, actions
  // 4 lq .. + 3, zero beyond A): every wave keeps its own copy and updates it
  // alike, so that the sampler's result feeds the next step's embedding
  // product from registers
  f32x4 xv[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = rb * 16 + lc, s = row_sample(rb);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int a = 4 * lq + i;
      xv[rb][i] = (s >= 0 && a < A) ? p.noise[((size_t)s * HZ + (row % HZ)) * A + a] : 0.f;
    }
  }

  // ---- per query: observation tokens and their keys/values in every layer
  // (folded: their fold records come from the observation pre-pass)
  if (!fold) {
    constexpr int MPWO = CB / NW;
    f32x4 acc[MPWO][1];
#pragma unroll
    for (int m = 0; m < MPWO; ++m) acc[m][0] = f32x4{0.f, 0.f, 0.f, 0.f};
    AT* ob = reinterpret_cast<AT*>(ybuf);
    const int nch = p.obs_pad / KOBS;
    for (int c = 0; c < nch; ++c) {
      __syncthreads();
      for (int it = tid; it < 16 * KOBS; it += NT) {
        const int row = it / KOBS, k = it % KOBS, kk = c * KOBS + k;
        float v = 0.f;
        if (row < SPT * nobs) {
          const int j = row / nobs, o = row % nobs;
          if (smp[j] >= 0 && kk < p.obs_dim) v = p.obs[((size_t)smp[j] * nobs + o) * p.obs_dim + kk];
        }
        O::store(ob, LDO, row, k, v);
      }
      __syncthreads();
      gemm_acc<AT, 1, MPWO, KOBS / O::KF>(acc, ob, LDO, p.pk + p.pk_obs, p.obs_pad / O::KF, c * (KOBS / O::KF),
                                           [&](int m) { return w + NW * m; }, lane);
    }
    // memory-token operand rows (row = slot*n_obs + token) in xa
    const int orow = lc, oj = orow / nobs, oo = orow % nobs;
    const bool olive = orow < SPT * nobs && smp[oj] >= 0;
#pragma unroll
    for (int m = 0; m < MPWO; ++m) {
      const int gcol = (w + NW * m) * 16 + lq * 4;
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (olive)
        v = acc[m][0] + *reinterpret_cast<const f32x4*>(raw + p.b_obs + gcol) +
            *reinterpret_cast<const f32x4*>(raw + p.P_mem + (size_t)(1 + oo) * D + gcol);
      O::store4(xa, LDA, orow, gcol, v);
    }
    __syncthreads();
    constexpr int MPWK = 2 * CB / NW;
    for (int l = 0; l < L; ++l) {
      f32x4 kv[MPWK][1];
#pragma unroll
      for (int m = 0; m < MPWK; ++m) kv[m][0] = f32x4{0.f, 0.f, 0.f, 0.f};
      gemm_acc<AT, 1, MPWK, D / O::KF>(kv, xa, LDA, p.pk + p.loff[l].pk_kv, D / O::KF, 0,
                                        [&](int m) { return w + NW * m; }, lane);
      const uint32_t bkv = p.loff[l].b_kv;
#pragma unroll
      for (int m = 0; m < MPWK; ++m) {
        const int gcol = (w + NW * m) * 16 + lq * 4;
        if (olive)
          *reinterpret_cast<f32x4*>(okv + (((size_t)smp[oj] * L + l) * nobs + oo) * (2 * D) + gcol) =
              kv[m][0] + *reinterpret_cast<const f32x4*>(raw + bkv + gcol);
      }
    }
    __syncthreads();
  }

  // sample slot of each of this lane's rows
  int jrow[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) jrow[rb] = HZ >= 16 ? rb * 16 / HZ : (rb * 16 + lc) / HZ;
  // residual caches of this workgroup: [3L][R*D] values in fragment order.
  // fp16 with bf16 operands (rounded once per stored residual, clamped to
  // the finite fp16 range; the stream and the layer sums stay fp32): half
  // the bytes of the reuse loads, which every tile of a shared schedule
  // issues at the same time.  fp16 rather than bf16: bf16 caches took the
  // 512-sample population's worst sample past the bf16 error bar
  // (3.04e-2).  fp32 with fp32 operands.  One format for every tile size,
  // so that a sample's result does not depend on the batch.
  constexpr int CE = (sizeof(AT) == 2) ? 2 : 4;
  unsigned char* const cbase = reinterpret_cast<unsigned char*>(p.cache) + (size_t)(tile * TEAM + member) * U * (R * D) * CE;
  // Team exchange slots: [tile][XS][XM][R*D] floats, slot n % XS carries the
  // n-th exchanged unit.  A slot word that still holds the sentinel has not
  // been written yet.  Wave w of a member reads only words that wave w of
  // another member writes, so the following holds wave by wave.
  //  * Three slots (XM = TEAM partials): a member empties its slot of unit n-1
  //    once it holds all partials of unit n.  A member publishes its partial
  //    of unit n after it has read everything of unit n-1, so nobody reads the
  //    slot any more.  Its next use is unit n+2, and its next reader polls it
  //    only after reading this member's partial of unit n+1, which is stored
  //    after the wait (vmcnt 0) for the emptying stores.
  //  * Four slots (SCATTER; XM = TEAM partials and the sums): a member empties
  //    its slot of unit n-2, and its own columns of that slot's sums, together
  //    with the stores of its partial of unit n, before any of unit n is read.
  //    It then holds all sums of unit n-1, each published by an owner that had
  //    read everything of unit n-2, so nobody reads the slot any more.  Its
  //    next use is unit n+2, and its next reader polls it only after reading
  //    this member's partials and sums of unit n+1, stored after the wait for
  //    the emptying stores.
  // SC1 cache-policy bit: device-coherent access; at width 768 also the
  // non-temporal bit, so that the exchange traffic (three 96 KiB slots per
  // member and unit) does not displace the weights from the L2
  constexpr int kCoherent = D > 256 ? (16 | 2) : 16;
  constexpr unsigned kEmpty = 0xFFFFFFFFu;  // never produced by arithmetic (canonical NaN differs)
  int nbar = 0;                             // evaluated units exchanged so far
  // Teams of more than two on a tile too wide to read every member's whole
  // partial (SCATTER): each member sums its share of the column blocks and
  // publishes the sums in a result slot beside the members' slots, so it
  // reads about two partials' worth a unit instead of TEAM - 1 (width 768,
  // teams of 6: 176 KiB instead of 480).
  constexpr bool SCATTER = TEAM > 2 && CBW * RB > 4;
  static_assert(!SCATTER || CBW % TEAM == 0, "column blocks per member");
  // SCATTER has a fourth slot, so that a slot is emptied two units after its
  // use, together with the stores of that unit's partials (the stores that
  // empty a slot of the unit just summed would be waited for by the next
  // unit's first loads)
  constexpr int XM = SCATTER ? TEAM + 1 : TEAM, OWN = SCATTER ? CBW / TEAM : 1, XS = SCATTER ? 4 : 3;
  float* const xb = TEAM > 1 ? p.xchg + (size_t)tile * (XS * XM) * (R * D) : nullptr;
  const auto xr = __builtin_amdgcn_make_buffer_rsrc(xb, (short)0, TEAM > 1 ? XS * XM * R * D * 4 : 0, 0x00020000);
  // byte offset of this lane's fragment (c, rb) in a member's slot, split
  // into a per-lane part (VGPR) and a constant part (SGPR), so that a wide
  // tile does not hold one offset register per fragment
  const auto xoff = [&](int slot, int m) { return ((slot * XM + m) * (R * D) + (w * RB * CBW * 64 + lane) * 4) * 4; };
  const auto xcst = [](int c, int rb) { return (rb * CBW + c) * 1024; };
  // Stores take the whole offset in the VGPR: with an SGPR offset the compiler
  // leaves out the wait states between a 16-byte store and the next write of
  // its data registers, and the last four lanes of each sixteen then stored
  // the new contents (seen when that write was the very next instruction)
  const auto xstore = [&](u32x4 v, int slot, int m, int c, int rb) {
    __builtin_amdgcn_raw_buffer_store_b128(v, xr, xoff(slot, m) + xcst(c, rb), 0, kCoherent);
  };
  if constexpr (TEAM > 1) {
    // all slots of this member start empty; one counter barrier makes
    // sure no member reads a slot before its owner has emptied it
    const u32x4 empty = {kEmpty, kEmpty, kEmpty, kEmpty};
#pragma unroll
    for (int sl = 0; sl < XS; ++sl)
#pragma unroll
      for (int c = 0; c < CBW; ++c)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          xstore(empty, sl, member, c, rb);
          if (SCATTER && c / OWN == member)
            xstore(empty, sl, TEAM, c, rb);
        }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    if (tid == 0) {
      unsigned* ctr = p.tctr + (size_t)tile * 16;
      __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned spins = 0;
      while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (unsigned)TEAM) {
        if (__hip_atomic_load(p.derr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u || ++spins > 4u * p.spin_limit) {
          __hip_atomic_store(p.derr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          s_abort = 1;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __syncthreads();
    if (s_abort) return;
  }
  // element index of this lane's fragment (c, rb) in a unit's cache slot
  const auto cidx = [&](int unit, int c, int rb) {
    return (size_t)unit * (R * D) + ((size_t)((w * RB + rb) * CBW + c) * 64 + lane) * 4;
  };
  // Cache-policy bits of the residual-cache accesses (and of the memory
  // tokens' keys and values).  At
  // width 768 a unit's weights exceed an XCD's L2 and a cached residual is
  // 48 KiB, so these reads and writes are non-temporal (evicted first) and
  // leave the L2 to the weights; at width 256 the default policy measured
  // faster.
  constexpr int CPOL = D > 256 ? 2 : 0;
  const auto cload = [&](int unit, int c, int rb) -> f32x4 {
    if constexpr (CE == 2) {
      const u32x2* q = reinterpret_cast<const u32x2*>(cbase + cidx(unit, c, rb) * 2);
      const u32x2 x = CPOL ? __builtin_nontemporal_load(q) : *q;
      return f16x4_to_f32(x[0], x[1]);
    } else {
      const f32x4* q = reinterpret_cast<const f32x4*>(cbase + cidx(unit, c, rb) * 4);
      return CPOL ? __builtin_nontemporal_load(q) : *q;
    }
  };
  const auto cstore = [&](int unit, int c, int rb, f32x4 v) {
    if constexpr (CE == 2) {
      u32x2* q = reinterpret_cast<u32x2*>(cbase + cidx(unit, c, rb) * 2);
      const u32x2 x = {f16x2_sat(v[0], v[1]), f16x2_sat(v[2], v[3])};
      if (CPOL) __builtin_nontemporal_store(x, q);
      else *q = x;
    } else {
      f32x4* q = reinterpret_cast<f32x4*>(cbase + cidx(unit, c, rb) * 4);
      if (CPOL) __builtin_nontemporal_store(v, q);
      else *q = v;
    }
  };
  const uint4* pk = p.pk;

  // embedding / head constants of this lane's columns (each lane writes and
  // later reads only its own LDS entries, so no barrier is needed)
  __shared__ uint4 s_win[EMB_LDS ? CB * 64 : 1], s_wout[EMB_LDS ? CB * 64 : 1];
  __shared__ f32x4 s_pb[PB_LDS ? CB * 64 : 1];
  __shared__ __attribute__((aligned(16))) float s_lf[EMB_LDS ? 2 * D : 4];
  constexpr int KE = KEEP_EMB ? CBW : 1, KP = (KEEP_EMB || (EMB_LDS && !PB_LDS)) ? CBW : 1;
  uint4 win[KE], wout[KE];
  f32x4 pb[KP][KP > 1 ? RB : 1];
  f32x4 lfg[KE], lfb[KE];
  // b_in + P_act of this lane's row and columns
  const auto row_bias = [&](int c, int rb) {
    const int col = (w * CBW + c) * 16 + lq * 4;
    return *reinterpret_cast<const f32x4*>(raw + p.b_in + col) +
           *reinterpret_cast<const f32x4*>(raw + p.P_act + (size_t)((rb * 16 + lc) % HZ) * D + col);
  };
  if constexpr (KEEP_EMB || EMB_LDS) {
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
      const int col = (w * CBW + c) * 16 + lq * 4, fi = (w * CBW + c) * 64 + lane;
      const uint4 wi = pk[p.pk_win + (size_t)fi], wo = pk[p.pk_wout + (size_t)fi];
      f32x4 pv[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) pv[rb] = row_bias(c, rb);
      const f32x4 g_ = *reinterpret_cast<const f32x4*>(raw + p.lnf_g + col);
      const f32x4 b_ = *reinterpret_cast<const f32x4*>(raw + p.lnf_b + col);
      if constexpr (EMB_LDS) {
        s_win[fi] = wi;
        s_wout[fi] = wo;
        if constexpr (PB_LDS) s_pb[fi] = pv[0];
        else pb[c][0] = pv[0];
        *reinterpret_cast<f32x4*>(s_lf + col) = g_;
        *reinterpret_cast<f32x4*>(s_lf + D + col) = b_;
      } else {
        win[c] = wi;
        wout[c] = wo;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) pb[c][rb] = pv[rb];
        lfg[c] = g_;
        lfb[c] = b_;
      }
    }
  }
  // head bias of this lane's actions (zero beyond A)
  f32x4 bout;
#pragma unroll
  for (int i = 0; i < 4; ++i) bout[i] = 4 * lq + i < A ? raw[p.b_out + 4 * lq + i] : 0.f;

  // residual stream, and the running sum of a layer-merged cache's residuals
  f32x4 h[CBW][RB], mac[CBW][RB];
#pragma unroll
  for (int c = 0; c < CBW; ++c)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) mac[c][rb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // LayerNorm gain/shift and output bias of the next unit to evaluate, for
  // this lane's columns.  Width 256: loaded one unit ahead, and every
  // prefetch is issued unconditionally (a merge of an in-flight load with an
  // older register value costs a wait for the load at the merge).  Width 768
  // has no registers for that: gain and shift are requested with the unit's
  // first weights, the bias before the residual is summed.
  constexpr bool AHEAD = D <= 256;
  f32x4 nlg[CBW], nlb[CBW], nrb[AHEAD ? CBW : 1];
  // four consecutive small parameters of the layers, at float offset off (a
  // scalar) from layer 0 plus the lane group's four columns
  const auto prs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(raw + p.raw_layers), (short)0, L * C::PLAYER * 4,
                                                     0x00020000);
  const auto lparam = [&](int off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(prs, lq * 16, off * 4, 0));
  };
  const auto load_unit_params = [&](int unit) {
    const int ul = unit / 3, uu = unit - 3 * ul, base = ul * C::PLAYER + w * CBW * 16;
    const int go = base + (uu == 0 ? C::pLN1 : (uu == 1 ? C::pLN2 : C::pLN3));
    const int ro = base + (uu == 0 ? C::pBO : (uu == 1 ? C::pBO2 : C::pB2));
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
      nlg[c] = lparam(go + c * 16);
      nlb[c] = lparam(go + D + c * 16);
      if constexpr (AHEAD) nrb[c] = lparam(ro + c * 16);
    }
  };
  // reuse-cache loads: a batch takes the NB lowest units of a mask
  const auto seg_mask = [](int lo, int hi) {
    const uint64_t lo_m = (lo >= 64) ? ~0ull : ((1ull << lo) - 1);
    const uint64_t hi_m = (hi >= 64) ? ~0ull : ((1ull << hi) - 1);
    return hi_m & ~lo_m;
  };
  uint64_t mru_cur[SPT];
  // The loads of a batch are issued unconditionally (an entry that is not
  // needed reads past the end of a buffer resource, which returns zeros
  // without a memory access), so that they are all in flight before the
  // first is consumed.
  const auto crs = __builtin_amdgcn_make_buffer_rsrc(cbase, (short)0, U * (R * D) * CE, 0x00020000);
  const auto issue_batch = [&](uint64_t& um, auto& ub, auto& v) {
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      ub[q] = um ? __builtin_ctzll(um) : -1;
      um = um ? (um & (um - 1)) : 0ull;
    }
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int c = 0; c < CBW; ++c)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          uint64_t mj = mru_cur[0];
#pragma unroll
          for (int jj = 1; jj < SPT; ++jj)
            if (jrow[rb] == jj) mj = mru_cur[jj];
          const bool use = ub[q] >= 0 && ((mj >> ub[q]) & 1ull);
          const int off = use ? (ub[q] * (R * D) + (w * RB * CBW * 64 + lane) * 4) * CE : 0x7FFFFFF0;
          const int cst = (rb * CBW + c) * 256 * CE;
          if constexpr (CE == 2) {
            const auto x = __builtin_amdgcn_raw_buffer_load_b64(crs, off, cst, CPOL);
            v[q][c][rb] = f16x4_to_f32(x[0], x[1]);
          } else {
            v[q][c][rb] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(crs, off, cst, CPOL));
          }
        }
  };

  constexpr int MPWQ = C::m1(0), MPWC = C::m1(1), MPWF = C::m1(2), GF = C::g1(2);
  // self-attention: one wave per SIMD (the score tile's MFMAs fill the
  // matrix unit, and waves that share a block repeat them)
  constexpr int WPS = attn_waves_per_pair(NW < 4 ? NW : 4, HG * RB, DH / 16);
  constexpr int WPP = attn_waves_per_pair(NW, HG * RB, DH / 16);  // cross-attention
  constexpr int P = C::ring_size(), K1 = C::K1;
  static_assert(C::total(0) % P == 0 && C::total(2) % P == 0 && C::total(1) >= P, "ring");

  // ---- weight streams (see Cfg)
  const auto wrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(pk + p.pk_layers), (short)0, L * C::LAYER, 0x00020000);
  const auto wload = [&](int soff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16, soff, 0));
  };
  // a group's sequence: the runtime parts of its two stages' offsets
  struct Seq {
    int b1, b2;
  };
  const auto seq_of = [&](auto ty, int ul, int g) {
    constexpr int TY = decltype(ty)::value;
    return Seq{ul * C::LAYER + C::wave1(TY, w, g), ul * C::LAYER + C::wave2(TY, w, g)};
  };
  const auto elem = [&](auto ty, const Seq& s, int i) {
    constexpr int TY = decltype(ty)::value;
    return wload((i < C::s1(TY) ? s.b1 : s.b2) + C::elem(TY, i));
  };
  // first P elements of a unit's first sequence, requested before its LayerNorm
  const auto fill = [&](auto ty, uint4 (&ring)[P], const Seq& s) {
#pragma unroll
    for (int i = 0; i < P; ++i) ring[i] = elem(ty, s, i);
  };
  // element i of sequence s has been multiplied: its slot takes element i +
  // P, or one of the unit's next sequence nx (its last one ends with s again:
  // loaded, never used)
  const auto refill = [&](auto ty, uint4 (&ring)[P], const Seq& s, const Seq& nx, bool more, int i) {
    constexpr int TY = decltype(ty)::value;
    const int j = i + P;
    if (j < C::total(TY)) ring[i % P] = elem(ty, s, j);
    else if (j >= C::padded(TY) && more) ring[i % P] = elem(ty, nx, j - C::padded(TY));
  };
  // stage 1, column blocks grp * G .. + G: acc[m] = (A W^T)^T over d
  const auto stage1 = [&](auto ty, uint4 (&ring)[P], auto& acc, int grp, const Seq& s, const Seq& nx, bool more) {
    constexpr int TY = decltype(ty)::value, G = C::g1(TY);
#pragma unroll
    for (int m = 0; m < G; ++m)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[m][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint4 a[2][RB];
    const auto aload = [&](int k) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        a[k & 1][rb] = *reinterpret_cast<const uint4*>(xa + (rb * 16 + lc) * LDA + k * O::KF + lq * O::VE);
    };
    if constexpr (KAHEAD) aload(0);
#pragma unroll
    for (int k = 0; k < K1; ++k) {
      if constexpr (KAHEAD) {
        if (k + 1 < K1) aload(k + 1);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        aload(k);
      }
#pragma unroll
      for (int m = 0; m < G; ++m) {
        const int i = (grp * K1 + k) * G + m;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) O::mma(acc[m][rb], ring[i % P], a[k & 1][rb]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < G; ++m) refill(ty, ring, s, nx, more, (grp * K1 + k) * G + m);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // stage 2: acc[c] += this wave's column blocks over the group's columns
  const auto stage2 = [&](auto ty, uint4 (&ring)[P], auto& acc, const AT* z, const Seq& s, const Seq& nx, bool more) {
    constexpr int TY = decltype(ty)::value;
    uint4 a[2][RB];
    const auto aload = [&](int k) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
        a[k & 1][rb] = *reinterpret_cast<const uint4*>(z + (rb * 16 + lc) * LDZ + k * O::KF + lq * O::VE);
    };
    if constexpr (KAHEAD) aload(0);
#pragma unroll
    for (int k = 0; k < C::k2(TY); ++k) {
      if constexpr (KAHEAD) {
        if (k + 1 < C::k2(TY)) aload(k + 1);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        aload(k);
      }
#pragma unroll
      for (int c = 0; c < CBW; ++c) {
        const int i = C::s1(TY) + k * CBW + c;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) O::mma(acc[c][rb], ring[i % P], a[k & 1][rb]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < CBW; ++c) refill(ty, ring, s, nx, more, C::s1(TY) + k * CBW + c);
      __builtin_amdgcn_sched_barrier(0);
    }
    // slots that the padded sequence leaves unused take the next one's too
#pragma unroll
    for (int i = C::total(TY); i < C::padded(TY); ++i) refill(ty, ring, s, nx, more, i);
  };

  for (int t = 0; t < T; ++t) {
    asm volatile("" : "+v"(lane), "+v"(lc), "+v"(lq));
    const int k = T - 1 - t;
    // schedule of this step for every sample slot
    uint64_t mev[SPT], mru[SPT], mst[SPT];
    bool mmg[SPT];
    uint64_t evT = 0, ruT = 0;
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
      const bool live = ssmp[j] >= 0;
      const uint64_t e0 = live ? uniform64(msk[(j * T + t) * 3 + 0]) : 0ull;
      mmg[j] = (e0 & kMergedBit) != 0;
      mev[j] = e0 & ~kMergedBit;
      mru[j] = live ? uniform64(msk[(j * T + t) * 3 + 1]) : 0ull;
      mst[j] = live ? uniform64(msk[(j * T + t) * 3 + 2]) : 0ull;
      evT |= mev[j];
      ruT |= mru[j];
      mru_cur[j] = mru[j];
    }

    const auto pick = [&](const uint64_t (&m)[SPT], int j) {
      uint64_t v = m[0];
#pragma unroll
      for (int jj = 1; jj < SPT; ++jj)
        if (j == jj) v = m[jj];
      return v;
    };
    // noise added by this step's update (prefetched; always loaded from an
    // existing slice and action: the last step adds none, and a dead slot's
    // rows, which read sample 0's noise, are never output)
    f32x4 zpre[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int row = rb * 16 + lc, s = row_sample(rb);
      const int tn = t + 1 < T ? t + 1 : T - 1;
      const float* zp = p.noise + (((size_t)tn * p.batch + (s >= 0 ? s : 0)) * HZ + (row % HZ)) * A;
#pragma unroll
      for (int i = 0; i < 4; ++i) zpre[rb][i] = zp[4 * lq + i < A ? 4 * lq + i : 0];
    }
    // parameters of this step's first evaluated unit (unit 0 if none)
    if constexpr (AHEAD) load_unit_params(evT ? __builtin_ctzll(evT) : 0);
    // sampler constants of this step's update (prefetched)
    // (a lane-indexed vector load: a uniform scalar load would be waited for
    // by the next LDS access)
    const float ddl = p.ddpm[(size_t)k * 8 + (lane & 7)];
    // ---- embedding of the current sample on fp32 MFMA: h = (b_in + P_act) + x W_in^T
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
      uint4 wv;
      if constexpr (EMB_LDS) wv = s_win[(w * CBW + c) * 64 + lane];
      else if constexpr (KEEP_EMB) wv = win[c];
      else wv = pk[p.pk_win + (size_t)(w * CBW + c) * 64 + lane];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        f32x4 acc;
        if constexpr (PB_LDS) acc = s_pb[(w * CBW + c) * 64 + lane];
        else if constexpr (KEEP_EMB || EMB_LDS) acc = pb[c][rb];
        else acc = row_bias(c, rb);
        OF::mma(acc, wv, __builtin_bit_cast(uint4, xv[rb]));
        h[c][rb] = acc;
      }
    }

    // ---- the cacheable units (Eq. 1)
    int b = 0;
    while (true) {
      const uint64_t rest = evT >> b;
      const int e = rest ? b + __builtin_ctzll(rest) : U;
      // reused residuals of the units in [b, e), in unit order, loaded in
      // batches of NB units
      {
        uint64_t um = ruT & seg_mask(b, e);
        while (um) {
          int ub[NB];
          f32x4 v[NB][CBW][RB];
          issue_batch(um, ub, v);
#pragma unroll
          for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int c = 0; c < CBW; ++c)
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) h[c][rb] += v[q][c][rb];
        }
      }
      if (e >= U) break;

      // ---- evaluate unit e for the tile
      asm volatile("" : "+v"(lane), "+v"(lc), "+v"(lq));
      const int l = e / 3, u = e - 3 * l;
      const int lp = l * C::PLAYER;
      f32x4 lg[CBW], lb[CBW], rbias[CBW];
      if constexpr (AHEAD) {
#pragma unroll
        for (int c = 0; c < CBW; ++c) {
          lg[c] = nlg[c];
          lb[c] = nlb[c];
          rbias[c] = nrb[c];
        }
        // request the parameters of the step's next evaluated unit now, so
        // that they have the whole unit to arrive (this unit's own again when
        // no later unit is evaluated: the next step loads its first)
        const uint64_t later = (e + 1 < 64) ? (evT >> (e + 1)) : 0ull;
        load_unit_params(later ? e + 1 + __builtin_ctzll(later) : e);
      }
      f32x4 r[CBW][RB];
#pragma unroll
      for (int c = 0; c < CBW; ++c)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) r[c][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
      // LayerNorm of the unit's input into the stage-1 operand buffer
      const auto layer_norm_to_xa = [&]() {
        if constexpr (!AHEAD) {
          load_unit_params(e);
#pragma unroll
          for (int c = 0; c < CBW; ++c) {
            lg[c] = nlg[c];
            lb[c] = nlb[c];
          }
        }
        float mu[RB], rs[RB];
        ln_stats<C>(h, red, mu, rs, w, lc, lq);
#pragma unroll
        for (int c = 0; c < CBW; ++c)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            O::store4(xa, LDA, rb * 16 + lc, (w * CBW + c) * 16 + lq * 4, (h[c][rb] - mu[rb]) * rs[rb] * lg[c] + lb[c]);
        __syncthreads();
      };

      if (u == 0) {
        // ---------------- self-attention unit (causal over the action tokens)
        const std::integral_constant<int, 0> ty;
        uint4 ring[P];
        fill(ty, ring, seq_of(ty, l, member));
        layer_norm_to_xa();
        for (int g = member; g < NH / HG; g += TEAM) {
          asm volatile("" : "+v"(lane), "+v"(lc), "+v"(lq));
          constexpr bool more = NH / HG > TEAM;
          const Seq s = seq_of(ty, l, g), nx = seq_of(ty, l, g + TEAM < NH / HG ? g + TEAM : g);
          f32x4 y[MPWQ][RB];
          f32x4 bq[MPWQ];  // stage-1 biases, requested before the GEMM so their latency is hidden
#pragma unroll
          for (int m = 0; m < MPWQ; ++m)
            bq[m] = lparam(lp + C::pBQKV + ((NW * m) / (GW / 16) * CB + (NW * m) % (GW / 16) + g * (GW / 16) + w) * 16);
          stage1(ty, ring, y, 0, s, nx, more);
#pragma unroll
          for (int m = 0; m < MPWQ; ++m)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              *reinterpret_cast<f32x4*>(ybuf + (rb * 16 + lc) * LDY + (w + NW * m) * 16 + lq * 4) = y[m][rb] + bq[m];
          __syncthreads();
          // scores, softmax and values on fp32 MFMA tiles: WPS waves per
          // (head, query block), each with DH / 16 / WPS value column blocks.
          // The lane's scores of its query against keys 4 lq .. + 3 are the
          // second operand of the value product as they stand (step i takes
          // key 4 lq + i of every lane group).
          for (int it = w; it < HG * RB * WPS; it += NW) {
            const int pr = it / WPS, part = it % WPS;
            const int hh = pr % HG, ib = pr / HG;
            const int jb0 = (HZ >= 16) ? ((ib * 16) / HZ) * (HZ / 16) : ib;
            const int gi = ib * 16 + lc;  // query row
            f32x4 s[NJB];
            float m = -INFINITY;
#pragma unroll
            for (int jj = 0; jj < NJB; ++jj) {
              s[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
              const int jb = jb0 + jj;
              if (jb <= ib)
                s[jj] = qk_tile<DH>(ybuf + (ib * 16 + lc) * LDY + hh * DH, ybuf + (jb * 16 + lc) * LDY + GW + hh * DH, lq);
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const int gj = jb * 16 + lq * 4 + i;
                const bool ok = (gj <= gi) && (gj / HZ == gi / HZ);
                s[jj][i] = ok ? s[jj][i] * (kScale * kLog2e) : -INFINITY;
                m = fmaxf(m, s[jj][i]);
              }
            }
            m = quad_rows_max(m);
            float su = 0.f;
#pragma unroll
            for (int jj = 0; jj < NJB; ++jj)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const float ev = (s[jj][i] == -INFINITY) ? 0.f : fast_exp2(s[jj][i] - m);
                s[jj][i] = ev;
                su += ev;
              }
            const float inv = fast_rcp(quad_rows_sum(su));
#pragma unroll
            for (int jj = 0; jj < NJB; ++jj) s[jj] *= inv;
#pragma unroll
            for (int cbi = 0; cbi < DH / 16 / WPS; ++cbi) {
              const int cb = part * (DH / 16 / WPS) + cbi;
              f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int jj = 0; jj < NJB; ++jj) {
                const int jb = jb0 + jj;
                if (jb <= ib) {
#pragma unroll
                  for (int i = 0; i < 4; ++i) {
                    const float v = ybuf[(jb * 16 + 4 * lq + i) * LDY + 2 * GW + hh * DH + cb * 16 + lc];
                    o = mfma4(v, s[jj][i], o);
                  }
                }
              }
              O::store4(zbuf, LDZ, ib * 16 + lc, hh * DH + cb * 16 + lq * 4, o);
            }
          }
          __syncthreads();
          stage2(ty, ring, r, zbuf, s, nx, more);
        }
      } else if (C::FOLD && fold && u == 1) {
        if constexpr (C::FOLD) {
          // ---------------- cross-attention unit, folded (time token + observation tokens)
          // Score columns n = j * NH + h (memory token j, head h) of the row
          // block's sample, padded to 16 with zero columns.  Every team
          // member evaluates the whole unit (no partials to exchange).
          constexpr int KPW = (D / O::KF) / NW, VQ = O::VE / 4;
          static_assert(KPW * NW == D / O::KF && NH == 4, "folded cross-attention split");
          const float* trec = p.tfold + ((size_t)k * L + l) * REC;
          // record of memory token j of the sample in row block rb, and
          // whether it exists (else the time-token record stands in)
          const auto rec = [&](int rb, int j, bool& ok) -> const float* {
            const int s_ = row_sample(rb);
            ok = s_ >= 0 && j < S;
            return (ok && j > 0) ? okv + (((size_t)s_ * L + l) * nobs + (j - 1)) * REC : trec;
          };
          // u columns of this wave's k-range (lane: column lc, memory token
          // lc / NH of head lc % NH; columns of tokens that do not exist read
          // the time token's record and are masked in the softmax)
          f32x4 ub[RB][KPW][VQ];
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            bool ok;
            const float* q = rec(rb, lc / NH, ok) + (lc % NH) * D + w * KPW * O::KF + lq * O::VE;
#pragma unroll
            for (int kf = 0; kf < KPW; ++kf)
#pragma unroll
              for (int v = 0; v < VQ; ++v) ub[rb][kf][v] = *reinterpret_cast<const f32x4*>(q + kf * O::KF + 4 * v);
          }
          // c terms of memory token lq (heads 0 .. 3) and its w vectors at
          // this wave's columns (the first operand of the output product)
          f32x4 cq[RB];
          bool cok[RB];
          f32x4 wv[RB][CBW];
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            const float* q = rec(rb, lq, cok[rb]) + NH * D;
            cq[rb] = *reinterpret_cast<const f32x4*>(q + NH * D);
#pragma unroll
            for (int c = 0; c < CBW; ++c)
#pragma unroll
              for (int i = 0; i < 4; ++i) wv[rb][c][i] = q[i * D + (w * CBW + c) * 16 + lc];
          }
          layer_norm_to_xa();
          // partial scores over this wave's k-range on MFMA (lane: row lc,
          // columns 4 lq .. + 3, i.e. memory token lq of the four heads)
          float* const sb = ybuf;  // [RB][NW][64 lanes][4]
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kf = 0; kf < KPW; ++kf) {
              const uint4 a =
                  *reinterpret_cast<const uint4*>(xa + (rb * 16 + lc) * LDA + (w * KPW + kf) * O::KF + lq * O::VE);
              uint4 bq;
              if constexpr (sizeof(AT) == 2) {
                const f32x4 x0 = ub[rb][kf][0], x1 = ub[rb][kf][1];
                bq.x = bf16x2_rne(x0[0], x0[1]);
                bq.y = bf16x2_rne(x0[2], x0[3]);
                bq.z = bf16x2_rne(x1[0], x1[1]);
                bq.w = bf16x2_rne(x1[2], x1[3]);
              } else {
                bq = __builtin_bit_cast(uint4, ub[rb][kf][0]);
              }
              O::mma(acc, bq, a);
            }
            *reinterpret_cast<f32x4*>(sb + ((rb * NW + w) * 64 + lane) * 4) = acc;
          }
          __syncthreads();
          // every wave sums the partials, takes the softmax over the memory
          // tokens (lane groups lq) of each head and forms its own columns of
          // the output, r = P W over the 16 columns
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) a += *reinterpret_cast<const f32x4*>(sb + ((rb * NW + ww) * 64 + lane) * 4);
            f32x4 pr;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float sc = lq < S ? (a[i] + (cok[rb] ? cq[rb][i] : 0.f)) * (kScale * kLog2e) : -INFINITY;
              const float mx = quad_rows_max(sc);  // (all lanes take part in the swaps)
              const float ev = lq < S ? fast_exp2(sc - mx) : 0.f;
              pr[i] = ev * fast_rcp(quad_rows_sum(ev));
            }
#pragma unroll
            for (int c = 0; c < CBW; ++c)
#pragma unroll
              for (int i = 0; i < 4; ++i) r[c][rb] = mfma4(wv[rb][c][i], pr[i], r[c][rb]);
          }
        }
      } else if (u == 1) {
        // ---------------- cross-attention unit (time token + observation tokens)
        const std::integral_constant<int, 1> ty;
        uint4 ring[P];
        fill(ty, ring, seq_of(ty, l, member));
        // memory keys/values of a head group: time token + observation tokens
        constexpr int KVN = SPT * SMAX * 2 * GW, KVQ = (KVN + NT - 1) / NT;
        float kvv[KVQ];
        bool kvok[KVQ];
        // branch-free: every lane loads (entries outside the memory tokens
        // read the time-token row and are zeroed), so the loads issue back
        // to back instead of one guarded branch each
        const auto load_kv = [&](int g) {
          const float* trow = p.tkv + ((size_t)k * L + l) * (2 * D);
#pragma unroll
          for (int q = 0; q < KVQ; ++q) {
            const int it = tid + q * NT;
            const int col = it % (2 * GW), sm_ = (it / (2 * GW)) % SMAX, j = it / (2 * GW * SMAX);
            const int gcol = col < GW ? g * GW + col : D + g * GW + (col - GW);
            const int s_ = smp[j < SPT ? j : 0];
            const bool ok = it < KVN && sm_ < S && s_ >= 0;
            const bool obs_tok = ok && sm_ > 0;
            // 32-bit offsets: the observation K/V of a member is below 2^31 floats
            const int off = obs_tok ? ((s_ * L + l) * nobs + (sm_ - 1)) * (2 * D) + gcol : gcol;
            const float* src = &(obs_tok ? okv : trow)[off];
            kvv[q] = CPOL ? __builtin_nontemporal_load(src) : *src;  // read once per evaluation
            kvok[q] = ok;
          }
        };
        load_kv(member);
        layer_norm_to_xa();
        for (int g = member; g < NH / HG; g += TEAM) {
          asm volatile("" : "+v"(lane), "+v"(lc), "+v"(lq));
          if (g != member) load_kv(g);
          constexpr bool more = NH / HG > TEAM;
          const Seq s = seq_of(ty, l, g), nx = seq_of(ty, l, g + TEAM < NH / HG ? g + TEAM : g);
          f32x4 y[MPWC][RB];
          f32x4 bq[MPWC];
#pragma unroll
          for (int m = 0; m < MPWC; ++m)
            bq[m] = lparam(lp + C::pBQ + (g * (GW / 16) + w + NW * m) * 16);
          stage1(ty, ring, y, 0, s, nx, more);
#pragma unroll
          for (int m = 0; m < MPWC; ++m)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              *reinterpret_cast<f32x4*>(ybuf + (rb * 16 + lc) * LDY + (w + NW * m) * 16 + lq * 4) = y[m][rb] + bq[m];
#pragma unroll
          for (int q = 0; q < KVQ; ++q)
            if (tid + q * NT < KVN) kvbuf[tid + q * NT] = kvok[q] ? kvv[q] : 0.f;
          __syncthreads();
          // Each row attends to the S = 1 + n_obs memory tokens of its own
          // sample: few keys, so the products run on the vector ALUs (fp32
          // MFMA tiles would be mostly padding).  Lane = (row, quarter of the
          // head's dims); a row's four lanes are adjacent, so the score
          // reduction is two quad shuffles.  WPP waves per (head, row block)
          // each produce DH / WPP output dims.
          for (int it = w; it < HG * RB * WPP; it += NW) {
            const int pr = it / WPP, part = it % WPP;
            const int hh = pr % HG, ib = pr / HG;
            const int qr = lane >> 2, qg = lane & 3;  // row in the block, dim quarter
            const int row = ib * 16 + qr, js = row / HZ;
            constexpr int DQ = DH / 4, OD = DH / 4 / WPP;
            const float* qrow = ybuf + row * LDY + hh * DH + qg * DQ;
            const int c0 = hh * DH + part * (DH / WPP) + qg * OD;  // first output column of this lane
            // one pass over the keys with a running maximum (online softmax)
            float mx = -INFINITY, den = 0.f, o[OD];
#pragma unroll
            for (int d = 0; d < OD; ++d) o[d] = 0.f;
#pragma unroll 1
            for (int j = 0; j < S; ++j) {
              const float* kr = kvbuf + (js * SMAX + j) * (2 * GW) + hh * DH + qg * DQ;
              float a = 0.f;
#pragma unroll
              for (int d4 = 0; d4 < DQ / 4; ++d4) {
                const f32x4 kv = *reinterpret_cast<const f32x4*>(kr + 4 * d4);
                const f32x4 qv = *reinterpret_cast<const f32x4*>(qrow + 4 * d4);
                a += qv[0] * kv[0] + qv[1] * kv[1] + qv[2] * kv[2] + qv[3] * kv[3];
              }
              a += dpp_mov<0xB1>(a);  // sum over the row's four lanes
              a += dpp_mov<0x4E>(a);
              a *= kScale * kLog2e;
              const float mn = fmaxf(mx, a);
              const float sc = fast_exp2(mx - mn), pj = fast_exp2(a - mn);
              den = den * sc + pj;
              mx = mn;
              const float* vr = kvbuf + (js * SMAX + j) * (2 * GW) + GW + c0;
#pragma unroll
              for (int d4 = 0; d4 < OD / 4; ++d4) {
                const f32x4 vv = *reinterpret_cast<const f32x4*>(vr + 4 * d4);
#pragma unroll
                for (int e = 0; e < 4; ++e) o[4 * d4 + e] = o[4 * d4 + e] * sc + pj * vv[e];
              }
            }
            const float inv = fast_rcp(den);
#pragma unroll
            for (int d = 0; d < OD; d += 4)
              O::store4(zbuf, LDZ, row, c0 + d, f32x4{o[d] * inv, o[d + 1] * inv, o[d + 2] * inv, o[d + 3] * inv});
          }
          __syncthreads();
          stage2(ty, ring, r, zbuf, s, nx, more);
        }
      } else {
        // ---------------- feed-forward unit, d_ff streamed in chunks of FC
        const std::integral_constant<int, 2> ty;
        uint4 ring[P];
        fill(ty, ring, seq_of(ty, l, member));
        layer_norm_to_xa();
        for (int ch = member; ch < DFF / FC; ch += TEAM) {
          asm volatile("" : "+v"(lane), "+v"(lc), "+v"(lq));
          constexpr bool more = DFF / FC > TEAM;
          const Seq s = seq_of(ty, l, ch), nx = seq_of(ty, l, ch + TEAM < DFF / FC ? ch + TEAM : ch);
          AT* const zb = zbuf + (ZB2 ? (((ch - member) / TEAM) & 1) * (R * LDZ) : 0);
          // biases of a pair of column blocks, requested one pair ahead
          const auto bias = [&](int m) { return lparam(lp + C::pB1 + ch * FC + (w + NW * m) * 16); };
          f32x4 bn[GF];
#pragma unroll
          for (int m = 0; m < GF; ++m) bn[m] = bias(m);
#pragma unroll
          for (int grp = 0; grp < MPWF / GF; ++grp) {
            f32x4 y[GF][RB], b1v[GF];
#pragma unroll
            for (int m = 0; m < GF; ++m) {
              b1v[m] = bn[m];
              if (grp + 1 < MPWF / GF) bn[m] = bias((grp + 1) * GF + m);
            }
            stage1(ty, ring, y, grp, s, nx, more);
#pragma unroll
            for (int m = 0; m < GF; ++m)
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) {
                f32x4 v = y[m][rb] + b1v[m];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = gelu_erf(v[i]);
                O::store4(zb, LDZ, rb * 16 + lc, (w + NW * (grp * GF + m)) * 16 + lq * 4, v);
              }
          }
          __syncthreads();
          stage2(ty, ring, r, zb, s, nx, more);
          // (with one buffer, the next chunk's GELU outputs wait for every
          // wave's reads of this one)
          if constexpr (!ZB2 && DFF / FC > TEAM) __syncthreads();
        }
      }
      if constexpr (!AHEAD) {  // requested here, added after the exchange
        const int ro = lp + w * CBW * 16 + (u == 0 ? C::pBO : (u == 1 ? C::pBO2 : C::pB2));
#pragma unroll
        for (int c = 0; c < CBW; ++c) rbias[c] = lparam(ro + c * 16);
      }
      if constexpr (TEAM > 1) if (!(fold && u == 1)) {
        // Sum the members' partial residuals in member order, so that every
        // member obtains the same bits.  The partials travel through memory
        // with device-coherent (SC1) buffer stores and loads, which leave no
        // stale or dirty lines in the per-XCD caches (the weight stream stays
        // in L2).  Each thread waits only for the words it sums: a word is
        // ready once it no longer holds the sentinel.  Waits are bounded;
        // on a timeout the device error flag is set and every later wait
        // ends at once, so the kernel always finishes.
        const int cur = nbar % XS, prev = (nbar + 2) % XS;  // prev: the last unit's slot, or with four the one before
        const u32x4 empty = {kEmpty, kEmpty, kEmpty, kEmpty};
        const auto empty_prev = [&]() {
#pragma unroll
          for (int c = 0; c < CBW; ++c)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              xstore(empty, prev, SCATTER && c / OWN == member ? TEAM : member, c, rb);
        };
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the last emptying stores (this slot's among them, or sooner) have landed
        // (a word equal to the sentinel becomes the canonical NaN)
        const auto canonical = [&](f32x4 x) {
          u32x4 v = __builtin_bit_cast(u32x4, x);
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = v[q] == kEmpty ? 0x7FC00000u : v[q];
          return v;
        };
#pragma unroll
        for (int c = 0; c < CBW; ++c)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            const u32x4 v = canonical(r[c][rb]);
            if (!(p.withhold && member == 0) && !(SCATTER && c / OWN == member))
              xstore(v, cur, member, c, rb);
          }
        // (this member holds all sums of the last unit, so every member has
        // read everything of the one before)
        if constexpr (SCATTER) empty_prev();
        // bounded wait for every word of `v` (loaded by `load`) to be written;
        // polls back to back (each is a memory round trip), the error flag
        // and the limit are checked every 32 polls.  Width 256: the wave polls
        // until every lane's words are there (one scalar branch; Push-T batch
        // 1 and 64 with bf16 operands 3.37 and 3.39 ms, with lanes leaving one
        // by one 3.40 and 3.42); width 768 the reverse (batch 1 and 128 24.6
        // and 36.6 ms, against 24.1 and 36.1).
        const auto arrived = [](bool ok) { return D > 256 ? ok : __builtin_amdgcn_ballot_w64(!ok) == 0; };
        const auto poll = [&](auto& v, auto load, auto ready) {
          unsigned spins = 0;
          while (true) {
            load(v);
            if (arrived(ready(v))) break;
            if ((++spins & 31u) == 0u &&
                (__hip_atomic_load(p.derr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u || spins > p.spin_limit)) {
              __hip_atomic_store(p.derr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              break;
            }
          }
        };
        const auto full = [&](const u32x4& x) {
          return x[0] != kEmpty && x[1] != kEmpty && x[2] != kEmpty && x[3] != kEmpty;
        };
        if constexpr (TEAM == 2) {
          // two operands: r + other is the same sum on both members
          // (commutative), so only the other member's partial is held, a few
          // column blocks at a time
          constexpr int XC = (CBW * RB > 4) ? (4 / RB > 0 ? 4 / RB : 1) : CBW;
          static_assert(CBW % XC == 0, "exchange chunks");
          const int other = 1 - member;
#pragma unroll
          for (int c0 = 0; c0 < CBW; c0 += XC) {
            u32x4 part[XC][RB];
            poll(part,
                 [&](u32x4 (&v)[XC][RB]) {
#pragma unroll
                   for (int c = 0; c < XC; ++c)
#pragma unroll
                     for (int rb = 0; rb < RB; ++rb)
                       v[c][rb] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff(cur, other), xcst(c0 + c, rb), kCoherent);
                 },
                 [&](const u32x4 (&v)[XC][RB]) {
                   bool ok = true;
#pragma unroll
                   for (int c = 0; c < XC; ++c)
#pragma unroll
                     for (int rb = 0; rb < RB; ++rb) ok = ok && full(v[c][rb]);
                   return ok;
                 });
#pragma unroll
            for (int c = 0; c < XC; ++c)
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) r[c0 + c][rb] += __builtin_bit_cast(f32x4, part[c][rb]);
          }
        } else if constexpr (SCATTER) {
          // this member's column blocks: its own partial from registers, the
          // others' from their slots, summed in member order
          f32x4 own[OWN][RB];
#pragma unroll
          for (int c = 0; c < CBW; ++c)
            if (c / OWN == member) {
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) own[c % OWN][rb] = r[c][rb];
            }
          u32x4 part[TEAM][OWN][RB];
          unsigned pending = ((1u << TEAM) - 1u) & ~(1u << member);
          poll(part,
               [&](u32x4 (&v)[TEAM][OWN][RB]) {
#pragma unroll
                 for (int m = 0; m < TEAM; ++m)
                   if (pending >> m & 1u) {
#pragma unroll
                     for (int c = 0; c < OWN; ++c)
#pragma unroll
                       for (int rb = 0; rb < RB; ++rb)
                         v[m][c][rb] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff(cur, m), xcst(member * OWN + c, rb), kCoherent);
                   }
               },
               [&](const u32x4 (&v)[TEAM][OWN][RB]) {
#pragma unroll
                 for (int m = 0; m < TEAM; ++m)
                   if (pending >> m & 1u) {
                     bool ok = true;
#pragma unroll
                     for (int c = 0; c < OWN; ++c)
#pragma unroll
                       for (int rb = 0; rb < RB; ++rb) ok = ok && full(v[m][c][rb]);
                     if (arrived(ok)) pending &= ~(1u << m);
                   }
                 return pending == 0u;
               });
#pragma unroll
          for (int c = 0; c < OWN; ++c)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
              f32x4 acc = member == 0 ? own[c][rb] : __builtin_bit_cast(f32x4, part[0][c][rb]);
#pragma unroll
              for (int m = 1; m < TEAM; ++m)
                acc += member == m ? own[c][rb] : __builtin_bit_cast(f32x4, part[m][c][rb]);
              xstore(canonical(acc), cur, TEAM, member * OWN + c, rb);
            }
          // every member's sums (its own too)
          u32x4 sum[CBW][RB];
          poll(sum,
               [&](u32x4 (&v)[CBW][RB]) {
#pragma unroll
                 for (int c = 0; c < CBW; ++c)
#pragma unroll
                   for (int rb = 0; rb < RB; ++rb)
                     v[c][rb] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff(cur, TEAM), xcst(c, rb), kCoherent);
               },
               [&](const u32x4 (&v)[CBW][RB]) {
                 bool ok = true;
#pragma unroll
                 for (int c = 0; c < CBW; ++c)
#pragma unroll
                   for (int rb = 0; rb < RB; ++rb) ok = ok && full(v[c][rb]);
                 return ok;
               });
#pragma unroll
          for (int c = 0; c < CBW; ++c)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) r[c][rb] = __builtin_bit_cast(f32x4, sum[c][rb]);
        } else {
          // more operands: every member sums the partials in member order
          u32x4 part[TEAM][CBW][RB];
          unsigned pending = ((1u << TEAM) - 1u) & ~(1u << member);
          poll(part,
               [&](u32x4 (&v)[TEAM][CBW][RB]) {
#pragma unroll
                 for (int m = 0; m < TEAM; ++m)
                   if (pending >> m & 1u) {
#pragma unroll
                     for (int c = 0; c < CBW; ++c)
#pragma unroll
                       for (int rb = 0; rb < RB; ++rb)
                         v[m][c][rb] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff(cur, m), xcst(c, rb), kCoherent);
                   }
               },
               [&](const u32x4 (&v)[TEAM][CBW][RB]) {
#pragma unroll
                 for (int m = 0; m < TEAM; ++m)
                   if (pending >> m & 1u) {
                     bool ok = true;
#pragma unroll
                     for (int c = 0; c < CBW; ++c)
#pragma unroll
                       for (int rb = 0; rb < RB; ++rb) ok = ok && full(v[m][c][rb]);
                     if (arrived(ok)) pending &= ~(1u << m);
                   }
                 return pending == 0u;
               });
#pragma unroll
          for (int c = 0; c < CBW; ++c)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
              f32x4 acc = member == 0 ? r[c][rb] : __builtin_bit_cast(f32x4, part[0][c][rb]);
#pragma unroll
              for (int m = 1; m < TEAM; ++m)
                acc += member == m ? r[c][rb] : __builtin_bit_cast(f32x4, part[m][c][rb]);
              r[c][rb] = acc;
            }
        }
        // every member has read the partials of the previous unit: empty this
        // member's slot of it for its next use
        if constexpr (!SCATTER) empty_prev();
        ++nbar;
      }
#pragma unroll
      for (int c = 0; c < CBW; ++c)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) r[c][rb] += rbias[c];

      // Eq. 1 per sample at unit e: evaluated residual (and cache refresh) or
      // the residual cached at the unit's most recent refresh.
#pragma unroll
      for (int c = 0; c < CBW; ++c)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const int j = jrow[rb];
          const uint64_t bit = 1ull << e;
          bool mg = mmg[0];
#pragma unroll
          for (int jj = 1; jj < SPT; ++jj)
            if (j == jj) mg = mmg[jj];
          if (pick(mev, j) & bit) {
            const f32x4 v = r[c][rb];
            if (mg) mac[c][rb] = (u == 0) ? v : mac[c][rb] + v;
            if (pick(mst, j) & bit) cstore(e, c, rb, mg ? mac[c][rb] : v);
            h[c][rb] += v;
            if (p.acts != nullptr && member == 0) {
              // activation record of the uncached policy (Sec. 3.3): a[sample][unit][step][H][d]
              *reinterpret_cast<f32x4_dword*>(p.acts + (((size_t)smp[j] * U + e) * T + t) * (HZ * D) +
                                        (size_t)((rb * 16 + lc) % HZ) * D + (w * CBW + c) * 16 + lq * 4) = v;
            }
          } else if (pick(mru, j) & bit) {
            h[c][rb] += cload(e, c, rb);
          }
        }
      b = e + 1;
    }

    // ---- head (final LayerNorm + linear on fp32 MFMA) and DDPM update
    {
      float mu[RB], rs[RB];
      ln_stats<C>(h, red, mu, rs, w, lc, lq);
      f32x4 eacc[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) eacc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < CBW; ++c) {
        f32x4 g_, b_;
        const int col = (w * CBW + c) * 16 + lq * 4;
        if constexpr (EMB_LDS) {
          g_ = *reinterpret_cast<const f32x4*>(s_lf + col);
          b_ = *reinterpret_cast<const f32x4*>(s_lf + D + col);
        } else if constexpr (KEEP_EMB) {
          g_ = lfg[c];
          b_ = lfb[c];
        } else {
          g_ = *reinterpret_cast<const f32x4*>(raw + p.lnf_g + col);
          b_ = *reinterpret_cast<const f32x4*>(raw + p.lnf_b + col);
        }
        uint4 wo;
        if constexpr (EMB_LDS) wo = s_wout[(w * CBW + c) * 64 + lane];
        else if constexpr (KEEP_EMB) wo = wout[c];
        else wo = pk[p.pk_wout + (size_t)(w * CBW + c) * 64 + lane];
        // the normalised columns are the second operand as they stand
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          OF::mma(eacc[rb], wo, __builtin_bit_cast(uint4, (h[c][rb] - mu[rb]) * rs[rb] * g_ + b_));
      }
      // partial noise estimates of the waves' columns, summed by every wave
      // for the actions its lanes keep
      float* epsp = ybuf;  // [RB][NW][64 lanes][4]
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) *reinterpret_cast<f32x4*>(epsp + ((rb * NW + w) * 64 + lane) * 4) = eacc[rb];
      __syncthreads();
      const auto dd = [&](int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ddl), i)); };
      const float s1 = dd(0), rsa = dd(1), c0 = dd(2), ct = dd(3), sg = dd(4);
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        f32x4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) part += *reinterpret_cast<const f32x4*>(epsp + ((rb * NW + ww) * 64 + lane) * 4);
        const int row = rb * 16 + lc, s = row_sample(rb);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float e = bout[i] + part[i], x = xv[rb][i];
          float x0 = (x - s1 * e) * rsa;
          if (p.clip) x0 = fminf(fmaxf(x0, -1.f), 1.f);
          float xn = c0 * x0 + ct * x;
          if (k > 0) xn += sg * zpre[rb][i];
          const int a = 4 * lq + i;
          xv[rb][i] = a < A ? xn : 0.f;
          if (t == T - 1 && w == 0 && a < A && s >= 0 && member == 0)
            p.out[((size_t)s * HZ + (row % HZ)) * A + a] = xn;
        }
      }
    }
  }
}

// ---------------------------------------------------------------- observation pre-pass
// Folded cross-attention: observation tokens, their keys/values and fold
// records, computed once per query before the denoising launch.  Workgroup
// (g, l) takes the 16 (sample, token) rows g*16 .. g*16+15 of the flattened
// [batch][n_obs] tokens and layer l; the tokens' embedding (a product with
// the observation matrix) is repeated by every layer's workgroup.
template <class AT>
__global__ void __launch_bounds__(512) obs_fold_kernel(const KParams p) {
  using O = Op<AT>;
  constexpr int D = 256, DH = 64, NW = 8, NT = NW * 64, CB = D / 16, REC = 2 * (D / DH) * D + 16;
  constexpr int KOBS = 64, LDO = KOBS + O::PAD, LDA = D + O::PAD;
  __shared__ __attribute__((aligned(16))) AT ob[16 * LDO];
  __shared__ __attribute__((aligned(16))) AT xa[16 * LDA];
  __shared__ __attribute__((aligned(16))) float kvr[16 * 2 * D];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, lc = lane & 15, lq = lane >> 4;
  const int nobs = p.n_obs, L = p.L, l = blockIdx.y;
  const int row0 = blockIdx.x * 16, nrows = min(16, p.batch * nobs - row0);
  const float* raw = p.raw;
  constexpr int MPWO = CB / NW;
  f32x4 acc[MPWO][1];
#pragma unroll
  for (int m = 0; m < MPWO; ++m) acc[m][0] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nch = p.obs_pad / KOBS;
  for (int c = 0; c < nch; ++c) {
    __syncthreads();
    for (int it = tid; it < 16 * KOBS; it += NT) {
      const int row = it / KOBS, k = it % KOBS, kk = c * KOBS + k;
      const float v = (row < nrows && kk < p.obs_dim) ? p.obs[(size_t)(row0 + row) * p.obs_dim + kk] : 0.f;
      O::store(ob, LDO, row, k, v);
    }
    __syncthreads();
    gemm_acc<AT, 1, MPWO, KOBS / O::KF>(acc, ob, LDO, p.pk + p.pk_obs, p.obs_pad / O::KF, c * (KOBS / O::KF),
                                         [&](int m) { return w + NW * m; }, lane);
  }
#pragma unroll
  for (int m = 0; m < MPWO; ++m) {
    const int gcol = (w + NW * m) * 16 + lq * 4, o = (row0 + lc) % nobs;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (lc < nrows)
      v = acc[m][0] + *reinterpret_cast<const f32x4*>(raw + p.b_obs + gcol) +
          *reinterpret_cast<const f32x4*>(raw + p.P_mem + (size_t)(1 + o) * D + gcol);
    O::store4(xa, LDA, lc, gcol, v);
  }
  __syncthreads();
  const LayerOff lo = p.loff[l];
  constexpr int MPWK = 2 * CB / NW;
  f32x4 kv[MPWK][1];
#pragma unroll
  for (int m = 0; m < MPWK; ++m) kv[m][0] = f32x4{0.f, 0.f, 0.f, 0.f};
  gemm_acc<AT, 1, MPWK, D / O::KF>(kv, xa, LDA, p.pk + lo.pk_kv, D / O::KF, 0,
                                    [&](int m) { return w + NW * m; }, lane);
#pragma unroll
  for (int m = 0; m < MPWK; ++m) {
    const int gcol = (w + NW * m) * 16 + lq * 4;
    *reinterpret_cast<f32x4*>(kvr + lc * (2 * D) + gcol) = kv[m][0] + *reinterpret_cast<const f32x4*>(raw + lo.b_kv + gcol);
  }
  __syncthreads();
  fold_rows<D, DH, NT, 16, sizeof(AT) == 2>(
      raw, lo.w_q, lo.w_o2t, lo.b_q, kvr, 2 * D, nrows,
      [&](int row) -> float* {
        const int tok = row0 + row, s = tok / nobs, o = tok % nobs;
        return p.okv + (((size_t)s * L + l) * nobs + o) * REC;
      },
      tid);
}

hipError_t launch_obs_fold(const KParams& p, int dtype, hipStream_t stream) {
  const int rows = p.batch * p.n_obs;
  if (rows <= 0) return hipSuccess;
  const dim3 grid((unsigned)((rows + 15) / 16), (unsigned)p.L);
  if (dtype == 1) hipLaunchKernelGGL(obs_fold_kernel<__bf16>, grid, dim3(512), 0, stream, p);
  else hipLaunchKernelGGL(obs_fold_kernel<float>, grid, dim3(512), 0, stream, p);
  return hipGetLastError();
}
// ---------------------------------------------------------------- creation
__global__ void pack_kernel(const float* __restrict__ raw, size_t off, int N, int Nvalid, int K, int Kpad, int bf,
                            uint4* __restrict__ dst) {
  const int KF = bf ? 32 : 16;
  const int KBT = Kpad / KF;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t nfrag = (size_t)(N / 16) * KBT;
  if (gid >= nfrag * 64) return;
  const int lane = (int)(gid % 64);
  const size_t fr = gid / 64;
  const int kb = (int)(fr % KBT), nb = (int)(fr / KBT);
  const int n = nb * 16 + (lane & 15), q = lane >> 4;
  uint32_t e[4] = {0u, 0u, 0u, 0u};
  if (n < Nvalid) {
    const float* W = raw + off + (size_t)n * K;
    if (bf) {
      for (int i = 0; i < 4; ++i) {
        const int k0 = kb * 32 + q * 8 + 2 * i;
        const uint32_t lo = k0 < K ? bf16_rne(W[k0]) : 0u;
        const uint32_t hi = k0 + 1 < K ? bf16_rne(W[k0 + 1]) : 0u;
        e[i] = lo | (hi << 16);
      }
    } else {
      for (int j = 0; j < 4; ++j) {
        const int kk = kb * 16 + 4 * q + j;
        e[j] = kk < K ? __float_as_uint(W[kk]) : 0u;
      }
    }
  }
  dst[gid] = make_uint4(e[0], e[1], e[2], e[3]);
}

// memory row 0 of every timestep: sinusoid(k) + P_mem[0], fp64 -> fp32
__global__ void time_row_kernel(const float* __restrict__ raw, uint32_t pmem0, int T, int D,
                                float* __restrict__ rows) {
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= T * D) return;
  const int k = gid / D, j = gid % D, half = D / 2;
  const int jj = j < half ? j : j - half;
  const double om = exp(-log(10000.0) * (double)jj / (double)(half - 1));
  const double a = (double)k * om;
  const double v = (j < half ? sin(a) : cos(a)) + (double)raw[pmem0 + j];
  rows[gid] = (float)v;
}

// keys/values of the time token for every (timestep, layer)
__global__ void time_kv_kernel(const float* __restrict__ raw, const float* __restrict__ rows,
                               const uint32_t* __restrict__ wkv, const uint32_t* __restrict__ bkv, int T,
                               int L, int D, int bf, float* __restrict__ tkv) {
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (size_t)T * L * 2 * D) return;
  const int col = (int)(gid % (2 * D));
  const int l = (int)((gid / (2 * D)) % L);
  const int k = (int)(gid / ((size_t)2 * D * L));
  const float* W = raw + wkv[l] + (size_t)col * D;
  const float* m = rows + (size_t)k * D;
  float acc = 0.f;
  for (int j = 0; j < D; ++j) {
    const float wv = bf ? __uint_as_float(bf16_rne(W[j]) << 16) : W[j];
    acc = fmaf(m[j], wv, acc);
  }
  tkv[gid] = acc + raw[bkv[l] + col];
}

// DDPM constants (squared-cosine betas, fixed-small variance), fp64 -> fp32:
// per timestep i: sqrt(1-abar), sqrt(abar), c0, ct, sigma.
__global__ void ddpm_kernel(int T, float* tab) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  const double s = 0.008, half_pi = 1.5707963267948966;
  double abar = 1.0;
  for (int i = 0; i < T; ++i) {
    double f0 = cos(((double)i / T + s) / (1.0 + s) * half_pi);
    double f1 = cos(((double)(i + 1) / T + s) / (1.0 + s) * half_pi);
    f0 *= f0;
    f1 *= f1;
    const double beta = fmin(1.0 - f1 / f0, 0.999);
    const double alpha = 1.0 - beta;
    const double abar_prev = abar;
    abar *= alpha;
    const double c0 = sqrt(abar_prev) * beta / (1.0 - abar);
    const double ct = sqrt(alpha) * (1.0 - abar_prev) / (1.0 - abar);
    const double var = fmax((1.0 - abar_prev) / (1.0 - abar) * beta, 1e-20);
    float* r = tab + (size_t)i * 8;
    r[0] = (float)sqrt(1.0 - abar);
    r[1] = (float)(1.0 / sqrt(abar));  // stored as a reciprocal: the update multiplies
    r[2] = (float)c0;
    r[3] = (float)ct;
    r[4] = (float)sqrt(var);
    r[5] = r[6] = r[7] = 0.f;
  }
}

// fold records of the time token: one workgroup per (timestep, layer)
template <bool BF>
__global__ void __launch_bounds__(512) time_fold_kernel(const float* __restrict__ raw, const LayerOff* __restrict__ loff,
                                                        const float* __restrict__ tkv, int L, float* __restrict__ tfold) {
  constexpr int D = 256, DH = 64, REC = 2 * (D / DH) * D + 16;
  __shared__ __attribute__((aligned(16))) float kv[2 * D];
  const int kl = blockIdx.x, l = kl % L;
  for (int i = threadIdx.x; i < 2 * D; i += 512) kv[i] = tkv[(size_t)kl * 2 * D + i];
  __syncthreads();
  const LayerOff q = loff[l];
  fold_rows<D, DH, 512, 1, BF>(raw, q.w_q, q.w_o2t, q.b_q, kv, 2 * D, 1,
                            [&](int) -> float* { return tfold + (size_t)kl * REC; }, (int)threadIdx.x);
}

hipError_t launch_time_fold(const float* raw, const LayerOff* loff, const float* tkv, int T, int L, int d, int dh,
                            int dtype, float* tfold, hipStream_t stream) {
  if (d != 256 || dh != 64) return hipErrorInvalidValue;
  if (dtype == 1)
    hipLaunchKernelGGL(time_fold_kernel<true>, dim3(T * L), dim3(512), 0, stream, raw, loff, tkv, L, tfold);
  else
    hipLaunchKernelGGL(time_fold_kernel<false>, dim3(T * L), dim3(512), 0, stream, raw, loff, tkv, L, tfold);
  return hipGetLastError();
}

hipError_t launch_pack(const float* raw, size_t off, int N, int Nvalid, int K, int Kpad, int dtype, uint4* dst,
                       hipStream_t stream) {
  const int KF = dtype == 1 ? 32 : 16;
  const size_t n = (size_t)(N / 16) * (Kpad / KF) * 64;
  const int bs = 256;
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0, stream, raw, off, N, Nvalid,
                     K, Kpad, dtype == 1 ? 1 : 0, dst);
  return hipGetLastError();
}

hipError_t launch_time_kv(const float* raw, uint32_t pmem0, const uint32_t* wkv, const uint32_t* bkv, int T, int L,
                          int D, int dtype, float* rows_scratch, float* tkv, hipStream_t stream) {
  const int bs = 256;
  hipLaunchKernelGGL(time_row_kernel, dim3((T * D + bs - 1) / bs), dim3(bs), 0, stream, raw, pmem0, T, D,
                     rows_scratch);
  const size_t n = (size_t)T * L * 2 * D;
  hipLaunchKernelGGL(time_kv_kernel, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), 0, stream, raw,
                     rows_scratch, wkv, bkv, T, L, D, dtype == 1 ? 1 : 0, tkv);
  return hipGetLastError();
}

__global__ void zero_u32_kernel(unsigned* dst, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = 0u;
}

hipError_t launch_zero_u32(unsigned* dst, int n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_u32_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, dst, n);
  return hipGetLastError();
}

hipError_t launch_ddpm_table(int T, float* table, hipStream_t stream) {
  hipLaunchKernelGGL(ddpm_kernel, dim3(1), dim3(1), 0, stream, T, table);
  return hipGetLastError();
}

// ---------------------------------------------------------------- dispatch
#define EVO_SHAPES(X)                                     \
  X(float, 64, 32, 8, 2, 256, 4, 2, 256, 8, 1)            \
  X(__bf16, 64, 32, 8, 2, 256, 4, 2, 256, 8, 1)           \
  X(float, 256, 64, 16, 1, 1024, 8, 4, 256, 8, 1)         \
  X(float, 256, 64, 16, 2, 1024, 8, 2, 128, 8, 1)         \
  X(__bf16, 256, 64, 16, 1, 1024, 8, 4, 1024, 8, 1)       \
  X(__bf16, 256, 64, 16, 2, 1024, 8, 2, 256, 8, 1)        \
  X(__bf16, 768, 64, 32, 1, 3072, 8, 2, 256, 5, 1)        \
  X(float, 256, 64, 16, 1, 1024, 4, 1, 256, 8, 4)         \
  X(__bf16, 256, 64, 16, 1, 1024, 4, 1, 256, 8, 4)        \
  X(float, 256, 64, 16, 1, 1024, 8, 2, 256, 8, 2)         \
  X(__bf16, 256, 64, 16, 1, 1024, 8, 2, 512, 8, 2)        \
  X(__bf16, 768, 64, 32, 1, 3072, 8, 2, 256, 5, 2)        \
  X(__bf16, 768, 64, 32, 1, 3072, 8, 2, 512, 5, 6)

template <class AT> constexpr int dtype_of() { return std::is_same<AT, float>::value ? 0 : 1; }

#define EVO_MATCH(AT, D, DH, HZ, SPT, DFF, TEAM)                                                          \
  (key.d == D && key.dh == DH && key.horizon == HZ && key.d_ff == DFF && key.dtype == dtype_of<AT>() && \
   key.spt == SPT && key.team == TEAM)

bool kernel_available(const KernelKey& key, int* threads) {
#define X(AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM) \
  if (EVO_MATCH(AT, D, DH, HZ, SPT, DFF, TEAM)) {          \
    if (threads) *threads = NW * 64;                       \
    return true;                                           \
  }
  EVO_SHAPES(X)
#undef X
  return false;
}

bool kernel_layer_layout(const KernelKey& key, LayerLayout* out) {
#define X(AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM)                                                        \
  if (EVO_MATCH(AT, D, DH, HZ, SPT, DFF, TEAM)) {                                                                 \
    using C = Cfg<AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM>;                                               \
    *out = LayerLayout{{C::pLN1, C::pLN1 + D, C::pBQKV, C::pBO, C::pLN2, C::pLN2 + D, C::pBQ, C::pBO2, C::pLN3,   \
                        C::pLN3 + D, C::pB1, C::pB2},                                                             \
                       C::PLAYER,                                                                                 \
                       {C::off1(0), C::off2(0), C::off1(1), C::off2(1), C::off1(2), C::off2(2)},                  \
                       C::LAYER};                                                                                 \
    return true;                                                                                                  \
  }
  EVO_SHAPES(X)
#undef X
  return false;
}

int kernel_max_obs_tokens_for(const KernelKey& key) {
#define X(AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM) \
  if (EVO_MATCH(AT, D, DH, HZ, SPT, DFF, TEAM)) return (SMAX - 1) < 16 / SPT ? (SMAX - 1) : 16 / SPT;
  EVO_SHAPES(X)
#undef X
  return 0;
}

int kernel_max_action_dim() { return 16; }

int kernel_team_sizes(const KernelKey& key, int out[4]) {
  int n = 0;
#define X(AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM) \
  if (TEAM > 1 && n < 4 && key.d == D && key.dh == DH && key.horizon == HZ && key.d_ff == DFF &&      \
      key.dtype == dtype_of<AT>() && key.spt == SPT)                                                   \
    out[n++] = TEAM;
  EVO_SHAPES(X)
#undef X
  std::sort(out, out + n, [](int a, int b) { return a > b; });
  return n;
}

int kernel_max_steps_x_spt() { return kMaskEntries; }

hipError_t launch_denoise(const KernelKey& key, const KParams& p, hipStream_t stream) {
#define X(AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM)                                                   \
  if (EVO_MATCH(AT, D, DH, HZ, SPT, DFF, TEAM)) {                                                          \
    const void* fn = reinterpret_cast<const void*>(&denoise_kernel<AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM>); \
    if (TEAM == 1) {                                                                                       \
      hipLaunchKernelGGL((denoise_kernel<AT, D, DH, HZ, SPT, DFF, NW, HG, FC, SMAX, TEAM>), dim3(p.n_tiles), \
                         dim3(NW * 64), 0, stream, p);                                                     \
      return hipGetLastError();                                                                            \
    }                                                                                                      \
    /* team members wait for each other: all workgroups must be resident */                                \
    KParams pc = p;                                                                                        \
    void* args[] = {&pc};                                                                                  \
    return hipLaunchCooperativeKernel(fn, dim3(p.n_tiles * TEAM), dim3(NW * 64), args, 0, stream);         \
  }
  EVO_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace evo
