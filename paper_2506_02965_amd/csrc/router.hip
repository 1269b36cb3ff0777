// Gating (Alg. 7: scores, softmax, TopKIndices, w = p[I]) and its adjoint on the data owner.
//
// Scores are accumulated in fp64 (MFMA or FMA) from the products of the stored inputs (exact in fp64) and rounded once to
// fp32. The order of a score's sum follows the tiling, which goes by the batch size and the device's CU count: equal
// calls give equal bits, and where fp64 holds the sum exactly (bf16 inputs, as long as no product is smaller than about
// 2^-37 of the sum) so do other batches; else a score can differ in its last fp32 bit, in about one of 10^8, and a
// selection that hangs on that bit with it. Selection happens at wavefront level: k rounds of a 64-lane maximum over
// order-preserving keys, ties to the lowest expert index.
#include "pcmoe_internal.h"
#include <math.h>
#include <algorithm>

namespace pcmoe {

typedef double doublex4 __attribute__((ext_vector_type(4)));

// Wavefront maximum of unsigned keys on the vector ALU (DPP: row shifts, then row broadcasts), in every lane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define PCMOE_DPP_MAX(ctrl, rows) \
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false))
  PCMOE_DPP_MAX(0x111, 0xf);  // row_shr 1, 2, 4, 8: lane 15 of each row of 16 holds the row's maximum
  PCMOE_DPP_MAX(0x112, 0xf);
  PCMOE_DPP_MAX(0x114, 0xf);
  PCMOE_DPP_MAX(0x118, 0xf);
  PCMOE_DPP_MAX(0x142, 0xa);  // row_bcast 15 into rows 1 and 3, row_bcast 31 into rows 2 and 3
  PCMOE_DPP_MAX(0x143, 0xc);
#undef PCMOE_DPP_MAX
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Order-preserving key of a score: larger score, larger key; -0 and +0 share one; 0 (below every number's) for a
// NaN, which is never selected.
__device__ __forceinline__ uint32_t score_key(float f) {
  const uint32_t u = __float_as_uint(f);
  if (f != f) return 0u;
  if (f == 0.f) return 0x80000000u;
  return (u >> 31) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_score(uint32_t k) {
  return k == 0u ? -INFINITY : __uint_as_float((k >> 31) ? (k & 0x7fffffffu) : ~k);
}

// Scores of NTOK = TB * TT tokens against all E experts on the fp64 matrix cores, then top-k and gate weights.
// The WE x WK wavefronts split the experts into WE runs of 16 * NET and d into WK ranges of column steps (4 chunks
// each); the WK fp64 partial sums of a score are added in a fixed order, the bias is added in fp64 and the result is
// rounded once to fp32. Each lane feeds one 16-byte chunk of its token row and of its expert row (8 bf16 / 4 fp32
// consecutive k) into 8 / 4 MFMAs: MFMA s takes element s of every lane, so lane group q contributes
// k = 4*EPC*c + EPC*q + s (the same mapping on both operands).
//   TB = 16: v_mfma_f64_16x16x4f64, 16 tokens x 16 experts.
//   TB = 4:  v_mfma_f64_4x4x4_4b_f64, its four blocks one group of 4 tokens against 4 x 4 experts.
//   TB = 1:  one token on v_fma_f64; lane group q's partial sums are added across the groups at the end.
// All three do about 16 multiply-adds per cycle and SIMD (a 16 x 16 x 4 product takes 64 cycles, measured), and the
// vector ALU does not run beside an fp64 MFMA: the bound is the products and, at 8 cycles each, the conversions to
// fp64 (T = 16384, E = 64, d = 2048: 4.3 GFLOP, 56 us of products, 86 us measured, 108 before). A workgroup's
// products run on one CU, so a short batch takes workgroups of few tokens: 16 tokens x 64 experts x d = 2048 alone
// are 14 us of a CU's fp64 rate, whatever the token count. Long batches take TT token tiles per wavefront: an expert
// chunk is then converted once for TT products, a token chunk once for NET.
// PF column steps of loads are in flight per wavefront.
template <typename T, int TB, int TT, int NET, int WE, int WK, int PF>
__global__ __launch_bounds__(64 * WE * WK) void route_fwd_kernel(const T* __restrict__ x, const T* __restrict__ wr,
                                                              const float* __restrict__ bias, int bias_div, int Tn,
                                                              int d, int E, int k, int renorm,
                                                              float* __restrict__ logits, int32_t* __restrict__ idx,
                                                              float* __restrict__ gw) {
  constexpr int EP = EPC<T>::value;        // elements per 16-byte chunk
  constexpr int EW = 16 * NET * WE + 1;    // padded expert stride of the partial-sum table
  constexpr int NTOK = TB * TT;
  constexpr int W = WE * WK;
  extern __shared__ double part[];         // [WK][NTOK][EW]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int we = wave % WE, wk = wave / WE;
  const int i = lane & 15, q = lane >> 4;
  const int t0 = blockIdx.x * NTOK;
  const int e0 = we * 16 * NET;
  // Column steps [s0, s1) of this wavefront.
  const int steps = d / (4 * EP);
  const int s0 = (int)((long)steps * wk / WK), s1 = (int)((long)steps * (wk + 1) / WK);
  const T* xrow[TT];
  const T* wrow[NET];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    const int t = t0 + tt * TB + (TB == 16 ? i : TB == 4 ? (lane & 3) : 0);
    xrow[tt] = x + (size_t)(t < Tn ? t : Tn - 1) * d + EP * q;  // rows past the end: a valid row, never used
  }
#pragma unroll
  for (int et = 0; et < NET; ++et) {
    const int e = e0 + 16 * et + i;
    wrow[et] = wr + (size_t)(e < E ? e : E - 1) * d + EP * q;   // as above
  }
  typedef typename std::conditional<TB == 16, doublex4, double>::type Acc;
  // CH independent accumulator chains per product (column steps alternate between them), added in chain order
  // at the end: back-to-back MFMAs on one accumulator wait for each other.
  constexpr int CH = TT * NET >= 8 ? 1 : TT * NET >= 4 ? 2 : 4;
  Acc acc[CH][TT][NET];
#pragma unroll
  for (int ch = 0; ch < CH; ++ch)
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int et = 0; et < NET; ++et) {
        if constexpr (TB == 16) acc[ch][tt][et] = doublex4{0.0, 0.0, 0.0, 0.0};
        else acc[ch][tt][et] = 0.0;
      }
  Chunk xc[PF][TT], wc[PF][NET];
  auto load = [&](int st, Chunk (&xb)[TT], Chunk (&wb)[NET]) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) xb[tt] = ld_chunk(xrow[tt] + st * 4 * EP);
#pragma unroll
    for (int et = 0; et < NET; ++et) wb[et] = ld_chunk(wrow[et] + st * 4 * EP);
  };
  auto compute = [&](const Chunk (&xb)[TT], const Chunk (&wb)[NET]) {
    float xf[TT][EP], wf[NET][EP];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) chunk_to_f<T>(xb[tt], xf[tt]);
#pragma unroll
    for (int et = 0; et < NET; ++et) chunk_to_f<T>(wb[et], wf[et]);
#pragma unroll
    for (int s = 0; s < EP; ++s) {
      double xd[TT], wd[NET];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) xd[tt] = (double)xf[tt][s];
#pragma unroll
      for (int et = 0; et < NET; ++et) wd[et] = (double)wf[et][s];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int et = 0; et < NET; ++et) {
          Acc& a = acc[s % CH][tt][et];
          if constexpr (TB == 16) a = __builtin_amdgcn_mfma_f64_16x16x4f64(xd[tt], wd[et], a, 0, 0, 0);
          else if constexpr (TB == 4) a = __builtin_amdgcn_mfma_f64_4x4x4f64(wd[et], xd[tt], a, 0, 0, 0);
          else a = fma(xd[tt], wd[et], a);
        }
    }
  };
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (s0 + u < s1) load(s0 + u, xc[u], wc[u]);
  for (int st = s0; st < s1; st += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      if (st + u < s1) {
        compute(xc[u], wc[u]);
        if (st + u + PF < s1) load(st + u + PF, xc[u], wc[u]);
      }
    }
  }
  // 16x16x4: register r of lane group q holds D[token 4r + q][expert i]. 4x4x4: lane l holds token l & 3 and expert
  // 4 * ((l >> 2) & 3) + (l >> 4). One token: every lane group holds its own columns' sum for expert i.
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int et = 0; et < NET; ++et) {
      Acc a = acc[0][tt][et];
#pragma unroll
      for (int ch = 1; ch < CH; ++ch) a += acc[ch][tt][et];
      if constexpr (TB == 16) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          part[(wk * NTOK + tt * 16 + 4 * r + q) * EW + e0 + 16 * et + i] = a[r];
      } else if constexpr (TB == 4) {
        part[(wk * NTOK + tt * 4 + (lane & 3)) * EW + e0 + 16 * et + (lane & 12) + q] = a;
      } else {
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (q == 0) part[(wk * NTOK + tt) * EW + e0 + 16 * et + i] = a;
      }
    }
  __syncthreads();

  // Each wavefront finishes tokens wave, wave + W, ...: fixed-order sum of the WK partials, bias, one rounding, then
  // k rounds of the wavefront maximum over order-preserving keys (lowest expert index among equal scores).
  constexpr int QE = (16 * NET * WE + 63) / 64;  // experts per lane: lane, lane + 64, ...
  for (int row = wave; row < NTOK; row += W) {
    const int tt = t0 + row;
    if (tt >= Tn) break;
    uint32_t key[QE];
    float v[QE];
#pragma unroll
    for (int qq = 0; qq < QE; ++qq) {
      const int e = lane + 64 * qq;
      v[qq] = -INFINITY;
      key[qq] = 0u;
      if (e < E) {
        double sum = part[row * EW + e];
#pragma unroll
        for (int w = 1; w < WK; ++w) sum += part[(w * NTOK + row) * EW + e];
        if (bias) sum += (double)bias[(size_t)(tt / bias_div) * E + e];
        const float L = (float)sum;
        logits[(size_t)tt * E + e] = L;
        v[qq] = L;
        key[qq] = score_key(L);
      }
    }
    float myv = -INFINITY;
    int myi = 0;
    for (int j = 0; j < k; ++j) {
      uint32_t m = key[0];
#pragma unroll
      for (int qq = 1; qq < QE; ++qq) m = max(m, key[qq]);
      m = wave_max_u32(m);
      int best = 0x7fffffff;  // no selectable score is left (NaN scores only)
      if (m != 0u) {
#pragma unroll
        for (int qq = QE - 1; qq >= 0; --qq) {
          const uint64_t b = __ballot(key[qq] == m);
          if (b) best = 64 * qq + __builtin_ctzll(b);
        }
      }
#pragma unroll
      for (int qq = 0; qq < QE; ++qq)
        if (lane + 64 * qq == best) key[qq] = 0u;
      if (lane == j) {
        myv = key_score(m);
        myi = best;
      }
    }
    const float m = __shfl(myv, 0, 64);  // the largest score of the token
    const float ex = (lane < k) ? expf(myv - m) : 0.f;
    float zp = ex;
    if (!renorm) {
      zp = 0.f;
#pragma unroll
      for (int qq = 0; qq < QE; ++qq)
        if (lane + 64 * qq < E) zp += expf(v[qq] - m);
    }
    zp = wave_sum(zp);
    if (lane < k) {
      idx[(size_t)tt * k + lane] = myi;
      gw[(size_t)tt * k + lane] = ex / zp;
    }
  }
}

template <typename T, int TB, int TT, int NET, int WE, int WK, int PF>
static hipError_t route_fwd_run(const moe_desc& d, const void* x, const void* wr, const float* bias, int div,
                                float* logits, int32_t* idx, float* w, hipStream_t s) {
  constexpr int NTOK = TB * TT;
  constexpr size_t LDS = (size_t)WK * NTOK * (16 * NET * WE + 1) * sizeof(double);
  static_assert(LDS <= 160 * 1024, "partial-sum table");
  auto kern = route_fwd_kernel<T, TB, TT, NET, WE, WK, PF>;
  if (LDS > 65536) {
    static std::atomic<uint64_t> lds_set{0};
    if (hipError_t e = lds_limit_once((const void*)kern, (int)LDS, lds_set); e != hipSuccess) return e;
  }
  KernelTimer kt("route_fwd", s);
  hipLaunchKernelGGL(kern, dim3((d.T + NTOK - 1) / NTOK), dim3(64 * WE * WK), LDS, s, (const T*)x, (const T*)wr, bias,
                     div, d.T, d.d_model, d.n_experts, d.top_k, d.renormalize, logits, idx, w);
  return hipGetLastError();
}

template <typename T>
static hipError_t route_fwd_t(const moe_desc& d, const void* x, const void* wr, const float* bias, int bg,
                              float* logits, int32_t* idx, float* w, hipStream_t s) {
  const int E = d.n_experts;
  const int div = d.T / (bg > 0 ? bg : 1);
  // Tokens per workgroup: the fewest (1, 4, 16 or 32) whose workgroups are at most one per CU, since a workgroup costs
  // its padded tokens' products and a second round costs as much as the first. Measured on MI355X (d = 2048, E = 64;
  // us for 1 / 4 / 16 / 32 tokens): T = 24 12 / 14 / - / -, T = 300 22 / 15 / 26 / 43, T = 3000 - / 48 / 26 / 43,
  // T = 8192 - / - / 50 / 44; the 16-token workgroups of 4 wavefronts used before took 36, 37, 37 and 57.
  // Past one round of 32 tokens a full one costs 0.9 of two rounds of 16, but a last round that is nearly empty as much
  // as a full one: 32 tokens are taken while their rounds cost less (bf16, E = 64, d = 2048, us for 16 / 32 tokens:
  // T = 8300 68 / 80, 12,288 69 / 80, 16,384 88 / 82, 16,500 108 / 119, 24,576 128 / 121). With up to 32 bf16 experts
  // 16 tokens of 4 wavefronts are always the better past one round (E = 32, T = 16,384, d = 128: 12.1 / 15.3, T = 8300,
  // d = 2048: 36 / 47).
  // Wavefronts: as many as fit the LDS table and, at 16 of them, 128 VGPRs without spills; 4 to a workgroup of 16 tokens
  // in long batches, where several workgroups share a CU.
#define RT(TB, TT, NET, WE, WK, PF) \
  return route_fwd_run<T, TB, TT, NET, WE, WK, PF>(d, x, wr, bias, div, logits, idx, w, s)
  const int cus = device_cus();
  const int r16 = (d.T + 16 * cus - 1) / (16 * cus), r32 = (r16 + 1) / 2;  // rounds of 16 and of 32 tokens per CU
  const bool by32 = r32 == 1 || ((E > 32 || d.dtype == MOE_F32) && 20 * r32 <= 11 * r16);
  const int tok = d.T <= cus ? 1 : d.T <= 4 * cus ? 4 : r16 == 1 ? 16 : by32 ? 32 : 64;  // 64: 16, in a long batch
  if (E <= 16) {
    if (tok == 1) RT(1, 1, 1, 1, 16, 4);
    if (tok == 4) RT(4, 1, 1, 1, 16, 4);
    if (tok == 16) RT(16, 1, 1, 1, 16, 4);
    RT(16, 1, 1, 1, 8, 4);  // one expert tile: 32 tokens per workgroup measured slower (28 against 30 us at d = 4096)
  } else if (E <= 32) {
    if (tok == 1) RT(1, 1, 2, 1, 16, 4);
    if (tok == 4) RT(4, 1, 2, 1, 16, 4);
    if (tok == 16) RT(16, 1, 2, 1, 8, 3);
    if (tok == 32) RT(16, 2, 2, 1, 8, 2);
    RT(16, 1, 2, 1, 4, 4);
  } else if (E <= 64) {
    if (tok == 1) RT(1, 1, 4, 1, 16, 2);
    if (tok == 4) RT(4, 1, 4, 1, 16, 2);
    if (tok == 16) RT(16, 1, 4, 1, 8, 2);
    if (tok == 32) RT(16, 2, 4, 1, 8, 2);
    RT(16, 1, 4, 1, 4, 2);
  } else if (E <= 128) {
    if (tok == 1) RT(1, 1, 4, 2, 8, 2);
    if (tok == 4) RT(4, 1, 4, 2, 8, 2);
    if (tok == 32) RT(16, 2, 4, 2, 4, 2);
    RT(16, 1, 4, 2, 4, 2);
  } else {
    if (tok == 1) RT(1, 1, 4, 4, 4, 2);
    if (tok == 4) RT(4, 1, 4, 4, 4, 2);
    if (tok == 32) RT(16, 2, 4, 4, 2, 2);
    RT(16, 1, 4, 4, 2, 2);
  }
#undef RT
}

hipError_t launch_route_fwd(const moe_desc& d, const void* x, const void* wr, const float* bias, int bg,
                            float* logits, int32_t* idx, float* w, hipStream_t s) {
  if (d.dtype == MOE_BF16) return route_fwd_t<bf16>(d, x, wr, bias, bg, logits, idx, w, s);
  return route_fwd_t<float>(d, x, wr, bias, bg, logits, idx, w, s);
}

// ------------------------------------------------------------------------------ backward

// dscores per token (one wavefront per token).
__global__ __launch_bounds__(256) void route_dlogits_kernel(int Tn, int E, int k, int renorm,
                                                            const float* __restrict__ logits,
                                                            const int32_t* __restrict__ idx,
                                                            const float* __restrict__ gw,
                                                            const float* __restrict__ dgate,
                                                            float* __restrict__ dl) {
  const int lane = threadIdx.x & 63;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int nwaves = (gridDim.x * blockDim.x) >> 6;
  for (int t = wave; t < Tn; t += nwaves) {
    float wj = 0.f, gj = 0.f;
    int ij = -1;
    if (lane < k) {
      wj = gw[(size_t)t * k + lane];
      gj = dgate[(size_t)t * k + lane];
      ij = idx[(size_t)t * k + lane];
    }
    if (renorm) {
      const float sgw = wave_sum(wj * gj);
      for (int e0 = 0; e0 < E; e0 += 64) {
        int e = e0 + lane;
        float val = 0.f;
        for (int jj = 0; jj < k; ++jj) {
          int i2 = __shfl(ij, jj, 64);
          float w2 = __shfl(wj, jj, 64), g2 = __shfl(gj, jj, 64);
          if (e == i2) val = w2 * (g2 - sgw);
        }
        if (e < E) dl[(size_t)t * E + e] = val;
      }
    } else {
      // p over all E experts (up to 4 per lane); g = dgate scattered onto E
      constexpr int NQ = 4;  // E <= 256
      float p[NQ], g[NQ], M = -INFINITY, zp = 0.f, spg = 0.f;
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const int e = lane + 64 * n;
        p[n] = e < E ? logits[(size_t)t * E + e] : -INFINITY;
        M = fmaxf(M, p[n]);
      }
      M = wave_max(M);
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        p[n] = lane + 64 * n < E ? expf(p[n] - M) : 0.f;
        zp += p[n];
        g[n] = 0.f;
      }
      const float Z = wave_sum(zp);
      for (int jj = 0; jj < k; ++jj) {
        const int i2 = __builtin_amdgcn_readlane(ij, jj);
        const float g2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gj), jj));
#pragma unroll
        for (int n = 0; n < NQ; ++n)
          if (lane + 64 * n == i2) g[n] = g2;
      }
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        p[n] = p[n] / Z;
        spg += p[n] * g[n];
      }
      const float S = wave_sum(spg);
#pragma unroll
      for (int n = 0; n < NQ; ++n)
        if (lane + 64 * n < E) dl[(size_t)t * E + lane + 64 * n] = p[n] * (g[n] - S);
    }
  }
}

// Partial dW_router over one chunk of tokens, part[chunk][e][c] = sum_{t in chunk} dl[t][e] * x[t][c], as an
// fp32 MFMA contraction (v_mfma_f32_16x16x4f32, tokens as K). Lane (q, i) of a wavefront loads JJ contiguous
// columns c0 + JJ*i .. + JJ-1 of token rows t + q (one coalesced load of the row segment per 16 lanes) and
// feeds column c0 + JJ*i + jj of MFMA number jj; its A operand is dl[t + q][16 et + i]. 8 token-steps of 4
// tokens are loaded before their MFMAs.
template <typename T, int JJ>
struct alignas(JJ * sizeof(T) < 16 ? JJ * sizeof(T) : 16) XRow {  // tensors are 16-byte aligned
  T v[JJ];
};

// JJ columns per lane: 4 for up to 16 experts (narrower workgroups, so that 256 of them need only 64 token
// chunks of partial sums: measured 9 us against 12 us for 8 columns and 128 chunks at T=4096, d=1024), 8 up to 32.
// For more experts, fewer while the accumulators (JJ x NET tiles) fit.
constexpr int dw_cols_per_lane(int net) { return net == 1 ? 4 : net <= 2 ? 8 : 16 / net; }

template <typename T, int NET, int JJ>
__global__ __launch_bounds__(256) void route_dw_partial_kernel(int Tn, int d, int E, int tok_per_chunk,
                                                               const T* __restrict__ x,
                                                               const float* __restrict__ dl,
                                                               float* __restrict__ part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int q = lane >> 4, i = lane & 15;
  const int c0 = (blockIdx.x * 4 + wave) * 16 * JJ;  // first column of this wavefront
  if (c0 >= d) return;                               // d is a multiple of 16 * JJ: all or nothing
  const int chunk = blockIdx.y;
  const int tb = chunk * tok_per_chunk;
  const int te = min(Tn, tb + tok_per_chunk);
  floatx4 acc[JJ][NET];
#pragma unroll
  for (int jj = 0; jj < JJ; ++jj)
#pragma unroll
    for (int et = 0; et < NET; ++et) acc[jj][et] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int t0 = tb; t0 < te; t0 += 32) {
    XRow<T, JJ> xv[8];
    float a[8][NET];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int t = t0 + 4 * u + q;
      const bool ok = t < te;
      if (ok) xv[u] = *reinterpret_cast<const XRow<T, JJ>*>(x + (size_t)t * d + c0 + JJ * i);
      else xv[u] = XRow<T, JJ>{};
#pragma unroll
      for (int et = 0; et < NET; ++et) {
        const int e = 16 * et + i;
        a[u][et] = (ok && e < E) ? dl[(size_t)t * E + e] : 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int jj = 0; jj < JJ; ++jj) {
        const float b = to_f(xv[u].v[jj]);
#pragma unroll
        for (int et = 0; et < NET; ++et)
          acc[jj][et] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][et], b, acc[jj][et], 0, 0, 0);
      }
  }
  // register r of lane group q holds D[expert 16 et + 4q + r][n = i], column c0 + JJ*i + jj
#pragma unroll
  for (int et = 0; et < NET; ++et)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int e = 16 * et + 4 * q + r;
      if (e >= E) continue;
      float* o = part + ((size_t)chunk * E + e) * d + c0 + JJ * i;
#pragma unroll
      for (int jj = 0; jj < JJ; ++jj) o[jj] = acc[jj][et][r];
    }
}

// The same partial sums for more than 32 experts and many tokens. A wavefront holds 64 experts x 16 groups of N columns
// (16 bytes of x) and steps through its tokens 4 at a time with one 16-byte load of dl (lane (q, i): token t + q, experts
// 4 i .. 4 i + 3, one per MFMA row) and one of x (its columns of token t + q) per 4 N MFMAs, 16 tokens ahead of the MFMAs.
// Bound by the fp32 MFMAs. Bit for bit the sums of the narrow kernel. Both launches, narrow and wide: T = 8192, d = 2048,
// E = 256 181 and 96 us (56 us of MFMA at the peak rate); T = 16384, E = 64 78 and 62.
template <typename T, bool VEC>
__global__ __launch_bounds__(256, 2) void route_dw_wide_kernel(int Tn, int d, int E, int tok_per_chunk, int col_blocks,
                                                               const T* __restrict__ x, const float* __restrict__ dl,
                                                               float* __restrict__ part) {
  constexpr int N = EPC<T>::value, U = 4;
  const int lane = threadIdx.x & 63, q = lane >> 4, i = lane & 15;
  const int groups = (E + 63) >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  // a workgroup's wavefronts: the expert groups of one column block first (they read the same x)
  const int cb = wave / groups, eg = wave - cb * groups;
  if (cb >= col_blocks) return;
  const int c0 = (cb * 16 + i) * N, e0 = eg * 64 + 4 * i;
  const int tb = blockIdx.y * tok_per_chunk, te = min(Tn, tb + tok_per_chunk);
  floatx4 acc[N][4];
#pragma unroll
  for (int s = 0; s < N; ++s)
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[s][m] = floatx4{0.f, 0.f, 0.f, 0.f};
  struct Buf {
    Chunk x[U];
    float a[U][4];
  };
  // the chunk's rows of x and dl as buffers: tokens past its end read as zeros
  const auto xr = buf_rsrc(x + (size_t)tb * d, (size_t)(te - tb) * d * sizeof(T));
  const auto gr = buf_rsrc(dl + (size_t)tb * E, (size_t)(te - tb) * E * 4);
  int xo = (q * d + c0) * (int)sizeof(T), go = (q * E + e0) * 4;
  auto load = [&](Buf& b) {  // the next 4 U tokens
#pragma unroll
    for (int u = 0; u < U; ++u) {
      b.x[u] = buf_ld16(xr, xo);
      if (VEC) {
        const Chunk v = buf_ld16(gr, e0 < E ? go : kBufPast);
#pragma unroll
        for (int m = 0; m < 4; ++m) b.a[u][m] = __uint_as_float(v.w[m]);
      } else {
#pragma unroll
        for (int m = 0; m < 4; ++m)
          b.a[u][m] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(gr, e0 + m < E ? go + 4 * m : kBufPast, 0, 0));
      }
      xo += 4 * d * (int)sizeof(T);
      go += 16 * E;
    }
  };
  auto mul = [&](const Buf& b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xf[N];
      chunk_to_f<T>(b.x[u], xf);
#pragma unroll
      for (int s = 0; s < N; ++s)
#pragma unroll
        for (int m = 0; m < 4; ++m)
          acc[s][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(b.a[u][m], xf[s], acc[s][m], 0, 0, 0);
    }
  };
  Buf b0, b1;
  load(b0);
  for (int t0 = tb; t0 < te; t0 += 8 * U) {
    load(b1);
    __builtin_amdgcn_sched_barrier(0);
    mul(b0);
    __builtin_amdgcn_sched_barrier(0);
    load(b0);
    __builtin_amdgcn_sched_barrier(0);
    mul(b1);
    __builtin_amdgcn_sched_barrier(0);
  }
  // register r of lane (q, i), MFMA (s, m): expert 64 eg + 4 (4 q + r) + m, column c0 + s
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int e = eg * 64 + 4 * (4 * q + r) + m;
      if (e >= E) continue;
      float* o = part + ((size_t)blockIdx.y * E + e) * d + c0;
#pragma unroll
      for (int s = 0; s < N; s += 4)
        *reinterpret_cast<float4*>(o + s) = float4{acc[s][m][r], acc[s + 1][m][r], acc[s + 2][m][r], acc[s + 3][m][r]};
    }
}

// dW_router[o] = sum over chunks of part[chunk][o], in a fixed order: thread (g, o) of a workgroup sums
// the chunks g, g + 16, g + 32, ... in turn, then the 16 partial sums of an output are added in g order.
constexpr int RED_G = 16;  // chunk lanes per output
__global__ __launch_bounds__(256) void route_dw_reduce_kernel(int n4, int nchunks, const float4* __restrict__ part,
                                                              float4* __restrict__ out) {
  __shared__ float4 red[RED_G][256 / RED_G];
  const int g = threadIdx.x / (256 / RED_G), ol = threadIdx.x % (256 / RED_G);
  const int o = blockIdx.x * (256 / RED_G) + ol;
  float4 s = float4{0.f, 0.f, 0.f, 0.f};
  if (o < n4)
    for (int c = g; c < nchunks; c += RED_G) {
      const float4 v = part[(size_t)c * n4 + o];
      s.x += v.x;
      s.y += v.y;
      s.z += v.z;
      s.w += v.w;
    }
  red[g][ol] = s;
  __syncthreads();
  if (g == 0 && o < n4) {
    float4 t = red[0][ol];
    for (int h = 1; h < RED_G; ++h) {
      const float4 v = red[h][ol];
      t.x += v.x;
      t.y += v.y;
      t.z += v.z;
      t.w += v.w;
    }
    out[o] = t;
  }
}

// Column blocks of a wavefront's 16 chunks (route_dw_wide_kernel).
static int dw_wide_cols(const moe_desc& d) { return (int)(d.d_model * elem_bytes(d) / 256); }

static int dw_net(int E) { return E <= 16 ? 1 : E <= 32 ? 2 : E <= 64 ? 4 : E <= 128 ? 8 : 16; }

// Token chunks of the weight-gradient contraction, a multiple of 32 tokens each: as many as give the narrow kernel about
// 256 workgroups for up to 16 experts and 1024 above (4 wavefronts x 16 x JJ columns each). The chunk is the length of an
// fp32 accumulator and so sets the error of dW_router (T = 8192, d = 2048, E = 256: 3.0e-7 of its norm over 256 tokens,
// 4.1e-7 over 512): the wide kernel takes the same chunks, though it would fill the chip with fewer. Chunks of 32 tokens
// are too short for its loop body, which then runs once, from cold instruction caches; more than 64 experts, whose
// narrow kernel reads x several times, gain all the same once there are two of its wavefronts per SIMD (both launches,
// us for narrow / wide: E = 256, bf16, T = 4096, d = 512 47 / 39, T = 1000, d = 1024 26.6 / 28.3; E = 128, T = 4096,
// d = 1024 42.8 / 36.4, T = 2048, d = 512 24.1 / 25.5; E = 64, T = 2048, d = 2048 27.3 / 26.2, T = 3000, d = 1024
// 24.7 / 25.0; E = 33, T = 3000, d = 2048 25.8 / 28.8).
static void route_bwd_chunks(const moe_desc& d, int* nch, int* tpc, bool* wide) {
  const int E = d.n_experts;
  const int wg_cols = 64 * dw_cols_per_lane(dw_net(E));
  const int ncol = (d.d_model + wg_cols - 1) / wg_cols;
  const int maxch = (d.T + 31) / 32;
  const int want = ((E <= 16 ? 256 : 1024) + ncol - 1) / ncol;
  const int n = std::max(std::min(want, maxch), 1);
  const int per = ((d.T + n - 1) / n + 31) / 32 * 32;
  *tpc = per;
  *nch = (d.T + per - 1) / per;
  const int waves = dw_wide_cols(d) * ((E + 63) / 64) * *nch;  // of the wide kernel
  *wide = E > 32 && (per >= 64 || (E > 64 && waves >= 2048));
}

size_t route_bwd_ws_bytes(const moe_desc& d) {
  int nch, tpc;
  bool wide;
  route_bwd_chunks(d, &nch, &tpc, &wide);
  return align256((size_t)nch * d.n_experts * d.d_model * sizeof(float));
}

template <typename T>
static hipError_t route_bwd_t(const moe_desc& d, const void* x, const float* logits, const int32_t* idx,
                              const float* w, const float* dgate, float* dl, float* dwr, void* ws,
                              hipStream_t s) {
  const int E = d.n_experts;
  {
    KernelTimer kt("route_dlogits", s);
    int blocks = (d.T + 3) / 4;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(route_dlogits_kernel, dim3(blocks), dim3(256), 0, s, d.T, E, d.top_k, d.renormalize,
                       logits, idx, w, dgate, dl);
  }
  int nch, tpc;
  bool wide;
  route_bwd_chunks(d, &nch, &tpc, &wide);
  // one chunk (up to 32 tokens, or column blocks enough to fill the chip): its sums are the result, without the sum over
  // chunks and its launch (6 us)
  float* part = nch == 1 ? dwr : (float*)ws;
  {
    KernelTimer kt("route_dw_partial", s);
    if (wide) {
      const int cb = dw_wide_cols(d);
      const dim3 grid((cb * ((E + 63) / 64) + 3) / 4, nch);
      if (E % 4 == 0)
        hipLaunchKernelGGL((route_dw_wide_kernel<T, true>), grid, dim3(256), 0, s, d.T, d.d_model, E, tpc, cb,
                           (const T*)x, dl, part);
      else
        hipLaunchKernelGGL((route_dw_wide_kernel<T, false>), grid, dim3(256), 0, s, d.T, d.d_model, E, tpc, cb,
                           (const T*)x, dl, part);
    } else {
      const int wg_cols = 64 * dw_cols_per_lane(dw_net(E));
      const dim3 grid((d.d_model + wg_cols - 1) / wg_cols, nch);
#define RB_LAUNCH(NET)                                                                                       \
  hipLaunchKernelGGL((route_dw_partial_kernel<T, NET, dw_cols_per_lane(NET)>), grid, dim3(256), 0, s, d.T, \
                     d.d_model, E, tpc, (const T*)x, dl, part)
      if (E <= 16) RB_LAUNCH(1);
      else if (E <= 32) RB_LAUNCH(2);
      else if (E <= 64) RB_LAUNCH(4);
      else if (E <= 128) RB_LAUNCH(8);
      else RB_LAUNCH(16);
#undef RB_LAUNCH
    }
  }
  if (nch > 1) {
    KernelTimer kt("route_dw_reduce", s);
    const int n4 = E * d.d_model / 4;
    const int blocks = (n4 + 256 / RED_G - 1) / (256 / RED_G);
    hipLaunchKernelGGL(route_dw_reduce_kernel, dim3(blocks), dim3(256), 0, s, n4, nch, (const float4*)part,
                       (float4*)dwr);
  }
  return hipGetLastError();
}

hipError_t launch_route_bwd(const moe_desc& d, const void* x, const float* logits, const int32_t* idx,
                            const float* w, const float* dgate, float* dl, float* dwr, void* ws, hipStream_t s) {
  if (d.dtype == MOE_BF16) return route_bwd_t<bf16>(d, x, logits, idx, w, dgate, dl, dwr, ws, s);
  return route_bwd_t<float>(d, x, logits, idx, w, dgate, dl, dwr, ws, s);
}

}  // namespace pcmoe
