// Expert passes of Alg. 6 (ForwardExpert / BackwardExpert) as grouped GEMMs — fp32 storage path
// (v_mfma_f32_16x16x4_f32). The bf16 path is grouped_gemm_bf16.hip.
//
// One kernel template covers the six contractions of a SwiGLU expert:
//   FWD_GU   [G|U] = h W_{gate|up}^T, epilogue H = silu(G) * U    (M = rows, N = 2f, K = d)
//   FWD_DOWN O = H W_down^T                                       (M = rows, N = d,  K = f)
//   BWD_DH   dH = dO W_down, epilogue dG, dU (SwiGLU adjoint)      (M = rows, N = f,  K = d)
//   BWD_DX   dh = [dG|dU] [W_gate;W_up]                            (M = rows, N = d,  K = 2f)
//   WG_DOWN  dW_down = dO^T H                                      (M = d,  N = f,  K = rows)
//   WG_GU    [dW_gate;dW_up] = [dG|dU]^T h                         (M = 2f, N = d,  K = rows)
// Groups are the hosted routed experts (rows from the dispatch offsets, read on the device) and
// the shared experts (all T tokens).
//
// What bounds it: the fp32 matrix rate (154 TFLOP/s measured; a 16x16x4 MFMA takes 32 cycles), so operand traffic is
// cheap and the design spends it on balance and on wavefronts in flight: 64 x 64 tiles of 4 wavefronts, four
// workgroups per CU. Measured on T = 1500, d = 512, f = 1024, E = 8, top-2, one shared expert (forward and backward,
// 43 GFLOP): 481 us against 494 with three stages (three workgroups per CU), 526 with 128 x 64 tiles and 697 with
// 128 x 128 ones (1,240 before); the order is the same at 6,000 rows of d = 1024 (119 TFLOP/s) and at 10 rows.
// Operands stream global -> LDS through direct loads into a two-stage ring of 32-deep K-tiles; rows past a group's
// end read as zeros through the buffer range check. Both operand layouts are kept as they lie in memory: K-contiguous
// rows are read as 16-byte chunks (lane group q holds k = 4q .. 4q + 3 and feeds four MFMAs), K-major rows word by
// word at the same k, so nothing is transposed. The MFMAs multiply B by A, which leaves four consecutive output columns in a lane: the
// epilogue stores 16 bytes straight from the accumulators. The backward runs each weight gradient in one launch with
// an independent input gradient.
#include "grouped_gemm.h"

namespace pcmoe {

struct CfgF {
  static constexpr int BM = 64, BN = 64, STAGES = 2;
  static constexpr int BK = 32, ROWB = 128;  // K-tile depth; bytes of a K-contiguous tile row (8 chunks)
  static constexpr int NW = 4, NT = 256;     // 2 x 2 wavefronts
  static constexpr int WTM = BM / 2, WTN = BN / 2, FM = WTM / 16, FN = WTN / 16;
  // 1 KB per direct load: 8 K-contiguous rows or 4 K-major rows. K-major blocks are followed by 64 bytes of padding,
  // which puts the rows of lane groups q = 0 .. 3 (four rows apart) 16 banks apart.
  static constexpr int IA = BM * ROWB / 1024, IB = BN * ROWB / 1024;
  static constexpr int KM_BLOCK = 1024 + 64;
  static constexpr int A_BYTES = IA * KM_BLOCK;
  static constexpr int STAGE = A_BYTES + IB * KM_BLOCK;
  static constexpr int LDS = STAGES * STAGE;
  static constexpr int LA = IA / NW, LB = IB / NW, LOADS = LA + LB;
};
typedef CfgF C;

// 16-byte chunk c of K-contiguous tile row r lies at slot c ^ f_swz(r).
__device__ __forceinline__ int f_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

template <int KIND>
__device__ __forceinline__ void gemm_tile_f32(const GemmArgs& p, int bid, char* smem) {
  using KT = KindTraits<KIND>;
  constexpr int ES = 4, BM = C::BM, BN = C::BN, BK = C::BK, NW = C::NW;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, q = lane >> 4;

  TileIdx ti;
  if (!decode_tile<KT::ragged_m>(p, bid, ti)) return;
  const int g = ti.g, d = p.d, f = p.f;
  const bool routed = g < p.Eloc;
  const int rows = ti.rows;
  const size_t rs = routed ? (size_t)ti.row0 : (size_t)p.rows_cap + (size_t)(g - p.Eloc) * p.T;  // row-space base
  const int m0 = ti.mt * BM, n0 = ti.nt * BN;
  int K;
  if (KIND == FWD_GU || KIND == BWD_DH) K = d;
  else if (KIND == FWD_DOWN) K = f;
  else if (KIND == BWD_DX) K = 2 * f;
  else K = rows;

  // ------------------------------------------------------------------ operand sources (as in the bf16 kernel)
  const char *a_base, *b0_base, *b1_base;
  uint32_t b_bytes;
  int a_ld, b_ld;
  if (KIND == FWD_GU) { a_base = routed ? (const char*)p.xp + rs * d * ES : (const char*)p.x; a_ld = d * ES; }
  else if (KIND == FWD_DOWN) { a_base = (const char*)p.h + rs * f * ES; a_ld = f * ES; }
  else if (KIND == BWD_DH || KIND == WG_DOWN) {
    a_base = routed ? (const char*)p.dyp + rs * d * ES : (const char*)p.dy;
    a_ld = d * ES;
  } else { a_base = (const char*)p.dgu + rs * 2 * f * ES; a_ld = 2 * f * ES; }
  if (KIND == FWD_GU || KIND == BWD_DX) {
    b0_base = (const char*)p.wg + (size_t)g * f * d * ES;
    b1_base = (const char*)p.wu + (size_t)g * f * d * ES;
    b_bytes = (uint32_t)((size_t)f * d * ES);
    b_ld = d * ES;
  } else if (KIND == FWD_DOWN || KIND == BWD_DH) {
    b0_base = b1_base = (const char*)p.wd + (size_t)g * d * f * ES;
    b_bytes = (uint32_t)((size_t)d * f * ES);
    b_ld = f * ES;
  } else if (KIND == WG_DOWN) {
    b0_base = b1_base = (const char*)p.h + rs * f * ES;
    b_bytes = (uint32_t)((size_t)rows * f * ES);
    b_ld = f * ES;
  } else {  // WG_GU
    b0_base = b1_base = routed ? (const char*)p.xp + rs * d * ES : (const char*)p.x;
    b_bytes = (uint32_t)((size_t)rows * d * ES);
    b_ld = d * ES;
  }
  const int32x4 ra = make_rsrc(a_base, (uint32_t)((size_t)rows * a_ld)), rb0 = make_rsrc(b0_base, b_bytes),
                rb1 = make_rsrc(b1_base, b_bytes);

  // Per-lane byte offset at K-tile 0 of this wavefront's direct loads jj = wave + 4 j of each operand.
  int va[C::LA], vb[C::LB];
  bool bup[C::LB];
#pragma unroll
  for (int j = 0; j < C::LA; ++j) {
    const int jj = wave + NW * j;
    if (KT::a_kc) {
      const int r = 8 * jj + (lane >> 3), c = (lane & 7) ^ f_swz(r);
      va[j] = (m0 + r) * a_ld + 16 * c;
    } else {
      constexpr int CPR = BM / 4;  // chunks per K-major row
      const int slot = 64 * jj + lane;
      va[j] = (slot / CPR) * a_ld + (m0 + 4 * (slot % CPR)) * ES;
    }
  }
#pragma unroll
  for (int j = 0; j < C::LB; ++j) {
    const int jj = wave + NW * j;
    bup[j] = false;
    if (KT::b_kc) {
      const int r = 8 * jj + (lane >> 3), c = (lane & 7) ^ f_swz(r);
      int wrow = n0 + r;
      if (KIND == FWD_GU) {  // wave column: its first WTN / 2 rows are gate rows, the others the same up rows
        constexpr int HALF = C::WTN / 2;
        const int within = r % C::WTN;
        wrow = ti.nt * (BN / 2) + (r / C::WTN) * HALF + within % HALF;
        bup[j] = (8 * jj) % C::WTN >= HALF;  // the load's 8 rows are all gate or all up rows
      }
      vb[j] = wrow * b_ld + 16 * c;
    } else {
      constexpr int CPR = BN / 4;
      const int slot = 64 * jj + lane;
      vb[j] = (slot / CPR) * b_ld + (n0 + 4 * (slot % CPR)) * ES;
    }
  }
  const uint32_t lds_base = lds_addr(smem);
  const auto issue = [&](int kt, int stage) {
    const int k0 = kt * BK;
    const uint32_t st = lds_base + stage * C::STAGE;
#pragma unroll
    for (int j = 0; j < C::LA; ++j) {
      const int jj = wave + NW * j;
      dma16(ra, st + jj * (KT::a_kc ? 1024 : C::KM_BLOCK), va[j] + (KT::a_kc ? k0 * ES : k0 * a_ld));
    }
#pragma unroll
    for (int j = 0; j < C::LB; ++j) {
      const int jj = wave + NW * j;
      const uint32_t dst = st + C::A_BYTES + jj * (KT::b_kc ? 1024 : C::KM_BLOCK);
      if (KIND == BWD_DX) {
        const bool hi = k0 >= f;  // K rows >= f are W_up rows
        dma16(hi ? rb1 : rb0, dst, vb[j] + (hi ? k0 - f : k0) * b_ld);
      } else {
        dma16(bup[j] ? rb1 : rb0, dst, vb[j] + (KT::b_kc ? k0 * ES : k0 * b_ld));
      }
    }
  };

  floatx4 acc[C::FM][C::FN];
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // Fragment i (16 rows) of 16-deep step kk: element s is row (or column) 16 i + li at k = 16 kk + 4 q + s.
  const auto frag = [&](const char* S, auto kc, int w0, int kk, int i, float (&v)[4]) {
    if constexpr (decltype(kc)::value) {
      const int r = w0 + 16 * i + li;
      const Chunk c = ld_chunk(S + r * C::ROWB + (((4 * kk + q) ^ f_swz(r)) << 4));
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = __uint_as_float(c.w[s]);
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int k = 16 * kk + 4 * q + s;
        v[s] = *reinterpret_cast<const float*>(S + (k / 4) * C::KM_BLOCK + (k % 4) * 256 + (w0 + 16 * i + li) * 4);
      }
    }
  };
  const int KTN = (K + BK - 1) / BK;
  const bool wave_rows = !KT::ragged_m || m0 + wm * C::WTM < rows;  // wave-uniform
#pragma unroll
  for (int s = 0; s < C::STAGES - 1; ++s)
    if (s < KTN) issue(s, s);
  int stage = 0, fill = C::STAGES - 1;
  for (int kt = 0; kt < KTN; ++kt) {
    // K-tile kt has landed when at most the later tiles' loads are outstanding
    if (kt + C::STAGES - 2 < KTN) wait_vmcnt<(C::STAGES - 2) * C::LOADS>();
    else wait_vmcnt<0>();
    // every wave's loads of kt have landed, and its reads of the stage about to be refilled are done
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (kt + C::STAGES - 1 < KTN) issue(kt + C::STAGES - 1, fill);
    const char* As = smem + stage * C::STAGE;
    const char* Bs = As + C::A_BYTES;
    stage = stage + 1 == C::STAGES ? 0 : stage + 1;
    fill = fill + 1 == C::STAGES ? 0 : fill + 1;
    if (!wave_rows) continue;  // all rows lie past the group's end: only loads and syncs
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      float a[C::FM][4], b[C::FN][4];
#pragma unroll
      for (int i = 0; i < C::FM; ++i) frag(As, std::bool_constant<KT::a_kc>{}, wm * C::WTM, kk, i, a[i]);
#pragma unroll
      for (int j = 0; j < C::FN; ++j) frag(Bs, std::bool_constant<KT::b_kc>{}, wn * C::WTN, kk, j, b[j]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
          for (int j = 0; j < C::FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][s], a[i][s], acc[i][j], 0, 0, 0);
    }
  }

  // ------------------------------------------------------------------ epilogue: lane (li, q) of block (i, j) holds
  // row 16 i + li, columns 16 j + 4 q .. + 3
#pragma unroll
  for (int i = 0; i < C::FM; ++i) {
    const int m = m0 + wm * C::WTM + 16 * i + li;
    if (KT::ragged_m && m >= rows) continue;
    if (KIND == FWD_GU) {
#pragma unroll
      for (int j = 0; j < C::FN / 2; ++j) {
        const floatx4 gv = acc[i][j], uv = acc[i][j + C::FN / 2];
        floatx4 hv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float sg = 1.f / (1.f + __expf(-gv[e]));
          hv[e] = gv[e] * sg * uv[e];
        }
        const int col = ti.nt * (BN / 2) + wn * (C::WTN / 2) + 16 * j + 4 * q;
        float* gu = (float*)p.gu + (rs + m) * 2 * f + col;
        *reinterpret_cast<floatx4*>(gu) = gv;
        *reinterpret_cast<floatx4*>(gu + f) = uv;
        *reinterpret_cast<floatx4*>((float*)p.h + (rs + m) * f + col) = hv;
      }
      continue;
    }
#pragma unroll
    for (int j = 0; j < C::FN; ++j) {
      const floatx4 v = acc[i][j];
      const int col = n0 + wn * C::WTN + 16 * j + 4 * q;
      if (KIND == FWD_DOWN || KIND == BWD_DX) {
        *reinterpret_cast<floatx4*>((float*)p.out + (rs + m) * d + col) = v;
      } else if (KIND == BWD_DH) {
        const float* gu = (const float*)p.gu + (rs + m) * 2 * f + col;
        const floatx4 gv = *reinterpret_cast<const floatx4*>(gu), uv = *reinterpret_cast<const floatx4*>(gu + f);
        floatx4 dg, du;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float sg = 1.f / (1.f + __expf(-gv[e]));
          du[e] = v[e] * gv[e] * sg;
          dg[e] = v[e] * uv[e] * sg * (1.f + gv[e] * (1.f - sg));
        }
        float* o = (float*)p.dgu + (rs + m) * 2 * f + col;
        *reinterpret_cast<floatx4*>(o) = dg;
        *reinterpret_cast<floatx4*>(o + f) = du;
      } else if (KIND == WG_DOWN) {
        *reinterpret_cast<floatx4*>((float*)p.out + ((size_t)g * d + m) * f + col) = v;
      } else {  // WG_GU
        float* o = m < f ? (float*)p.out + ((size_t)g * f + m) * d + col
                         : (float*)p.out2 + ((size_t)g * f + (m - f)) * d + col;
        *reinterpret_cast<floatx4*>(o) = v;
      }
    }
  }
}

// Workgroups [0, grid_a) take tiles of KA, the others tiles of KB (independent contractions).
template <int KA, int KB>
__global__ __launch_bounds__(C::NT) void gemm_f32_kernel(GemmArgs pa, GemmArgs pb, int grid_a) {
  extern __shared__ __align__(16) char smem[];
  const int bid = blockIdx.x;
  if (KA == KB || bid < grid_a) gemm_tile_f32<KA>(pa, bid, smem);
  else gemm_tile_f32<KB>(pb, bid - grid_a, smem);
}

// ------------------------------------------------------------------------- host side

static int round8(long v) { return (int)((v + 7) / 8 * 8); }

template <int KA, int KB>
static hipError_t run_f32(const GemmArgs& a, long tiles_a, const GemmArgs& b, long tiles_b, hipStream_t s,
                          const char* name) {
  auto kern = gemm_f32_kernel<KA, KB>;
  static_assert(C::LDS <= 65536, "more LDS needs the kernel's limit raised");
  const int grid_a = round8(tiles_a), grid = grid_a + (KA == KB ? 0 : round8(tiles_b));
  if (grid <= 0) return hipSuccess;
  KernelTimer kt(name, s);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(C::NT), C::LDS, s, a, b, grid_a);
  return hipGetLastError();
}

static GemmArgs base_args(const moe_desc& d, const int32_t* offsets) {
  GemmArgs a{};
  a.T = d.T; a.k = d.top_k; a.d = d.d_model; a.f = d.d_ff; a.Eloc = d.local_count; a.S = d.n_shared;
  a.rows_cap = d.T * d.top_k;
  a.offsets = offsets;
  return a;
}

// Workgroups of a contraction with `cols` output columns: row-ragged kinds (an upper bound on their m-tiles, since the
// per-expert counts stay on the device) and weight gradients.
static long ragged_tiles(const moe_desc& d, GemmArgs& a, int cols) {
  a.n_tiles = cols / C::BN;
  const long m_tiles = ((long)d.T * d.top_k + (long)d.local_count * (C::BM - 1)) / C::BM +
                       (long)d.n_shared * ((d.T + C::BM - 1) / C::BM);
  return m_tiles * a.n_tiles;
}
static long wgrad_tiles(const moe_desc& d, GemmArgs& a, int M, int N) {
  a.m_tiles = M / C::BM;
  a.n_tiles = N / C::BN;
  return (long)(d.local_count + d.n_shared) * a.m_tiles * a.n_tiles;
}

hipError_t ffn_fwd_f32(const moe_desc& d, const void* x, const void* xp, const int32_t* offsets, const void* wg,
                       const void* wu, const void* wd, void* yp, void* saved, const int32_t* pre64, hipStream_t s) {
  const size_t R = (size_t)rows_total(d), es = sizeof(float);
  GemmArgs a = base_args(d, offsets);
  a.x = x; a.xp = xp; a.wg = wg; a.wu = wu; a.wd = wd;
  a.gu = saved;
  a.h = (char*)saved + align256(R * 2 * d.d_ff * es);
  a.out = yp;
  a.mt_prefix = pre64;
  const long t_gu = ragged_tiles(d, a, 2 * d.d_ff);
  if (hipError_t e = run_f32<FWD_GU, FWD_GU>(a, t_gu, a, 0, s, "gemm_fwd_gate_up"); e != hipSuccess) return e;
  const long t_dn = ragged_tiles(d, a, d.d_model);
  return run_f32<FWD_DOWN, FWD_DOWN>(a, t_dn, a, 0, s, "gemm_fwd_down");
}

hipError_t ffn_bwd_f32(const moe_desc& d, const void* x, const void* xp, const void* dy, const void* dyp,
                       const int32_t* offsets, const void* wg, const void* wu, const void* wd, const void* saved,
                       void* dxp, void* dwg, void* dwu, void* dwd, void* dgu, const int32_t* pre64,
                       const int32_t* order, hipStream_t s) {
  const size_t R = (size_t)rows_total(d), es = sizeof(float);
  GemmArgs a = base_args(d, offsets);
  a.x = x; a.xp = xp; a.dy = dy; a.dyp = dyp; a.wg = wg; a.wu = wu; a.wd = wd;
  a.gu = (void*)saved;
  a.h = (char*)saved + align256(R * 2 * d.d_ff * es);
  a.dgu = dgu;
  a.mt_prefix = pre64;
  GemmArgs dh = a, dwn = a, dx = a, wgu = a;
  dwn.out = dwd;
  dwn.order = wgu.order = order;
  wgu.out = dwg;
  wgu.out2 = dwu;
  dx.out = dxp;
  const long t_dh = ragged_tiles(d, dh, d.d_ff), t_wd = wgrad_tiles(d, dwn, d.d_model, d.d_ff);
  const long t_dx = ragged_tiles(d, dx, d.d_model), t_wgu = wgrad_tiles(d, wgu, 2 * d.d_ff, d.d_model);
  // the weight gradients first, heaviest groups first: their K loops (a group's rows) vary, the others' do not
  if (hipError_t e = run_f32<WG_DOWN, BWD_DH>(dwn, t_wd, dh, t_dh, s, "gemm_bwd_dh+wgrad_down"); e != hipSuccess)
    return e;
  return run_f32<WG_GU, BWD_DX>(wgu, t_wgu, dx, t_dx, s, "gemm_bwd_dx+wgrad_gate_up");
}

}  // namespace pcmoe
