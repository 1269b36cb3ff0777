// Expert passes over few rows per expert (decode steps, short prompts, small micro-batches) in bf16.
//
// With few rows per expert a contraction is bound by reading the weights once. The LDS-tiled kernels
// (grouped_gemm_bf16.hip) then run one workgroup per CU that waits for each K-tile's round trip. Here the weights
// never pass through LDS: each wavefront reads 64 contiguous bytes of 16 weight rows per load straight into MFMA
// operand registers, several loads ahead, and the small register and LDS footprint leaves two and more workgroups on a
// CU. The weights are the MFMA's first operand, the activations' rows the second, so that a lane's four accumulators
// are four consecutive output columns of one row.
//   * stream_cols_kernel (up to 8 rows per group): a wavefront owns 16 or 32 output columns of 16 rows and shares nothing;
//   * stream_rows_kernel (up to 32 to 200 rows, stream_pick): the wavefronts split the columns and share 32, 64 or 128
//     rows through LDS.
// Both sum over K in the order of the LDS tiles (one accumulator per output, 32 k per MFMA): the results are the same bits
// whichever kernel a batch size selects.
// The group, row chunk and columns of a workgroup come from the offsets alone (a scan over the wavefront), so no tile
// plan has to be launched first; the plan that the backward reads is written by extra workgroups of FWD_GU.
// Measured (layer forward, us, LDS tiles -> now):
//   T=24, d=4096, f=14336, E=8, top-2: gate/up 350 -> 310, down 279 -> 171 (bound by the weights, 5.4-5.8 TB/s);
//   T=1, d=2048, f=1408, E=64, top-6, 2 shared: gate/up 29 -> 19, down 34 -> 12 (4.8 and 3.9 TB/s).
//   T=777, d=1024, f=2816, E=16, top-2: gate/up 58 -> 52, down 61 -> 33 (3.5 and 2.8 TB/s).
#include "grouped_gemm.h"

#include <algorithm>
#include <cmath>

namespace pcmoe {

// Workgroup -> (group, row chunk of `chunk` rows, column block). Lane l of a wavefront counts the chunks of the groups
// [l NS, l NS + NS) (one batch of loads), a scan over the lanes finds the lane whose groups hold the tile, and its
// groups are then walked. Consecutive tiles, the row chunks of one column block first, stay on one XCD, whose L2 then
// serves the chunks' repeated weight reads.
struct StreamTile {
  int g, row0, rows, ch, nb;
};
template <int NS>
__device__ __forceinline__ bool stream_decode_ns(const GemmArgs& p, int bid, int chunk, int n_blocks, StreamTile& t) {
  const int G = p.Eloc + p.S, lane = threadIdx.x & 63, g0 = lane * NS;
  int off[NS + 1], sum = 0;
#pragma unroll
  for (int s = 0; s <= NS; ++s) off[s] = p.offsets[min(g0 + s, p.Eloc)];
  auto rows_of = [&](int g, int lo, int hi) { return g < p.Eloc ? hi - lo : g < G ? p.T : 0; };
#pragma unroll
  for (int s = 0; s < NS; ++s) sum += (rows_of(g0 + s, off[s], off[s + 1]) + chunk - 1) / chunk;
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(incl, o, 64);
    if (lane >= o) incl += u;
  }
  const int total = __builtin_amdgcn_readlane(incl, 63) * n_blocks;
  const int x = bid & 7, lb = bid >> 3, q = total >> 3, r = total & 7;
  if (lb >= q + (x < r ? 1 : 0)) return false;
  const int L = x * q + min(x, r) + lb;
  const int j = __popcll(__ballot(incl * n_blocks <= L));  // the lane holding tile L (L < total: j < 64)
  int l = L - __builtin_amdgcn_readlane(incl - sum, j) * n_blocks, nch = 1;
  bool found = false;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int lo = __builtin_amdgcn_readlane(off[s], j), hi = __builtin_amdgcn_readlane(off[s + 1], j);
    const int rows = rows_of(j * NS + s, lo, hi), n = (rows + chunk - 1) / chunk;
    if (!found && l < n * n_blocks) {
      found = true;
      t.g = j * NS + s;
      t.row0 = lo;
      t.rows = rows;
      nch = n;
    }
    if (!found) l -= n * n_blocks;
  }
  t.nb = __builtin_amdgcn_readfirstlane(l / nch);
  t.ch = __builtin_amdgcn_readfirstlane(l - (l / nch) * nch);
  return true;
}
__device__ __forceinline__ bool stream_decode(const GemmArgs& p, int bid, int chunk, int n_blocks, StreamTile& t) {
  const int G = p.Eloc + p.S;
  if (G <= 64) return stream_decode_ns<1>(p, bid, chunk, n_blocks, t);
  if (G <= 128) return stream_decode_ns<2>(p, bid, chunk, n_blocks, t);
  return stream_decode_ns<8>(p, bid, chunk, n_blocks, t);
}

__device__ __forceinline__ uint2 pack4(const floatx4& v) {
  return uint2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}
// Four consecutive columns of one row: G, U and H = silu(G) U, or the down projection's output.
__device__ __forceinline__ void store_gu(const GemmArgs& p, size_t row, int col, const floatx4& g, const floatx4& u) {
  floatx4 h;
#pragma unroll
  for (int e = 0; e < 4; ++e) h[e] = g[e] * __builtin_amdgcn_rcpf(1.f + __expf(-g[e])) * u[e];
  bf16* gu = (bf16*)p.gu + row * 2 * p.f + col;
  *reinterpret_cast<uint2*>(gu) = pack4(g);
  *reinterpret_cast<uint2*>(gu + p.f) = pack4(u);
  *reinterpret_cast<uint2*>((bf16*)p.h + row * p.f + col) = pack4(h);
}
__device__ __forceinline__ void store_out(const GemmArgs& p, size_t row, int col, const floatx4& v) {
  *reinterpret_cast<uint2*>((bf16*)p.out + row * p.d + col) = pack4(v);
}

// Up to 16 rows of a group, KIND FWD_GU or FWD_DOWN: a workgroup is one wavefront, which owns 16 M weight rows (FWD_GU:
// 16 M gate rows and the same up rows) over the whole K and reads them and the group's rows straight into MFMA operands,
// D steps of 64 k ahead. Bound by the round trips of a wavefront's loads as long as few groups are active, then by the
// weights: single wavefronts spread evenly over the CUs and wait for no one (T = 1 of the 64-expert layer above: gate/up
// 19 us, 23 by workgroups of four). M = 2 halves the reads of the rows, which matter from a few rows per group on; it
// leaves half the wavefronts. (A split of K over four wavefronts, summed through LDS, took 23 and 12 us there and 84 and
// 63, now 82 and 49, at T = 1 of 8 experts, d = 4096, f = 14336; and its results were other bits than the tiles'.)
template <int KIND, int M, int D>
__global__ __launch_bounds__(64, 2) void stream_cols_kernel(GemmArgs p, PlanArgs plan, int n_blocks, int tiles) {
  constexpr int NF = KIND == FWD_GU ? 2 * M : M;
  if (KIND == FWD_GU && (int)blockIdx.x >= tiles) {
    __shared__ int rows_s[512];
    plan_part(plan, blockIdx.x - tiles, rows_s);
    return;
  }
  StreamTile t;
  if (!stream_decode(p, blockIdx.x, 16, n_blocks, t)) return;
  const int lane = threadIdx.x & 63, q = lane >> 4, li = lane & 15;
  const int K = KIND == FWD_GU ? p.d : p.f, KB = K * 2, units = K / 64;
  const bool routed = t.g < p.Eloc;
  // rows of the activations: x_perm / H rows of a routed group, x / H rows of a shared expert
  const size_t rs = routed ? (size_t)t.row0 : (size_t)p.rows_cap + (size_t)(t.g - p.Eloc) * p.T;
  const char* xb = KIND == FWD_GU ? (routed ? (const char*)p.xp + (size_t)t.row0 * KB : (const char*)p.x)
                                  : (const char*)p.h + rs * KB;
  const int m0 = t.ch * 16, m_rows = min(t.rows - m0, 16);
  const auto xr = buf_rsrc(xb + (size_t)m0 * KB, (size_t)m_rows * KB);
  const size_t wsz = (size_t)p.d * p.f * 2;
  const int wrow = t.nb * 16 * M;  // first output column and weight row
  const char* w0 = (const char*)(KIND == FWD_GU ? p.wg : p.wd) + t.g * wsz + (size_t)wrow * KB;
  const char* w1 = KIND == FWD_GU ? (const char*)p.wu + t.g * wsz + (size_t)wrow * KB : w0;
  const auto wr0 = buf_rsrc(w0, (size_t)16 * M * KB);
  const auto wr1 = buf_rsrc(w1, (size_t)16 * M * KB);

  floatx4 acc[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  Chunk wb[D][NF][2], xv[D][2];
  // step u: bytes [128 u, 128 u + 128) of each row (zeros past the last)
  auto load = [&](int u, Chunk(&wbuf)[NF][2], Chunk(&xbuf)[2]) {
    const int vo = li * KB + q * 16 + u * 128;
#pragma unroll
    for (int h = 0; h < 2; ++h) xbuf[h] = buf_ld16(xr, u < units ? vo + 64 * h : kBufPast);
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        wbuf[i][h] = buf_ld16(i < M ? wr0 : wr1, u < units ? vo + (i % M) * 16 * KB + 64 * h : kBufPast);
  };
  // the scheduling barriers keep each step's loads behind the MFMAs before them: left alone, the compiler gathers the
  // steps' loads at the loop's end and waits for all of them at its top
#pragma unroll
  for (int s = 0; s < D; ++s) {
    load(s, wb[s], xv[s]);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int u0 = 0; u0 < units; u0 += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < NF; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wb[s][i][h]),
                                                           __builtin_bit_cast(bf16x8, xv[s][h]), acc[i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      load(u0 + s + D, wb[s], xv[s]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // lane (q, li), block i: columns 16 i + 4 q .. 16 i + 4 q + 3 of row li
  if (li >= m_rows) return;
  const size_t row = rs + m0 + li;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    if (KIND == FWD_GU) store_gu(p, row, wrow + 16 * i + 4 * q, acc[i], acc[NF - M + i]);
    else store_out(p, row, wrow + 16 * i + 4 * q, acc[i]);
  }
}

// Up to 16 MT rows of a group: the wavefronts share the rows and split the columns.
//   * each of the 4 wavefronts owns 16 NF weight rows (FWD_GU: 16 gate rows and the same 16 up rows) over the whole K
//     and keeps D steps of 64 k of them in flight in registers;
//   * the group's rows (up to 16 MT) pass through LDS, 64 k at a time in two stages, filled from registers that are
//     loaded D - 1 steps before they are put there: one barrier per step. With D > 2 no load is waited for in the step
//     that issues it; with D = 2 (gate/up of 128 rows) the next step's rows are, at the step's end;
//   * the accumulators hold four consecutive output columns of one row per lane, so SwiGLU and the stores need no LDS.
// X stage: 128-byte rows, 16-byte chunk c of row r at c ^ swz(r).
__device__ __forceinline__ int xs_swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

template <int KIND, int MT, int NF, int D>
__global__ __launch_bounds__(256, 2) void stream_rows_kernel(GemmArgs p, PlanArgs plan, int n_blocks, int tiles) {
  static_assert(D % 2 == 0 && (KIND != FWD_GU || NF == 2), "");
  constexpr int ROWS = 16 * MT, XL = ROWS * 8 / 256 > 0 ? ROWS * 8 / 256 : 1;  // 16-byte chunks of X per thread and step
  constexpr int COLS = KIND == FWD_GU ? 64 : 64 * NF;                           // output columns of the workgroup
  __shared__ __align__(16) char xs[2][ROWS * 128 > 2048 ? ROWS * 128 : 2048];
  if (KIND == FWD_GU && (int)blockIdx.x >= tiles) {
    plan_block<256>(plan, (int*)xs);
    return;
  }
  StreamTile t;
  if (!stream_decode(p, blockIdx.x, ROWS, n_blocks, t)) return;
  const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, li = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = KIND == FWD_GU ? p.d : p.f, KB = K * 2, units = K / 64;
  const bool routed = t.g < p.Eloc;
  const size_t rs = routed ? (size_t)t.row0 : (size_t)p.rows_cap + (size_t)(t.g - p.Eloc) * p.T;
  const char* xb = KIND == FWD_GU ? (routed ? (const char*)p.xp + (size_t)t.row0 * KB : (const char*)p.x)
                                  : (const char*)p.h + rs * KB;
  const int m0 = t.ch * ROWS, m_rows = min(t.rows - m0, ROWS);
  const auto xr = buf_rsrc(xb + (size_t)m0 * KB, (size_t)m_rows * KB);
  const size_t wsz = (size_t)p.d * p.f * 2;
  const int wrow = t.nb * COLS + w * (KIND == FWD_GU ? 16 : 16 * NF);  // the wavefront's first output column
  const char* w0 = (const char*)(KIND == FWD_GU ? p.wg : p.wd) + t.g * wsz + (size_t)wrow * KB;
  const char* w1 = KIND == FWD_GU ? (const char*)p.wu + t.g * wsz + (size_t)wrow * KB : w0;
  constexpr int F0 = KIND == FWD_GU ? 1 : NF;
  const auto wr0 = buf_rsrc(w0, (size_t)16 * F0 * KB);
  const auto wr1 = buf_rsrc(w1, (size_t)16 * F0 * KB);

  Chunk wb[D][NF][2], xv[D][XL];
  auto load_w = [&](int u, Chunk(&buf)[NF][2]) {
    const int vo = li * KB + q * 16 + u * 128;
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        buf[i][h] = buf_ld16(i < F0 ? wr0 : wr1, u < units ? vo + (i % F0) * 16 * KB + 64 * h : kBufPast);
  };
  auto load_x = [&](int u, Chunk(&buf)[XL]) {
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int c = tid + 256 * i;  // rows past the chunk's last one lie past the buffer: zeros
      buf[i] = buf_ld16(xr, u < units ? (c >> 3) * KB + (c & 7) * 16 + u * 128 : kBufPast);
    }
  };
  auto put_x = [&](int stage, const Chunk(&buf)[XL]) {
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int c = tid + 256 * i, r = c >> 3;
      if (ROWS * 8 >= 256 || r < ROWS) st_chunk(xs[stage] + r * 128 + (((c & 7) ^ xs_swz(r)) << 4), buf[i]);
    }
  };
  floatx4 acc[MT][NF];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int i = 0; i < NF; ++i) acc[m][i] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int swz = xs_swz(li);  // every 16-row block repeats it
  auto mul = [&](int stage, const Chunk(&buf)[NF][2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const Chunk x = ld_chunk(xs[stage] + (16 * m + li) * 128 + (((4 * h + q) ^ swz) << 4));
#pragma unroll
        for (int i = 0; i < NF; ++i)
          acc[m][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, buf[i][h]),
                                                              __builtin_bit_cast(bf16x8, x), acc[m][i], 0, 0, 0);
      }
  };
  // Loads complete in order: a step's rows are issued ahead of its weights and as early, so that waiting for them never
  // means waiting for weights of a later step.
#pragma unroll
  for (int s = 0; s < D - 1; ++s) {
    load_x(s, xv[s]);
    load_w(s, wb[s]);
    __builtin_amdgcn_sched_barrier(0);
  }
  put_x(0, xv[0]);
  for (int u0 = 0; u0 < units; u0 += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const int u = u0 + s;
      if (u >= units) break;
      // stage u is filled, and every wavefront has left step u - 1, whose stage this step refills
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      load_x(u + D - 1, xv[(s + D - 1) % D]);
      load_w(u + D - 1, wb[(s + D - 1) % D]);
      __builtin_amdgcn_sched_barrier(0);
      mul(s & 1, wb[s]);
      __builtin_amdgcn_sched_barrier(0);
      put_x((s + 1) & 1, xv[(s + 1) % D]);
    }
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int r = 16 * m + li;
    if (r >= m_rows) continue;
    const size_t row = rs + m0 + r;
    if (KIND == FWD_GU) {
      store_gu(p, row, wrow + 4 * q, acc[m][0], acc[m][NF - 1]);
    } else {
#pragma unroll
      for (int i = 0; i < NF; ++i) store_out(p, row, wrow + 16 * i + 4 * q, acc[m][i]);
    }
  }
}

// dX = dG W_gate + dU W_up of few rows, where the LDS tiles of d columns are too few for the length of K = 2 f. K is the
// slow dimension of the weights here, so a wavefront reads 32 k-rows x 128 columns per step, each load 256 contiguous
// bytes of 4 rows, and turns a lane's 8 k x 8 n block into 8 MFMA operands with 32 byte permutes: operand s of lane (q, i)
// holds column 8 i + s, k = 8 q .. 8 q + 7. A lane's accumulators of one row are then 8 consecutive columns. The DX_KS
// wavefronts split K and their partial sums meet in LDS, in wavefront order, 64 columns of 16 rows at a time.
constexpr int DX_KS = 8, DX_COLS = 128;
template <int MT>
__global__ __launch_bounds__(64 * DX_KS, 2) void stream_dx_kernel(GemmArgs p, int n_blocks) {
  constexpr int KS = DX_KS, PITCH = 64 + 4, D = 3;  // D: steps of weights in registers
  __shared__ __align__(16) float red[KS * 16 * PITCH];
  StreamTile t;
  if (!stream_decode(p, blockIdx.x, 16 * MT, n_blocks, t)) return;
  const int lane = threadIdx.x & 63, q = lane >> 4, li = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KB = 4 * p.f, NB = 2 * p.d;  // bytes of a row of dG|dU and of a weight matrix
  const bool routed = t.g < p.Eloc;
  const size_t rs = routed ? (size_t)t.row0 : (size_t)p.rows_cap + (size_t)(t.g - p.Eloc) * p.T;
  const char* xb = (const char*)p.dgu + rs * KB;
  const int m0 = t.ch * 16 * MT, m_rows = min(t.rows - m0, 16 * MT);
  const auto xr = buf_rsrc(xb + (size_t)m0 * KB, (size_t)m_rows * KB);
  const int n0 = t.nb * DX_COLS;
  const size_t wsz = (size_t)p.d * p.f * 2;
  const char* w0 = (const char*)p.wg + t.g * wsz;
  const char* w1 = (const char*)p.wu + t.g * wsz;

  const int half = p.f / 32, units = 2 * half, rounds = (units + KS - 1) / KS;  // units >= half are W_up rows
  floatx4 acc[8][MT];
#pragma unroll
  for (int s = 0; s < 8; ++s)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[s][m] = floatx4{0.f, 0.f, 0.f, 0.f};
  Chunk wb[D][8], xv[D][MT];
  // step r of this wavefront: k-rows 32 u .. 32 u + 31, u = r KS + w (zeros past the last)
  auto load = [&](int r, Chunk(&wbuf)[8], Chunk(&xbuf)[MT]) {
    const int u = r * KS + w;
    const bool up = u >= half;
    const auto wr = buf_rsrc(up ? w1 : w0, wsz);
    const int vo = u < units ? ((up ? u - half : u) * 32 + 8 * q) * NB + (n0 + 8 * li) * 2 : kBufPast;
    const int xo = u < units ? li * KB + u * 64 + q * 16 : kBufPast;
#pragma unroll
    for (int m = 0; m < MT; ++m) xbuf[m] = buf_ld16(xr, u < units ? xo + m * 16 * KB : kBufPast);
#pragma unroll
    for (int j = 0; j < 8; ++j) wbuf[j] = buf_ld16(wr, u < units ? vo + j * NB : kBufPast);
  };
  auto mul = [&](const Chunk(&wbuf)[8], const Chunk(&xbuf)[MT]) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      // halves (s & 1) of dword s / 2 of rows 2 j and 2 j + 1
      Chunk a;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        a.w[j] = __builtin_amdgcn_perm(wbuf[2 * j + 1].w[s / 2], wbuf[2 * j].w[s / 2],
                                       (s & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
      for (int m = 0; m < MT; ++m)
        acc[s][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                            __builtin_bit_cast(bf16x8, xbuf[m]), acc[s][m], 0, 0, 0);
    }
  };
#pragma unroll
  for (int s = 0; s < D; ++s) {
    load(s, wb[s], xv[s]);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (int r = 0; r < rounds; r += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      mul(wb[s], xv[s]);  // (steps past the last are zeros)
      __builtin_amdgcn_sched_barrier(0);
      load(r + s + D, wb[s], xv[s]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Sum and store. Round (m, h): rows 16 m .. 16 m + 15, the 8-column blocks 4 q + 2 h and 4 q + 2 h + 1; thread ->
  // (row, 4 columns).
  const int rr = threadIdx.x >> 4, c = (threadIdx.x & 15) * 4;  // (threads past 16 rows only write partials)
  const int col = n0 + 8 * (4 * ((c & 31) >> 3) + (c >> 5)) + (c & 7);
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (16 * m >= m_rows) break;  // uniform
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (m + h) __syncthreads();
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float* o = &red[(w * 16 + li) * PITCH + 32 * b + 8 * q];
        const int r = 2 * h + b;
        *reinterpret_cast<floatx4*>(o) = floatx4{acc[0][m][r], acc[1][m][r], acc[2][m][r], acc[3][m][r]};
        *reinterpret_cast<floatx4*>(o + 4) = floatx4{acc[4][m][r], acc[5][m][r], acc[6][m][r], acc[7][m][r]};
      }
      __syncthreads();
      if (rr < 16 && 16 * m + rr < m_rows) {
        floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) v += *reinterpret_cast<const floatx4*>(&red[(k * 16 + rr) * PITCH + c]);
        const size_t row = rs + m0 + 16 * m + rr;
        store_out(p, row, col + 16 * h, v);
      }
    }
  }
}

// ------------------------------------------------------------------------- host side

// Upper bound on the row chunks: each routed chunk holds at least one row, and all but one per group are full.
static long chunk_bound(const moe_desc& d, int chunk) {
  const long slots = (long)d.T * d.top_k;
  const long routed = std::min(slots, (slots + (long)d.local_count * (chunk - 1)) / chunk);
  return routed + (long)d.n_shared * ((d.T + chunk - 1) / chunk);
}

static unsigned grid_of(long wgs) { return (unsigned)((wgs + 7) / 8 * 8); }

template <int KIND, int M, int D>
static hipError_t run_cols(const moe_desc& d, const GemmArgs& a, const PlanArgs& plan, hipStream_t s,
                           const char* name) {
  const int n_blocks = (KIND == FWD_GU ? d.d_ff : d.d_model) / (16 * M);
  const unsigned tiles = grid_of(chunk_bound(d, 16) * n_blocks);
  const unsigned extra = KIND == FWD_GU ? plan_parts(d.local_count + d.n_shared) : 0;
  KernelTimer kt(name, s);
  hipLaunchKernelGGL((stream_cols_kernel<KIND, M, D>), dim3(tiles + extra), dim3(64), 0, s, a, plan, n_blocks,
                     (int)tiles);
  return hipGetLastError();
}
template <int KIND, int MT, int NF, int D>
static hipError_t run_rows(const moe_desc& d, const GemmArgs& a, const PlanArgs& plan, hipStream_t s,
                           const char* name) {
  const int n_blocks = KIND == FWD_GU ? d.d_ff / 64 : d.d_model / (64 * NF);
  const unsigned tiles = grid_of(chunk_bound(d, 16 * MT) * n_blocks);
  KernelTimer kt(name, s);
  hipLaunchKernelGGL((stream_rows_kernel<KIND, MT, NF, D>), dim3(tiles + (KIND == FWD_GU ? 1 : 0)), dim3(256), 0, s,
                     a, plan, n_blocks, (int)tiles);
  return hipGetLastError();
}

// Rows per group: `mean` where every expert is equally likely, `most` where every slot goes to a hosted expert (a shard
// cannot know how hot its experts are; a full layer's two are equal).
struct GroupRows {
  double mean, most;
};
static GroupRows group_rows(const moe_desc& d) {
  const double slots = (double)d.T * d.top_k, shared = (double)d.T * d.n_shared, G = d.local_count + d.n_shared;
  return {(slots * d.local_count / d.n_experts + shared) / G, (slots + shared) / G};
}

// Which streaming kernel a contraction takes, by the rows per group and the workgroups its grid has. The counts stay on
// the device, so a line has to hold however the rows are spread: a group of many rows reads its weights once per chunk,
// where the LDS tiles read them once per 256 rows. Each line was drawn from timings of all the variants and of the LDS
// tiles over 40 layers (d 256 to 4096, f 512 to 14336, 3 to 128 groups, with and without shared experts, whole layers
// and shards) at 1 to 200 rows per group, spread uniformly, Zipf-skewed (exponent 1.1) and with one expert in every
// token; no call was more than 2% slower than on the tiles. Times are tiles -> streamed, us, uniform and skewed rows:
//   * up to 8 rows: the single wavefronts, as long as they are at most 10 per CU for gate/up and 20 for the down
//     projection (at twice as many the 32-row chunks are 5-15% faster). Two column blocks each past 2 rows in gate/up (d =
//     4096, f = 2816, 8 experts: 2 rows 72 us either way, 8 rows 83 and 79) and past one row in the down projection where
//     that leaves a wavefront per CU (d = 1024, f = 2816, 16 experts, 8 rows: 22.5 and 19.2). Where the experts with a row
//     fill 1.6 workgroups per CU, the 32-row chunks of the down projection are as fast or faster (d = 2048, f = 8192, 16
//     experts, 8 rows: 127 and 108; d = 4096, f = 14336, 8 experts, 6 rows: 185 and 172; d = 4096, f = 2816: 45 and 37);
//   * up to 24, 50 and 100 rows: 32-, 64- and 128-row chunks (the next size up costs 5-30% more below each line, the
//     previous one 5-50% above it). A shard takes the size for twice its even share;
//   * where the tiles would leave half the CUs or more idle, chunks up to 200 rows: 10-60% faster, skewed or not;
//   * else the down projection goes to the tiles past 50 rows (d = 2048, f = 1408, 16 groups, 64 rows: 34 -> 25, 35 ->
//     40; d = 4096, f = 2816, 8 groups: 64 -> 44, 64 -> 78);
//   * gate/up, which also saves the launch of the tile plan (6 us) when streamed: where the tiles take one round of the
//     chip, past 80 rows (d = 2048, f = 1408, 16 groups, 99 rows: 54 -> 63, 61 -> 75); up to two rounds, past 100 rows
//     with d_model up to 1536 (d = 1024, f = 2816, 16 groups, 99 rows: 58 -> 52, 56 -> 63), 50 above (d = 2048, 79 rows:
//     103 -> 93, 98 -> 110); a shard, past 64 slots of its tokens per hosted expert (16 of 64 experts, top-4, T = 320:
//     41 -> 41, 57 -> 86);
//   * both go to the tiles past 32 rows with more than 16 groups (down, 64 experts, 39 rows: 109 -> 89, 91 -> 96) or
//     where the tiles take more than two rounds (gate/up, d = 2048, f = 5632, 16 groups, 50 rows: 159 -> 159, 149 ->
//     178), there also past 1,024 tokens (gate/up, 64 experts, top-1, T = 1280: 149 -> 145, all to one expert 51 -> 69).
// FWD_DOWN at 25 rows and more takes 128 columns per workgroup as long as that leaves one workgroup per CU (at 64 rows
// 16% faster with d = 4096, 14% slower with d = 1024 and 16 experts). A grid of few workgroups is bound by the round
// trips of each: 64-row chunks in place of 128 below 3/4 of a workgroup per CU (f = 8192, d = 1536, 5 groups, 64 rows:
// 83 -> 60 us), and 8 steps in flight in place of 4 up to two per CU (f = 8192, 12 rows: 55 -> 49 us; f = 2816, d = 1024:
// 25 -> 22; 128 experts, d = 512, are 10% slower with 8).
StreamPick stream_pick(const moe_desc& d, int kind, long tile_grid) {
  const StreamPick none{0, 0, 0};
  if (d.dtype != MOE_BF16) return none;
  const int G = d.local_count + d.n_shared;
  const GroupRows gr = group_rows(d);
  const double rows = std::min(2 * gr.mean, gr.most);
  const int cols = kind == FWD_GU ? d.d_ff : d.d_model, cus = device_cus();
  if (rows <= 8 && chunk_bound(d, 16) * (cols / 16) <= (kind == FWD_GU ? 10L : 20L) * cus) {
    if (kind == FWD_GU) return rows <= 2 ? StreamPick{1, 1, 4} : StreamPick{1, 2, 2};
    const double active = d.local_count * (1 - std::pow(1 - (double)d.top_k / d.n_experts, d.T)) + d.n_shared;
    if (active * (cols / 64) < 1.6 * cus) return StreamPick{1, rows > 1 && active * (cols / 32) >= cus ? 2 : 1, 4};
    return StreamPick{2, 1, d.d_ff >= 1024 ? 8 : 4};
  }
  if (tile_grid <= cus / 2) {
    if (gr.mean > 200) return none;
  } else {
    int limit = 50;
    if (kind == FWD_GU) {
      limit = tile_grid <= cus ? 80 : d.d_model <= 1536 ? 100 : 50;
      if (d.local_count < d.n_experts) limit = std::min(limit, 64);
    }
    const bool rounds = tile_grid > 2L * cus;  // the tiles fill more than two rounds
    if (G > 16 || rounds) limit = 32;
    if (gr.most > limit || (rounds && d.T > 1024)) return none;
  }
  int mt = rows <= 24 ? 2 : rows <= 50 ? 4 : 8;
  if (kind == FWD_GU) return StreamPick{mt, 2, mt == 8 ? 2 : 4};
  const auto wgs = [&](int m, int nf) { return chunk_bound(d, 16 * m) * (cols / (64 * nf)); };
  if (mt == 8 && wgs(8, 1) < cus * 3 / 4) mt = 4;
  const int nf = mt > 2 && wgs(mt, 2) >= cus ? 2 : 1;
  return StreamPick{mt, nf, mt < 8 && nf == 1 && wgs(mt, 1) <= 2L * cus && d.d_ff >= 1024 ? 8 : 4};
}

hipError_t stream_gate_up(const moe_desc& d, const StreamPick& k, const GemmArgs& a, const PlanArgs& plan,
                          hipStream_t s, const char* name) {
  switch (k.mt) {
    case 1: return k.nf == 2 ? run_cols<FWD_GU, 2, 2>(d, a, plan, s, name) : run_cols<FWD_GU, 1, 4>(d, a, plan, s, name);
    case 2: return run_rows<FWD_GU, 2, 2, 4>(d, a, plan, s, name);
    case 4: return run_rows<FWD_GU, 4, 2, 4>(d, a, plan, s, name);
    default: return run_rows<FWD_GU, 8, 2, 2>(d, a, plan, s, name);
  }
}
hipError_t stream_down(const moe_desc& d, const StreamPick& k, const GemmArgs& a, hipStream_t s, const char* name) {
  const PlanArgs none{};
  switch (k.mt) {
    case 1: return k.nf == 2 ? run_cols<FWD_DOWN, 2, 4>(d, a, none, s, name) : run_cols<FWD_DOWN, 1, 4>(d, a, none, s, name);
    case 2:
      return k.depth == 8 ? run_rows<FWD_DOWN, 2, 1, 8>(d, a, none, s, name)
                          : run_rows<FWD_DOWN, 2, 1, 4>(d, a, none, s, name);
    case 4:
      return k.nf == 2      ? run_rows<FWD_DOWN, 4, 2, 4>(d, a, none, s, name)
             : k.depth == 8 ? run_rows<FWD_DOWN, 4, 1, 8>(d, a, none, s, name)
                            : run_rows<FWD_DOWN, 4, 1, 4>(d, a, none, s, name);
    default:
      return k.nf == 2 ? run_rows<FWD_DOWN, 8, 2, 4>(d, a, none, s, name)
                       : run_rows<FWD_DOWN, 8, 1, 4>(d, a, none, s, name);
  }
}

// The LDS tiles of dX take about 1.25 us per 64-deep step (the round trip of a K-tile's loads), 2 f / 64 of them in a
// chain, beside the weight gradient's stores in the same launch; streamed, dX reads its weights at the memory's rate, but
// before those stores. So it is streamed where the chain is longer than both together: up to 50 rows per group where it
// is less than 1.4 times as long, else up to 128 (and 256 where a shard's experts take every slot); at d_model >= 4096,
// whose pipelined tiles take a step in less time, only where it is twice as long. us, paired tiles -> dX and
// dW_gate, dW_up streamed, uniform and Zipf-skewed rows (one expert in every token is between them or gains more):
//   d = 1536, f = 8192, 5 groups, 14 rows: 318 -> 175, 317 -> 175;
//   d = 1024, f = 14336, 8 groups, 125 rows: 638 -> 499, 695 -> 492;
//   d = 1024, f = 2816, 16 groups: 6 rows 108 -> 86, 76 -> 75; 50 rows 124 -> 121, 141 -> 134;
//     not streamed: 99 rows 139 -> 142, 152 -> 149; 125 rows 147 -> 175, 161 -> 178;
//   8 of 32 experts, top-4, d = 1024, f = 2816: 20 rows 71 -> 55, 100 -> 73; not streamed: 125 rows 104 -> 91, 136 -> 167;
//   d = 768, f = 1408, 16 groups, not streamed: 36 rows 42 -> 47, 64 -> 46;
//   d = 4096, f = 14336, 2 groups, 50 rows: 478 -> 328, 563 -> 352;
//   d = 4096, f = 2816, 4 groups, not streamed: 24 rows 95 -> 93, 98 -> 106; 128 rows 144 -> 179, 144 -> 176.
// 16-row chunks up to 24 rows, 32 above (32 rows: 112 and 101 us with d = 1024).
// (The same kernel for dG|dU lost to the paired tiles wherever it was timed.)
int stream_dx_pick(const moe_desc& d) {
  const int G = d.local_count + d.n_shared;
  const GroupRows gr = group_rows(d);
  const double chain_us = 1.25 * (2.0 * d.d_ff / 64), bytes = 8.0 * d.d_ff * d.d_model * G;
  const double stream_us = 1.2 * bytes / 5.2e6 + 24;
  if (chain_us <= stream_us) return 0;
  if (d.d_model >= 4096 && chain_us < 2 * stream_us) return 0;
  if (chain_us < 1.4 * stream_us ? gr.most > 50 : gr.mean > 128 || gr.most > 256) return 0;
  return gr.mean <= 24 ? 1 : 2;
}
hipError_t stream_dx(const moe_desc& d, int mt, const GemmArgs& a, hipStream_t s, const char* name) {
  const int n_blocks = d.d_model / DX_COLS;
  const dim3 grid(grid_of(chunk_bound(d, 16 * mt) * n_blocks));
  KernelTimer kt(name, s);
  if (mt == 1) hipLaunchKernelGGL(stream_dx_kernel<1>, grid, dim3(64 * DX_KS), 0, s, a, n_blocks);
  else hipLaunchKernelGGL(stream_dx_kernel<2>, grid, dim3(64 * DX_KS), 0, s, a, n_blocks);
  return hipGetLastError();
}

}  // namespace pcmoe
