// bf16 MFMA GEMM for gfx950 with fused epilogues.
//
// Every dense contraction of the fine-tuning step (QKV, out-projection, MLP,
// LM / class head, ViT patch embedding; forward, input-gradient and
// weight-gradient products) runs through this kernel:
//   C[m, n] = sum_k A(m, k) B(n, k), bf16 operands, fp32 accumulation.
//
// Design (CDNA4):
//  * BT x BT x 64 block tile, BT = 128 or 64 (256 x 256 tiles are gemm256.hip),
//    4 wavefronts in a 2 x 2 grid, each with a BT/2 x BT/2 sub-tile of
//    v_mfma_f32_32x32x16_bf16 accumulators.  Two workgroups share a CU (64 KB
//    of LDS each), so one's prologue, barriers and epilogue overlap the
//    other's MFMAs: two stages of 128 x 128, or four of 64 x 64, which run
//    three K-tiles ahead where a grid of few tiles is bound by latency
//    (128 x 4096 x 4096: 32 us with two stages, 15.5 with four).
//  * What bounds it: a 64 x 64 wave tile reads its operands from LDS at the
//    LDS's full 128 bytes per clock when the MFMAs run at full rate, and a
//    128 x 128 tile needs 64 bytes per clock from L2, so long products stop at
//    about 1.0 PFLOP/s (8192 x 1024 x 4096: 68 us); the 256 x 256 kernel's ceiling
//    is higher, its grid coarser (gemm_plan below).
//  * Operands go HBM -> LDS directly with buffer_load ... lds (no VGPR
//    staging); out-of-range rows and the K tail are given an out-of-range buffer
//    offset and read as zeros.  K-contiguous tiles lie [row][k] in LDS,
//    M/N-contiguous ones [k][row] and are read with the transposing LDS read
//    (2048 x 2048 x 2048, both M/N-contiguous: 32 us; staged through registers and
//    transposed with byte permutes 65 us; K-contiguous 31 us).
//  * Unaligned operands are gathered with scalar loads (gemm_kernel_simple).
//  * Workgroups are renumbered so that consecutive tiles land on the same XCD
//    (the dispatcher deals workgroups round-robin over the 8 XCDs), then
//    ordered in groups of 8 tile-rows for L2 reuse of the B tiles.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int BK = 64;
constexpr int NT = 256;      // 4 wavefronts in a 2 x 2 grid
constexpr int KV = BK / 8;   // 16-byte chunks per K-row of a tile
constexpr uint32_t OOB = 0x80000000u;  // buffer offset that reads as zero

#define LDS_PTR(p) ((void __attribute__((address_space(3)))*)(p))


// Element offset of (row, chunk) in a swizzled tile.  A 128-bit LDS read is
// served 16 lanes at a time; the 16 lanes of a fragment read cover 16
// consecutive rows (8 even, 8 odd) at one logical chunk, so XOR-ing the chunk
// with bits 1..3 of the row spreads each parity class over all 8 positions.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int sw(int row, int chunk) { return row * BK + ((chunk ^ swz(row)) << 3); }

// Scalar gather of up to 8 consecutive bf16, zero beyond `n_ok`.
__device__ __forceinline__ u32x4 load_scalar8(const bf16* g, int n_ok) {
  uint16_t h[8];
  const uint16_t* gs = reinterpret_cast<const uint16_t*>(g);
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = (e < n_ok) ? gs[e] : (uint16_t)0;
  u32x4 r;
  r[0] = h[0] | ((uint32_t)h[1] << 16);
  r[1] = h[2] | ((uint32_t)h[3] << 16);
  r[2] = h[4] | ((uint32_t)h[5] << 16);
  r[3] = h[6] | ((uint32_t)h[7] << 16);
  return r;
}

// ---- K-contiguous operand through registers (scalar fallback path).
template <int ROWS>
struct KReg {
  static constexpr int N = ROWS * KV / NT;
  __device__ __forceinline__ static void load(const bf16* G, long ld, int r0, int nrows, int k0,
                                              int K, u32x4* regs) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int v = threadIdx.x + i * NT;
      int r = v / KV, kv = (v % KV) * 8;
      int gr = r0 + r, gk = k0 + kv;
      regs[i] = load_scalar8(G + (long)gr * ld + gk, (gr < nrows) ? min(8, K - gk) : 0);
    }
  }
  __device__ __forceinline__ static void store(bf16* S, const u32x4* regs) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int v = threadIdx.x + i * NT;
      *reinterpret_cast<u32x4*>(S + sw(v / KV, v % KV)) = regs[i];
    }
  }
};

// ---- M/N-contiguous operand: (row r, k) at G[k * ld + r].  Each thread owns
// 8 x 8 blocks (8 rows x 8 k), loaded as 8 row vectors and transposed in
// registers.  Block b = (rb = b / KV, kb = b % KV): eight consecutive lanes
// cover the eight k-blocks of one row block, so their global loads form
// 128-byte segments.
template <int ROWS>
struct MNReg {
  static constexpr int NB = (ROWS / 8) * KV;          // 8 x 8 blocks per tile
  static constexpr int NPT = (NB + NT - 1) / NT;      // blocks per thread
  static constexpr int N = 8 * NPT;
  __device__ __forceinline__ static void load(const bf16* G, long ld, int r0, int nrows, int k0,
                                              int K, u32x4* regs) {
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
      int b = threadIdx.x + j * NT;
      if (b >= NB) break;
      int rb = b / KV, kb = b % KV;
      int gr = r0 + rb * 8;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        int gk = k0 + kb * 8 + kk;
        const bf16* src = G + (long)gk * ld + gr;
        regs[8 * j + kk] = load_scalar8(src, (gk < K) ? max(0, min(8, nrows - gr)) : 0);
      }
    }
  }
  __device__ __forceinline__ static void store(bf16* S, const u32x4* regs) {
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
      int b = threadIdx.x + j * NT;
      if (b >= NB) break;
      int rb = b / KV, kb = b % KV;
      const u32x4* x = regs + 8 * j;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        u32x4 lo, hi;
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
          uint32_t a = x[2 * w2][w], c = x[2 * w2 + 1][w];
          lo[w2] = __builtin_amdgcn_perm(c, a, 0x05040100u);  // (a.lo, c.lo)
          hi[w2] = __builtin_amdgcn_perm(c, a, 0x07060302u);  // (a.hi, c.hi)
        }
        *reinterpret_cast<u32x4*>(S + sw(rb * 8 + 2 * w, kb)) = lo;
        *reinterpret_cast<u32x4*>(S + sw(rb * 8 + 2 * w + 1, kb)) = hi;
      }
    }
  }
};

template <int LAY, int ROWS>
struct Operand {
  using Reg = std::conditional_t<LAY == LAY_MN, MNReg<ROWS>, KReg<ROWS>>;
  u32x4 regs[Reg::N];
  __device__ __forceinline__ void fetch(const bf16* G, long ld, int r0, int nrows, int k0, int K) {
    Reg::load(G, ld, r0, nrows, k0, K, regs);
  }
  __device__ __forceinline__ void commit(bf16* S) { Reg::store(S, regs); }
};

// One K-tile on stage `cur`: barrier (the tile has landed and no wave still
// reads `nxt`), fragment reads for k-steps 0 and 1, MFMAs of step 0 while the
// reads of steps 2 and 3 are issued, then the next tile's loads into `nxt`
// (issued only after every read of `cur`, so no LDS read waits on them), then
// the MFMAs of steps 1 to 3 while those loads are in flight.
template <int TM, int TN, class OA, class OB>
__device__ __forceinline__ void ktile(floatx16 (&acc)[TM][TN], OA& opA, OB& opB, const GemmArgs& p,
                                      int m0, int n0, const bf16* cur, bf16* nxt, int kt, int nk,
                                      int BMr, int aoff, int boff, int fhalf, int fsw) {
  __syncthreads();
  const bool more = kt + 1 < nk;
  const bf16* As = cur + aoff;
  const bf16* Bs = cur + BMr * BK + boff;
  bf16x8 af[BK / 16][TM], bfv[BK / 16][TN];
#define SAT_RD(ks)                                                                    \
  {                                                                                   \
    const int pos = ((2 * (ks) + fhalf) ^ fsw) << 3;                                 \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) af[ks][i] =                        \
        *reinterpret_cast<const bf16x8*>(As + i * 32 * BK + pos);                     \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) bfv[ks][j] =                       \
        *reinterpret_cast<const bf16x8*>(Bs + j * 32 * BK + pos);                     \
  }
#define SAT_MM(ks)                                                                    \
  {                                                                                   \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                    \
    _Pragma("unroll") for (int j = 0; j < TN; ++j) acc[i][j] =                        \
        __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks][i], bfv[ks][j], acc[i][j], 0, 0, 0); \
  }
  SAT_RD(0);
  SAT_RD(1);
  __builtin_amdgcn_sched_barrier(0);
  SAT_MM(0);
  SAT_RD(2);
  SAT_RD(3);
  __builtin_amdgcn_sched_barrier(0);
  if (more) {
    opA.fetch(p.A, p.lda, m0, p.M, (kt + 1) * BK, p.K);
    opB.fetch(p.B, p.ldb, n0, p.N, (kt + 1) * BK, p.K);
  }
  __builtin_amdgcn_sched_barrier(0);
  SAT_MM(1);
  SAT_MM(2);
  SAT_MM(3);
#undef SAT_RD
#undef SAT_MM
  if (more) {
    opA.commit(nxt);
    opB.commit(nxt + BMr * BK);
  }
}

// Epilogue shared by both main loops, staged through LDS one 32-row slab per
// wave at a time, each wave in its own region: the accumulators (lane = column
// lane & 31, rows 8*(r/4) + 4*(lane/32) + r%4) are written with compile-time
// indices, then each lane reads back four consecutive columns, so that an
// output store is 16 (fp32) or 8 (bf16) bytes per lane where the rows are
// aligned for it (`vec`) and one element otherwise.
template <int BT, int EPI, int GE>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& p, floatx16 (&acc)[BT / 64][BT / 64],
                                              bf16* smem, int m0, int n0, int wave, int lane, bool vec) {
  constexpr int WT = BT / 2, TT = WT / 32;
  const int M = p.M, N = p.N;
  const int wm = wave >> 1, wn = wave & 1;
  constexpr int SP = WT + 4;       // fp32 pitch of a slab row
  constexpr int LR = WT / 4;       // lanes per row
  constexpr int RP = 64 / LR;      // rows per pass
  static_assert(4 * 32 * SP * 4 <= 2 * 2 * BT * BK * 2, "epilogue slabs exceed the LDS tile space");
  float* stage = reinterpret_cast<float*>(smem) + wave * 32 * SP;
  const int cl = 4 * (lane % LR);
  const int col = n0 + wn * WT + cl;
  const bool whole = vec && col + 3 < N;
  floatx4 bias = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (p.bias != nullptr && col + e < N && col + e >= p.bias_col0) bias[e] = p.bias[col + e - p.bias_col0];
  const bool csum_on = EPI == EPI_DGELU_BF16 && p.colsum_part != nullptr;
  __amdgpu_buffer_rsrc_t rsE;
  if constexpr (EPI == EPI_RESID_F32)
    rsE = __builtin_amdgcn_make_buffer_rsrc((void*)(p.resid + (long)m0 * p.ldr), (short)0, 0x7FFFFFFF, 0x00020000);
  if constexpr (EPI == EPI_DGELU_BF16)
    rsE = __builtin_amdgcn_make_buffer_rsrc((void*)(p.aux + (long)m0 * p.ldaux), (short)0, 0x7FFFFFFF, 0x00020000);
  floatx4 csum = {0.f, 0.f, 0.f, 0.f};  // this lane's columns over its rows of the wave's WT
#pragma unroll
  for (int i = 0; i < TT; ++i) {
    const int rowbase = m0 + wm * WT + i * 32;
    // residual / pre-activation loads of the whole slab first, in flight
    // together (buffer loads: rows past M and ragged columns read as zeros)
    u32x4 rv[EPI == EPI_RESID_F32 ? 32 / RP : 1];
    u32x2 uv[EPI == EPI_DGELU_BF16 ? 32 / RP : 1];
    if constexpr (EPI == EPI_RESID_F32 || EPI == EPI_DGELU_BF16) {
#pragma unroll
      for (int q = 0; q < 32 / RP; ++q) {
        const int row = rowbase + q * RP + lane / LR;
        const bool ok = whole && row < M;
        const long at = (long)(row - m0) * (EPI == EPI_RESID_F32 ? p.ldr * 4 : p.ldaux * 2) +
                        col * (EPI == EPI_RESID_F32 ? 4 : 2);
        if constexpr (EPI == EPI_RESID_F32)
          rv[q] = __builtin_amdgcn_raw_buffer_load_b128(rsE, ok ? (uint32_t)at : OOB, 0, 0);
        else
          uv[q] = __builtin_amdgcn_raw_buffer_load_b64(rsE, ok ? (uint32_t)at : OOB, 0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stage[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * SP + j * 32 + (lane & 31)] = acc[i][j][r];
    wait_lgkm0();
#pragma unroll
    for (int q = 0; q < 32 / RP; ++q) {
      const int rl = q * RP + lane / LR;
      const long row = rowbase + rl;
      if (row >= M || col >= N) continue;
      const floatx4 x = *reinterpret_cast<const floatx4*>(stage + rl * SP + cl) + bias;
      const long o = row * p.ldo + col;
      if (whole) {
        if (EPI == EPI_F32) {
          __builtin_nontemporal_store(x, reinterpret_cast<floatx4*>(reinterpret_cast<float*>(p.out) + o));
        } else if (EPI == EPI_RESID_F32) {
          __builtin_nontemporal_store(floatx4(__builtin_bit_cast(floatx4, rv[EPI == EPI_RESID_F32 ? q : 0]) + x), reinterpret_cast<floatx4*>(reinterpret_cast<float*>(p.out) + o));
        } else if (EPI == EPI_BF16) {
          __builtin_nontemporal_store(bf16x4{f2bf(x[0]), f2bf(x[1]), f2bf(x[2]), f2bf(x[3])}, reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(p.out) + o));
          if (p.out2 != nullptr && col >= p.gelu_col0)
            *reinterpret_cast<bf16x4*>(p.out2 + row * p.ldo2 + (col - p.gelu_col0)) =
                bf16x4{f2bf(gelu_t<GE>(x[0])), f2bf(gelu_t<GE>(x[1])), f2bf(gelu_t<GE>(x[2])),
                       f2bf(gelu_t<GE>(x[3]))};
        } else {
          const bf16x4 u = __builtin_bit_cast(bf16x4, uv[EPI == EPI_DGELU_BF16 ? q : 0]);
          bf16x4 y;
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = f2bf(x[e] * gelu_grad_t<GE>(bf2f(u[e])));
          __builtin_nontemporal_store(y, reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(p.out) + o));
          if (csum_on) csum += floatx4{bf2f(y[0]), bf2f(y[1]), bf2f(y[2]), bf2f(y[3])};
        }
        continue;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = col + e;
        if (c >= N) break;
        if (EPI == EPI_F32) {
          reinterpret_cast<float*>(p.out)[o + e] = x[e];
        } else if (EPI == EPI_RESID_F32) {
          reinterpret_cast<float*>(p.out)[o + e] = p.resid[row * p.ldr + c] + x[e];
        } else if (EPI == EPI_BF16) {
          reinterpret_cast<bf16*>(p.out)[o + e] = f2bf(x[e]);
          if (p.out2 != nullptr && c >= p.gelu_col0)
            p.out2[row * p.ldo2 + (c - p.gelu_col0)] = f2bf(gelu_t<GE>(x[e]));
        } else {
          const bf16 y = f2bf(x[e] * gelu_grad_t<GE>(bf2f(p.aux[row * p.ldaux + c])));
          reinterpret_cast<bf16*>(p.out)[o + e] = y;
          if (csum_on) csum[e] += bf2f(y);
        }
      }
    }
  }
  if (csum_on && m0 + wm * WT < M) {
    // the RP lane groups of a column, added in group order; one partial row per WT rows
    wait_lgkm0();
    *reinterpret_cast<floatx4*>(stage + (lane / LR) * WT + cl) = csum;
    wait_lgkm0();
    const int c = n0 + wn * WT + lane;
    if (lane < WT && c < N) {
      float v = stage[lane];
#pragma unroll
      for (int g = 1; g < RP; ++g) v += stage[g * WT + lane];
      p.colsum_part[(long)((m0 + wm * WT) / WT) * N + c] = v;
    }
  }
}

// Whether the epilogue's 4-column vectors are aligned in every array it touches, and a
// tile's rows of the residual / pre-activation stay within 32-bit buffer offsets.
template <int BT, int EPI>
__device__ __forceinline__ bool epilogue_vec(const GemmArgs& p) {
  auto al = [](const void* q, int b) { return (reinterpret_cast<uintptr_t>(q) & (b - 1)) == 0; };
  bool ok = p.ldo % 4 == 0 && al(p.out, (EPI == EPI_F32 || EPI == EPI_RESID_F32) ? 16 : 8);
  if (EPI == EPI_RESID_F32) ok = ok && p.ldr % 4 == 0 && al(p.resid, 16) && p.ldr < (1L << 31) / (BT * 4);
  if (EPI == EPI_BF16 && p.out2 != nullptr)
    ok = ok && p.ldo2 % 4 == 0 && p.gelu_col0 % 4 == 0 && al(p.out2, 8);
  if (EPI == EPI_DGELU_BF16) ok = ok && p.ldaux % 4 == 0 && al(p.aux, 8) && p.ldaux < (1L << 31) / (BT * 2);
  return ok;
}

// This workgroup's tile, with workgroups renumbered so that each XCD walks a
// contiguous range of the tile order and tiles ordered in groups of 8
// tile-rows.  With split-K the grid is (slice, tile) pairs, slice-major: the
// arguments are narrowed to the slice's K range and output block.
// kb: first k of the slice (gathered operands keep their pointers).
constexpr int LAY_TAPS = 2;     // A gathered per ConvTaps, B K-contiguous within a tap
constexpr int LAY_TAPS_MN = 3;  // B gathered per ConvTaps, its pixels along k (the weight gradient)
template <int BT, int ALAY, int BLAY>
__device__ __forceinline__ void tile_setup(GemmArgs& p, int& m0, int& n0, int& kb) {
  kb = 0;
  const int tiles_m = (p.M + BT - 1) / BT, tiles_n = (p.N + BT - 1) / BT;
  const int nwg = gridDim.x;
  int bid = blockIdx.x;
  if ((nwg & 7) == 0) bid = (bid & 7) * (nwg >> 3) + (bid >> 3);
  if (p.splitk > 1) {
    const int split = bid / (tiles_m * tiles_n);
    bid -= split * tiles_m * tiles_n;
    kb = split * p.splitk_kc;
    if (ALAY != LAY_TAPS) p.A += ALAY == LAY_K ? (long)kb : (long)kb * p.lda;
    if (ALAY != LAY_TAPS && BLAY != LAY_TAPS_MN) p.B += BLAY == LAY_K ? (long)kb : (long)kb * p.ldb;
    p.K = min(p.splitk_kc, p.K - kb);
    p.out = reinterpret_cast<float*>(p.out) + split * p.split_stride;
  }
  constexpr int G = 8;
  const int per_group = G * tiles_n;
  const int group = bid / per_group;
  const int first_m = group * G;
  const int gsize = min(tiles_m - first_m, G);
  const int in_g = bid - group * per_group;
  m0 = (first_m + in_g % gsize) * BT;
  n0 = (in_g / gsize) * BT;
}

// Block tile BT x BT x 64; 4 waves in a 2 x 2 grid, wave tile (BT/2) x (BT/2)
// made of 32 x 32 MFMA tiles.
template <int BT, int ALAY, int BLAY, int EPI, int GE>
__global__ __launch_bounds__(NT) void gemm_kernel_simple(GemmArgs p) {
  constexpr int WT = BT / 2, TT = WT / 32;
  constexpr int STAGE = 2 * BT * BK;  // bf16 elements per stage
  __shared__ __attribute__((aligned(1024))) bf16 smem[2 * STAGE];

  int m0, n0, kb;
  tile_setup<BT, ALAY, BLAY>(p, m0, n0, kb);
  const int K = p.K;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  Operand<ALAY, BT> opA;
  Operand<BLAY, BT> opB;

  floatx16 acc[TT][TT];
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = (K + BK - 1) / BK;
  opA.fetch(p.A, p.lda, m0, p.M, 0, K);
  opB.fetch(p.B, p.ldb, n0, p.N, 0, K);
  opA.commit(smem);
  opB.commit(smem + BT * BK);

  // fragment addressing: row (lane & 31) of each 32-row tile, logical chunk
  // 2 * ks + (lane >> 5), swizzled with swz(row) == swz(lane & 31)
  const int frow = lane & 31, fhalf = lane >> 5, fsw = swz(lane & 31);
  const int aoff = (wm * WT + frow) * BK, boff = (wn * WT + frow) * BK;
  for (int kt = 0; kt < nk; ++kt) {
    bf16* cur = smem + (kt & 1) * STAGE;
    bf16* nxt = smem + ((kt + 1) & 1) * STAGE;
    ktile<TT, TT>(acc, opA, opB, p, m0, n0, cur, nxt, kt, nk, BT, aoff, boff, fhalf, fsw);
  }
  __syncthreads();

  gemm_epilogue<BT, EPI, GE>(p, acc, smem, m0, n0, wave, lane, epilogue_vec<BT, EPI>(p));
}

// ------------------------------------------------------------------------
// Pipelined main loop (16-byte aligned operands), NS stages of one K-tile.
//
// Per K-tile k (stage k % NS): MFMAs of k-step 0, fragment reads of k-steps 2
// and 3, MFMAs of steps 1 and 2, then [wait for this wave's copies of tile
// k + 1, barrier], fragment reads of steps 0 and 1 of tile k + 1, the copies of
// tile k + NS into the stage that tile k just left, and only then the MFMAs of
// step 3 of tile k, so the matrix cores keep working across the barrier.  Waits
// are explicit s_waitcnt and the barrier carries no memory fence: a fence would
// also wait for the copies that are meant to stay in flight.  The tile
// stages are passed to the inlined helpers as __restrict__ pointers, which
// tells the compiler that reads of one stage never wait on copies into the
// others.  Tiles past the last one copy zeros, so the wait counts are constant.

typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
__device__ __forceinline__ bf16x4 ds_read_tr(const lds_bf16x4* __restrict__ p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(const_cast<lds_bf16x4*>(p));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, 0x7FFFFFFF, 0x00020000);
}

// One operand: its copies HBM -> LDS (16 bytes per lane, 1 KB per instruction)
// and its fragment reads.
//
// K-contiguous: [BT rows][64 k], chunk c of row r at c ^ swz(r) (see `sw`); a
// fragment is one 16-byte read per lane.
//
// M/N-contiguous: [64 k][BT rows] as it lies in memory, read with the
// transposing LDS read: 16 lanes hand in a 4 (k) x 16 (rows) block, lane
// 4 e + q the 8 bytes at k-row e, rows 4 q .. 4 q + 3, and each receives one
// row's four k values, so a fragment (8 k values) is two such reads.  The 16-byte
// chunks of a k-row are XOR-swizzled by 4 * (k % 4) (128 rows: a k-row is 256
// bytes) or 4 * (k / 2 % 2) (64 rows: two k-rows per 256 bytes), so that the
// 4 k-rows x 4 chunks that 32 lanes read at once are on distinct banks.
template <int LAY, int BT>
struct TileOp {
  static constexpr int NI = BT / 32;           // copy instructions per wave
  static constexpr int CPR = BT / 8;           // M/N-contiguous: chunks per k-row
  uint32_t off[NI];
  int kof[NI];                                 // first k of this lane's chunk, within the tile
  int fr[LAY == LAY_K ? 4 : 1];                // fragment offsets (K-contiguous: per k-step)
  __device__ __forceinline__ static int swz_mn(int k) { return BT == 128 ? 4 * (k & 3) : 4 * ((k >> 1) & 1); }
  __device__ __forceinline__ void init(long ld, int nrows, int wave, int w0) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (LAY == LAY_K) {
        const int row = (i * 4 + wave) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ swz(row);
        off[i] = row < nrows ? (uint32_t)(((long)row * ld + c * 8) * 2) : OOB;
        kof[i] = c * 8;
      } else {
        const int k = ((i * 4 + wave) * 64 + lane) / CPR;
        const int r = 8 * ((lane % CPR) ^ swz_mn(k));
        off[i] = r < nrows ? (uint32_t)(((long)k * ld + r) * 2) : OOB;
        kof[i] = k;
      }
    }
    if constexpr (LAY == LAY_K) {
      const int r = lane & 31;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) fr[ks] = (w0 + r) * BK + (((2 * ks + (lane >> 5)) ^ swz(r)) << 3);
    } else {
      // lane group G = lane / 16: k-rows 8 (G / 2) + e, rows 16 (G % 2) + 4 q
      const int G = lane >> 4, ll = lane & 15;
      const int k = 8 * (G >> 1) + (ll >> 2);
      const int c = w0 / 8 + 2 * (G & 1) + ((ll >> 1) & 1);
      fr[0] = k * BT + 8 * (c ^ swz_mn(k)) + 4 * (ll & 1);
    }
  }
  // src: the operand at (tile row 0, k = k0)
  __device__ __forceinline__ void copy(const bf16* src, int k0, int K, bf16* __restrict__ S, int wave) const {
    __amdgpu_buffer_rsrc_t rs = make_rsrc(src);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const uint32_t o = k0 + kof[i] < K ? off[i] : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(S + (i * 4 + wave) * 512), 16, o, 0, 0, 0);
    }
  }
  // 32 x 16 fragment of rows w0 + 32 sub .. + 31 and k-step ks
  __device__ __forceinline__ bf16x8 frag(const bf16* __restrict__ S, int sub, int ks) const {
    if constexpr (LAY == LAY_K) {
      return *reinterpret_cast<const bf16x8*>(S + fr[ks] + sub * 32 * BK);
    } else {
      // rows + 32: chunk + 4.  With 128 rows the swizzle is 4 (k % 4), an XOR of
      // bits 2 - 3 of the chunk index, so the sum is formed before the XOR;
      // the wave's rows start at a multiple of 64 (128-row tiles) or 32.
      const int o = (BT == 128 && sub) ? fr[0] ^ 32 : fr[0];
      const bf16x4 lo = ds_read_tr((const lds_bf16x4*)LDS_PTR(const_cast<bf16*>(S) + o + ks * 16 * BT));
      const bf16x4 hi = ds_read_tr((const lds_bf16x4*)LDS_PTR(const_cast<bf16*>(S) + hi4(o) + ks * 16 * BT));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  }
  // k + 4: the same k % 4, and (64 rows) the same k / 2 % 2
  __device__ __forceinline__ static int hi4(int o) { return o + 4 * BT; }
};

// The gathered operand (a 3 x 3 convolution without its im2col matrix, which held the
// input nine times, and without the nine-fold fp32 column gradient of the input
// gradient): 12 ResNet blocks at batch 64, 19.9 ms per step through the matrices,
// 18.3 gathered; 12544 x 512 x 4608: 79 us where im2col and product took 33 + 67.
// The K-contiguous tile layout and fragments, each copied
// 16-byte piece from its pixel's place in the tensor.  A K-tile lies in one tap, so
// a copy adds one uniform offset per tap and checks the pixel's coordinates.
template <int BT>
struct TileOp<LAY_TAPS, BT> : TileOp<LAY_K, BT> {
  using Base = TileOp<LAY_K, BT>;
  int hw[Base::NI];  // h0 (low 16 bits) and w0 of this lane's row; far outside past M
  int a, b, c0;      // tap and first channel of the next K-tile
  __device__ __forceinline__ void init_taps(const GemmArgs& p, int m0, int kb, int wave, int w0) {
    Base::init(0, 0, wave, w0);  // fragment offsets
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < Base::NI; ++i) {
      const int row = (i * 4 + wave) * 8 + (lane >> 3);
      const int m = m0 + row;
      const int j = m % p.cv.oW, q = m / p.cv.oW;
      const int h0 = q % p.cv.oH * p.cv.stride + p.cv.org, v0 = j * p.cv.stride + p.cv.org;
      const int n = q / p.cv.oH;
      Base::off[i] = (uint32_t)((((n * p.cv.H + h0) * p.cv.W + v0) * p.cv.C + Base::kof[i]) * 2);
      hw[i] = m < p.M ? (h0 & 0xFFFF) | (int)((uint32_t)v0 << 16) : (int)0x80008000u;
    }
    const int tap = kb / p.cv.C;
    c0 = kb - tap * p.cv.C;
    a = tap / p.cv.ksize;
    b = tap - a * p.cv.ksize;
  }
  // the next K-tile of A (k0: its first k in the slice), then on to the tile after it
  __device__ __forceinline__ void copy_taps(const GemmArgs& p, int k0, int K, bf16* __restrict__ S, int wave) {
    __amdgpu_buffer_rsrc_t rs = make_rsrc(p.A);
    const int da = p.cv.sgn * a, db = p.cv.sgn * b;
    const uint32_t step = (uint32_t)(((da * p.cv.W + db) * p.cv.C + c0) * 2);
#pragma unroll
    for (int i = 0; i < Base::NI; ++i) {
      const int h = (int)(short)hw[i] + da, w = (hw[i] >> 16) + db;
      const bool ok = (uint32_t)h < (uint32_t)p.cv.H && (uint32_t)w < (uint32_t)p.cv.W && k0 < K;
      const uint32_t o = ok ? Base::off[i] + step : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(S + (i * 4 + wave) * 512), 16, o, 0, 0, 0);
    }
    c0 += BK;
    if (c0 == p.cv.C) {
      c0 = 0;
      if (++b == p.cv.ksize) {
        b = 0;
        ++a;
      }
    }
  }
};

// The weight gradient's gathered operand: the M/N-contiguous tile layout and
// fragments; k-row = one output pixel, columns = BT channels of one tap.  Every lane
// keeps its pieces' pixels and moves them on by a K-tile of 64 pixels: 64 = (dn
// images, di rows, dj columns), one carry each.  (12 ResNet blocks at batch 64:
// rebuilding the im2col matrix for these products took 0.7 ms of the step.)
template <int BT>
struct TileOp<LAY_TAPS_MN, BT> : TileOp<LAY_MN, BT> {
  using Base = TileOp<LAY_MN, BT>;
  int pn[Base::NI], pi[Base::NI], pj[Base::NI];
  int a, b;             // this tile's tap
  int dn, di, dj;
  __device__ __forceinline__ void init_taps(const GemmArgs& p, int n0, int kb, int wave, int w0) {
    Base::init(0, 0, wave, w0);  // fragment offsets, k of this lane's pieces
    const int lane = threadIdx.x & 63;
    const int tap = n0 / p.cv.C, c0 = n0 - tap * p.cv.C;
    a = tap / p.cv.ksize;
    b = tap - a * p.cv.ksize;
#pragma unroll
    for (int i = 0; i < Base::NI; ++i) {
      const int m = kb + Base::kof[i];
      const int q = m / p.cv.oW;
      pj[i] = m - q * p.cv.oW;
      pn[i] = q / p.cv.oH;
      pi[i] = q - pn[i] * p.cv.oH;
      Base::off[i] = (uint32_t)((c0 + 8 * ((lane % Base::CPR) ^ Base::swz_mn(Base::kof[i]))) * 2);
    }
    dn = BK / (p.cv.oH * p.cv.oW);
    const int rem = BK - dn * p.cv.oH * p.cv.oW;
    di = rem / p.cv.oW;
    dj = rem - di * p.cv.oW;
  }
  __device__ __forceinline__ void copy_taps(const GemmArgs& p, int k0, int K, bf16* __restrict__ S, int wave) {
    __amdgpu_buffer_rsrc_t rs = make_rsrc(p.B);
#pragma unroll
    for (int i = 0; i < Base::NI; ++i) {
      const int h = pi[i] * p.cv.stride + p.cv.org + a, w = pj[i] * p.cv.stride + p.cv.org + b;
      const bool ok = (uint32_t)h < (uint32_t)p.cv.H && (uint32_t)w < (uint32_t)p.cv.W && k0 + Base::kof[i] < K;
      const uint32_t o =
          ok ? (uint32_t)(((pn[i] * p.cv.H + h) * p.cv.W + w) * p.cv.C * 2) + Base::off[i] : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(S + (i * 4 + wave) * 512), 16, o, 0, 0, 0);
      pj[i] += dj;
      const int cj = pj[i] >= p.cv.oW ? 1 : 0;
      pj[i] -= cj ? p.cv.oW : 0;
      pi[i] += di + cj;
      const int ci = pi[i] >= p.cv.oH ? 1 : 0;
      pi[i] -= ci ? p.cv.oH : 0;
      pn[i] += dn + ci;
    }
  }
};

template <int BT, int AL, int BL>
__device__ __forceinline__ void frag_read(bf16x8 (&af)[2][BT / 64], bf16x8 (&bfv)[2][BT / 64],
                                          const TileOp<AL, BT>& A, const TileOp<BL, BT>& B,
                                          const bf16* __restrict__ stage, int ks0) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < BT / 64; ++i) af[h][i] = A.frag(stage, i, ks0 + h);
#pragma unroll
    for (int j = 0; j < BT / 64; ++j) bfv[h][j] = B.frag(stage + BT * BK, j, ks0 + h);
  }
}

// Copies of K-tile t into stage S (past the last tile every chunk is past K).
// GA, GB: the operands at (tile row 0, k = 0); called for t = 0, 1, 2, ... in order.
template <int BT, int AL, int BL>
__device__ __forceinline__ void tile_copy(TileOp<AL, BT>& A, TileOp<BL, BT>& B, const GemmArgs& p,
                                          const bf16* GA, const bf16* GB, int t, int nk, int K,
                                          bf16* __restrict__ S, int wave) {
  const int k0 = min(t, nk) * BK;
  if constexpr (AL == LAY_TAPS) {
    const bf16* src = GB + (long)(A.a * p.cv.ksize + A.b) * p.cv.b_tap + A.c0;
    B.copy(src, k0, K, S + BT * BK, wave);
    A.copy_taps(p, k0, K, S, wave);
  } else if constexpr (BL == LAY_TAPS_MN) {
    A.copy(GA + (long)k0 * p.lda, k0, K, S, wave);
    B.copy_taps(p, k0, K, S + BT * BK, wave);
  } else {
    A.copy(GA + (AL == LAY_K ? (long)k0 : (long)k0 * p.lda), k0, K, S, wave);
    B.copy(GB + (BL == LAY_K ? (long)k0 : (long)k0 * p.ldb), k0, K, S + BT * BK, wave);
  }
}

template <int TT>
__device__ __forceinline__ void mfma_step(floatx16 (&acc)[TT][TT], const bf16x8 (&af)[TT],
                                          const bf16x8 (&bfv)[TT]) {
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfv[j], acc[i][j], 0, 0, 0);
}

template <int BT, int NS, int ALAY, int BLAY, int EPI, int GE>
__global__ __launch_bounds__(NT, 2) void gemm_tile_kernel(GemmArgs p) {
  constexpr int WT = BT / 2, TT = WT / 32;
  constexpr int STAGE = 2 * BT * BK;
  __shared__ __attribute__((aligned(1024))) bf16 smem[NS * STAGE];

  int m0, n0, kb;
  tile_setup<BT, ALAY, BLAY>(p, m0, n0, kb);
  const int K = p.K;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const bf16* GA = p.A + (ALAY == LAY_K ? (long)m0 * p.lda : (long)m0);  // (gathered operands: unused)
  const bf16* GB = p.B + (BLAY == LAY_K ? (long)n0 * p.ldb : (long)n0);
  TileOp<ALAY, BT> A;
  TileOp<BLAY, BT> B;
  if constexpr (ALAY == LAY_TAPS) A.init_taps(p, m0, kb, wave, wm * WT);
  else A.init(p.lda, p.M - m0, wave, wm * WT);
  if constexpr (BLAY == LAY_TAPS_MN) B.init_taps(p, n0, kb, wave, wn * WT);
  else B.init(p.ldb, p.N - n0, wave, wn * WT);
  constexpr int NC = 2 * TileOp<LAY_K, BT>::NI;  // copies per wave and K-tile

  floatx16 acc[TT][TT];
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = (K + BK - 1) / BK;
#pragma unroll
  for (int t = 0; t < NS; ++t) tile_copy(A, B, p, GA, GB, t, nk, K, smem + t * STAGE, wave);
  wait_vm_lgkm0<(NS - 1) * NC>();
  cta_barrier();
  bf16x8 f01a[2][TT], f01b[2][TT], f23a[2][TT], f23b[2][TT];
  frag_read(f01a, f01b, A, B, smem, 0);

  int st = 0;
  for (int kt = 0; kt < nk; ++kt) {
    bf16* cur = smem + st * STAGE;
    st = st + 1 == NS ? 0 : st + 1;
    __builtin_amdgcn_sched_barrier(0);
    mfma_step<TT>(acc, f01a[0], f01b[0]);
    frag_read(f23a, f23b, A, B, cur, 2);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step<TT>(acc, f01a[1], f01b[1]);
    mfma_step<TT>(acc, f23a[0], f23b[0]);
    // tile kt + 1 resident, this wave's reads of tile kt done
    wait_vm_lgkm0<(NS - 2) * NC>();
    cta_barrier();
    frag_read(f01a, f01b, A, B, smem + st * STAGE, 0);
    tile_copy(A, B, p, GA, GB, kt + NS, nk, K, cur, wave);
    __builtin_amdgcn_sched_barrier(0);
    mfma_step<TT>(acc, f23a[1], f23b[1]);
  }
  wait_vm_lgkm0<0>();  // the zero-filling copies past the last tile
  __syncthreads();
  gemm_epilogue<BT, EPI, GE>(p, acc, smem, m0, n0, wave, lane, epilogue_vec<BT, EPI>(p));
}

template <int BT, int ALAY, int BLAY, int EPI, int GE>
hipError_t launch5(const GemmArgs& a, bool vec, hipStream_t s) {
  dim3 grid((unsigned)(sat_cdiv(a.M, BT) * sat_cdiv(a.N, BT) * std::max(a.splitk, 1)));
  if (vec) hipLaunchKernelGGL((gemm_tile_kernel<BT, BT == 64 ? 4 : 2, ALAY, BLAY, EPI, GE>), grid, dim3(NT), 0, s, a);
  else hipLaunchKernelGGL((gemm_kernel_simple<BT, ALAY, BLAY, EPI, GE>), grid, dim3(NT), 0, s, a);
  return hipGetLastError();
}

template <int BT, int ALAY, int BLAY, int EPI>
hipError_t launch4(const GemmArgs& a, bool vec, hipStream_t s) {
  if constexpr (EPI == EPI_BF16 || EPI == EPI_DGELU_BF16) {
    if (a.gelu_erf) return launch5<BT, ALAY, BLAY, EPI, 1>(a, vec, s);
  }
  return launch5<BT, ALAY, BLAY, EPI, 0>(a, vec, s);
}

template <int ALAY, int BLAY, int EPI>
hipError_t launch3(const GemmArgs& a, int bt, bool vec, hipStream_t s) {
  if (bt == 64) return launch4<64, ALAY, BLAY, EPI>(a, vec, s);
  return launch4<128, ALAY, BLAY, EPI>(a, vec, s);
}

template <int ALAY, int BLAY>
hipError_t launch2(const GemmArgs& a, int epi, int bt, bool vec, hipStream_t s) {
  switch (epi) {
    case EPI_F32: return launch3<ALAY, BLAY, EPI_F32>(a, bt, vec, s);
    case EPI_RESID_F32: return launch3<ALAY, BLAY, EPI_RESID_F32>(a, bt, vec, s);
    case EPI_BF16: return launch3<ALAY, BLAY, EPI_BF16>(a, bt, vec, s);
    case EPI_DGELU_BF16: return launch3<ALAY, BLAY, EPI_DGELU_BF16>(a, bt, vec, s);
  }
  return hipErrorInvalidValue;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// Whether both operands can be copied in 16-byte pieces.  Along K a partial
// piece would mix in values past K, so K must be a multiple of 8; along M / N a
// partial piece only feeds output rows / columns that are never stored, so it
// suffices that the rows are long enough (ld >= M or N rounded up to 8) to stay
// in bounds.  A tile's rows (128, or 64 k-rows) must stay within 32-bit buffer offsets.
bool tile_vec(const GemmArgs& a, int alay, int blay) {
  auto r8 = [](long x) { return (x + 7) / 8 * 8; };
  auto fits = [](long ld, int lay) { return ld < (1L << 31) / (lay == LAY_K ? 2 * 128 : 2 * BK); };
  return aligned16(a.A) && aligned16(a.B) && a.lda % 8 == 0 && a.ldb % 8 == 0 && fits(a.lda, alay) && fits(a.ldb, blay) &&
         (alay == LAY_K ? a.K % 8 == 0 : a.lda >= r8(a.M)) &&
         (blay == LAY_K ? a.K % 8 == 0 : a.ldb >= r8(a.N));
}

hipError_t launch_tiles(const GemmArgs& a, int bt, int alay, int blay, int epi, hipStream_t s) {
  const bool vec = tile_vec(a, alay, blay);
  if (alay == LAY_K && blay == LAY_K) return launch2<LAY_K, LAY_K>(a, epi, bt, vec, s);
  if (alay == LAY_K && blay == LAY_MN) return launch2<LAY_K, LAY_MN>(a, epi, bt, vec, s);
  if (alay == LAY_MN && blay == LAY_K) return launch2<LAY_MN, LAY_K>(a, epi, bt, vec, s);
  return launch2<LAY_MN, LAY_MN>(a, epi, bt, vec, s);
}

}  // namespace

bool gemm_tail_split(int M, int N, int K, int smax, int* M1, int* S, int* kc) {
  const long mt = sat_cdiv(M, 256), nt = sat_cdiv(N, 256), tiles = mt * nt;
  if (tiles <= 256 || tiles % 256 == 0 || nt > 256) return false;
  // head: the rows whose tiles fill whole rounds of 256 workgroups
  const long mh = 256 * (tiles / 256) / nt;
  if (mh <= 0 || mh >= mt) return false;
  const int m2 = M - (int)mh * 256;
  int c = 0;
  const int s = gemm_splitk(m2, N, K, &c, smax);
  if (s <= 1) return false;
  // the same estimate as gemm_splitk, in K-tile steps of one tile: the head's
  // rounds, the tail's slices and their reduction, against every round unsplit
  const double kt = (double)sat_cdiv(K, 64);
  const double head = (double)((mh * nt + 255) / 256) * kt;
  const double tail = (double)((sat_cdiv(m2, 256) * nt * s + 255) / 256) * (c / 64) +
                      (double)(s + 1) * m2 * N * 4.0 / 9e6;
  if (head + tail >= (double)((tiles + 255) / 256) * kt) return false;
  *M1 = (int)mh * 256;
  *S = s;
  *kc = c;
  return true;
}

long gemm_tail_ws_elems(int M, int N, int K, int smax) {
  int m1 = 0, s = 0, c = 0;
  return gemm_tail_split(M, N, K, smax, &m1, &s, &c) ? (long)s * (M - m1) * N : 0;
}

namespace {

// Estimated time (us) of an [M, N] product of depth K in S slices on tiles of
// bt x bt, from measured products (random operands, 0.5 to 300 GFLOP):
//  * 256: rounds of one tile per CU; a K-tile of 64 takes 1.5 us, a tile's
//    prologue and epilogue 6.5 us (1.6 with an M/N-contiguous operand);
//  * 128: two tiles share a CU; 0.39 us per K-tile and 4.5 us per tile of a CU,
//    0.62 and 5 us for a CU that has one;
//  * 64: 0.215 us per K-tile and 0.6 us per tile of a CU (1.8 past 16 tiles, where
//    the outputs stream to memory), 3 us in all;
//  * the reduction of the slices: 4 us and its traffic at 6 TB/s.
// Over 32 products of 0.004 to 960 GFLOP in both layouts single estimates are off by up to
// half (worst with operands past the Infinity Cache, which gemm_plan sets apart); the tile
// they choose is within 8 % of the fastest unsplit one.
double gemm_estimate(int bt, bool mn, long M, long N, long K, int S) {
  const double kt = (double)((sat_cdiv(K, S) + 63) / 64);
  const long n = ((long)sat_cdiv(M, bt) * sat_cdiv(N, bt) * S + 255) / 256;
  const double red = S > 1 ? 4.0 + (S + 1.0) * M * N * 4.0 / 6e6 : 0.0;
  if (bt == 256) return n * ((mn ? 1.6 : 1.5) * kt + 6.5) + red;
  if (bt == 128) return (n == 1 ? 0.62 * kt + 5.0 : n * (0.39 * kt + 4.5)) + red;
  return 3.0 + n * ((n > 16 ? 1.8 : 0.6) + 0.215 * kt) + red;
}

struct GemmPlan {
  int bt;  // 256: gemm256.hip, else the BT x BT kernel
  int S;   // K slices, kc deep
  int kc;
  double us;
};

// Which kernel runs a product, and in how many K slices.  Fewer than 256 tiles
// of 256 x 256 leave CUs idle, and the last of a few rounds is mostly empty:
// 128 x 128 tiles then win on a finer grid and on two workgroups per CU whose
// epilogues and main loops overlap (8192 x 768 x 3072: 60 us as two slices of
// 256 x 256 tiles and a reduction, 47 us; 1285 x 5120 x 1280: 30 and 26 us), 64 x 64
// tiles on a grid that would leave most CUs without a 128 x 128 tile
// (128 x 4096 x 4096: 48 and 16 us; 64 x 64 x 512: 8.5 and 4.5 us).
// Large products keep the 256 x 256 kernel: it moves half the bytes per FLOP
// (4096 x 28672 x 4096: 720 us, 128 x 128 1040 us).  So do products whose
// operands exceed the 256 MB Infinity Cache, where each re-read of a panel comes
// from HBM (the LM head's 8192 x 768 x 50264 input gradient: 630 us in eight
// slices of 256 x 256 tiles, 1070 us in two of 128 x 128).  bf16 outputs weigh the
// smaller tiles 15 % heavier: with cold operands and outputs their many small
// tiles lose what they win on warm ones (8192 x 2304 x 768 in a step: 47 us
// on 256 x 256 tiles, 60 on 128 x 128; called alone 46 and 45).
//
// Slices: an fp32-output product on K-contiguous operands splits as
// gemm_splitk says (never in more slices, so its workspace holds them), or
// not at all where unsplit 128 x 128 or 64 x 64 tiles fill the chip and are
// faster.  With an M/N-contiguous operand it splits where the workspace holds it.
GemmPlan gemm_plan(const GemmArgs& a, int alay, int blay, int epi) {
  const bool kl = alay == LAY_K && blay == LAY_K;
  const bool may_split = (epi == EPI_F32 || epi == EPI_RESID_F32) && a.splitk_ws != nullptr;
  const bool big = ((double)a.M + a.N) * a.K * 2.0 > 256e6;
  GemmPlan best{128, 1, 0, 1e30};
  auto consider = [&](int bt, int S, int kc) {
    const double us = gemm_estimate(bt, !kl, a.M, a.N, a.K, S) *
                      (bt != 256 && (epi == EPI_BF16 || epi == EPI_DGELU_BF16) ? 1.15 : 1.0);
    if (us < best.us) best = GemmPlan{bt, S, kc, us};
  };
  auto slices = [&](int bt, int smax) {
    for (int S = 2; S <= smax; ++S) {
      const int kc = (sat_cdiv(a.K, S) + BK - 1) / BK * BK;
      consider(bt, sat_cdiv(a.K, kc), kc);
    }
  };
  int kc256 = 0;
  int S256 = may_split && kl ? gemm_splitk(a.M, a.N, a.K, &kc256, a.splitk_max) : 1;
  if (S256 > 1 && (long)S256 * a.M * a.N > a.splitk_ws_elems) S256 = 1;
  GemmArgs b = a;
  if (S256 > 1) {
    b.out = a.splitk_ws;
    b.ldo = a.N;
    b.bias = nullptr;
    b.resid = nullptr;
    b.splitk = S256;
    b.splitk_kc = kc256;
    b.split_stride = (long)a.M * a.N;
    if (gemm256_eligible(b, LAY_K, LAY_K, EPI_F32)) {
      consider(256, S256, kc256);
      if (big) return best;
      slices(128, S256);
      slices(64, S256);
    } else {
      S256 = 1;
    }
  } else if (may_split && !kl && a.K >= 1024 && tile_vec(a, alay, blay)) {
    const long fit = a.splitk_ws_elems / std::max(1L, (long)a.M * a.N);
    const int smax = (int)std::min<long>(std::min<long>(a.splitk_max > 0 ? a.splitk_max : 16, a.K / 512), fit);
    slices(128, smax);
    slices(64, smax);
  }
  if (S256 <= 1 && big && gemm256_eligible(a, alay, blay, epi)) {
    consider(256, 1, 0);
    return best;
  }
  for (int bt : {128, 64})
    if (S256 <= 1 || (long)sat_cdiv(a.M, bt) * sat_cdiv(a.N, bt) >= 256) consider(bt, 1, 0);
  if (S256 <= 1 && gemm256_eligible(a, alay, blay, epi)) consider(256, 1, 0);
  return best;
}

}  // namespace

bool gemm_conv_eligible(const GemmArgs& a) {
  const ConvTaps& v = a.cv;
  const long lim = 1L << 31;
  return v.C % BK == 0 && a.K == v.ksize * v.ksize * v.C && aligned16(a.A) && aligned16(a.B) &&
         a.ldb % 8 == 0 && v.b_tap % 8 == 0 && v.H < (1 << 14) && v.W < (1 << 14) && v.oH < (1 << 14) &&
         v.oW < (1 << 14) && a.M % (v.oH * v.oW) == 0 &&
         (long)(a.M / (v.oH * v.oW)) * v.H * v.W * v.C * 2 < lim && 128L * a.ldb * 2 < lim;
}

bool gemm_conv_wgrad_eligible(const GemmArgs& a) {
  const ConvTaps& v = a.cv;
  const long lim = 1L << 31;
  return v.C % 64 == 0 && a.N == v.ksize * v.ksize * v.C && aligned16(a.A) && aligned16(a.B) &&
         a.lda % 8 == 0 && a.lda >= (a.M + 7) / 8 * 8 && a.K % (v.oH * v.oW) == 0 &&
         (long)(a.K / (v.oH * v.oW)) * v.H * v.W * v.C * 2 < lim && 64L * a.lda * 2 < lim;
}

namespace {

// A gathered product runs on 128 x 128 (wide: allowed) or 64 x 64 tiles, unsplit or in
// at most smax K slices where the workspace holds them, by the same estimate.
template <int AL, int BL>
hipError_t launch_conv(const GemmArgs& a, bool wide, long smax, hipStream_t s) {
  GemmPlan best{64, 1, 0, 1e30};
  const long fit = a.splitk_ws != nullptr ? a.splitk_ws_elems / std::max(1L, (long)a.M * a.N) : 1;
  smax = std::max(1L, std::min({smax, (long)a.K / 512, fit}));
  for (int bt : {128, 64})
    for (int S = 1; S <= (int)smax; ++S) {
      if (bt == 128 && !wide) break;
      const int kc = (sat_cdiv(a.K, S) + BK - 1) / BK * BK;
      const int Se = sat_cdiv(a.K, kc);
      const double us = gemm_estimate(bt, false, a.M, a.N, a.K, Se);
      if (us < best.us) best = GemmPlan{bt, Se, kc, us};
    }
  GemmArgs b = a;
  if (best.S > 1) {
    b.out = a.splitk_ws;
    b.ldo = a.N;
    b.splitk = best.S;
    b.splitk_kc = best.kc;
    b.split_stride = (long)a.M * a.N;
  }
  const dim3 grid((unsigned)(sat_cdiv(a.M, best.bt) * sat_cdiv(a.N, best.bt) * best.S));
  if (best.bt == 128) hipLaunchKernelGGL((gemm_tile_kernel<128, 2, AL, BL, EPI_F32, 0>), grid, dim3(NT), 0, s, b);
  else hipLaunchKernelGGL((gemm_tile_kernel<64, 4, AL, BL, EPI_F32, 0>), grid, dim3(NT), 0, s, b);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || best.S <= 1) return e;
  return launch_splitk_reduce(a.splitk_ws, best.S, b.split_stride, a.M, a.N,
                              reinterpret_cast<float*>(a.out), a.ldo, nullptr, 0, nullptr, 0, s);
}

}  // namespace

hipError_t launch_gemm_conv(const GemmArgs& a, hipStream_t s) {
  if (!gemm_conv_eligible(a)) return hipErrorInvalidValue;
  return launch_conv<LAY_TAPS, LAY_K>(a, true, 16, s);
}

hipError_t launch_gemm_conv_wgrad(const GemmArgs& a, hipStream_t s) {
  if (!gemm_conv_wgrad_eligible(a)) return hipErrorInvalidValue;
  // a tile's columns lie in one tap
  return launch_conv<LAY_MN, LAY_TAPS_MN>(a, a.cv.C % 128 == 0, a.splitk_max > 0 ? a.splitk_max : 16, s);
}

int gemm_colsum_rows(const GemmArgs& a) {
  const GemmPlan p = gemm_plan(a, LAY_K, LAY_K, EPI_DGELU_BF16);
  return p.bt / 2;
}

int gemm_planned_tile(const GemmArgs& a, int alay, int blay, int epi, int* slices) {
  const GemmPlan p = gemm_plan(a, alay, blay, epi);
  *slices = p.S;
  return p.bt == 256 || tile_vec(a, alay, blay) ? p.bt : -p.bt;
}

hipError_t launch_gemm(const GemmArgs& a, int alay, int blay, int epi, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (a.K <= 0) return hipErrorInvalidValue;
  if (epi == EPI_ADAMW)  // the optimizer epilogue exists in the 256 x 256 kernel only
    return gemm256_eligible(a, alay, blay, epi) ? launch_gemm256(a, alay, blay, epi, s)
                                                : hipErrorInvalidValue;
  // more than 256 tiles with a mostly empty last round: whole rounds of rows
  // unsplit, the remaining rows split-K into the workspace
  if ((epi == EPI_F32 || epi == EPI_RESID_F32) && alay == LAY_K && blay == LAY_K &&
      a.splitk_ws != nullptr && !a.no_tail_split) {
    int M1 = 0, S = 0, kc = 0;
    if (gemm_tail_split(a.M, a.N, a.K, a.splitk_max, &M1, &S, &kc) &&
        (long)S * (a.M - M1) * a.N <= a.splitk_ws_elems) {
      GemmArgs h = a;
      h.M = M1;
      GemmArgs t = a;
      t.A = a.A + (long)M1 * a.lda;
      t.M = a.M - M1;
      t.out = a.splitk_ws;
      t.ldo = a.N;
      t.bias = nullptr;
      t.resid = nullptr;
      t.splitk = S;
      t.splitk_kc = kc;
      t.split_stride = (long)t.M * a.N;
      if (gemm256_eligible(h, LAY_K, LAY_K, epi) && gemm256_eligible(t, LAY_K, LAY_K, EPI_F32)) {
        hipError_t e = launch_gemm256(h, LAY_K, LAY_K, epi, s);
        if (e != hipSuccess) return e;
        e = launch_gemm256(t, LAY_K, LAY_K, EPI_F32, s);
        if (e != hipSuccess) return e;
        return launch_splitk_reduce(a.splitk_ws, S, t.split_stride, t.M, a.N,
                                    reinterpret_cast<float*>(a.out) + (long)M1 * a.ldo, a.ldo,
                                    a.bias, a.bias_col0,
                                    epi == EPI_RESID_F32 ? a.resid + (long)M1 * a.ldr : nullptr,
                                    a.ldr, s);
      }
    }
  }
  const GemmPlan plan = gemm_plan(a, alay, blay, epi);
  if (plan.S <= 1)
    return plan.bt == 256 ? launch_gemm256(a, alay, blay, epi, s)
                          : launch_tiles(a, plan.bt, alay, blay, epi, s);
  // K slices into the caller's workspace, then one reduction that applies bias
  // and residual
  GemmArgs b = a;
  b.out = a.splitk_ws;
  b.ldo = a.N;
  b.bias = nullptr;
  b.resid = nullptr;
  b.splitk = plan.S;
  b.splitk_kc = plan.kc;
  b.split_stride = (long)a.M * a.N;
  const hipError_t e = plan.bt == 256 ? launch_gemm256(b, alay, blay, EPI_F32, s)
                                      : launch_tiles(b, plan.bt, alay, blay, EPI_F32, s);
  if (e != hipSuccess) return e;
  return launch_splitk_reduce(a.splitk_ws, plan.S, b.split_stride, a.M, a.N,
                              reinterpret_cast<float*>(a.out), a.ldo, a.bias, a.bias_col0,
                              epi == EPI_RESID_F32 ? a.resid : nullptr, a.ldr, s);
}
