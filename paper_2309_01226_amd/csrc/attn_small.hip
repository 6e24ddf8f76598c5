// Attention forward and backward for 64-, 80- and 128-wide heads (GPT-2-style
// decoders, ViT-H/14), causal or bidirectional, on gfx950 MFMA
// (v_mfma_f32_32x32x16_bf16, bf16 operands, fp32 accumulation).
//
// Forward: O = softmax(scale * Q K^T + mask) V per head and the per-query
// natural-log log-sum-exp.  Backward: dV = P^T dO, dP = dO V^T,
// dS = P * (dP - delta), dK = scale dS^T Q, dQ = scale dS K, with P
// recomputed from the saved log-sum-exp and delta = rowsum(dO * O).
//
// Small heads make the softmax, not the matrix cores, the scarce resource:
// per score there are only 4 dh (forward) or 8 dh (backward) MFMA flops
// against one exp and a handful of vector instructions.  So these kernels
// keep the vector work per score minimal (scores are scaled inside the FMA
// that feeds exp2, the running max is raised lazily, masks are evaluated
// only on blocks that cross the diagonal or the sequence end) and keep
// several waves per SIMD so that one wave's exp overlaps another's MFMAs.
//
// They are bound by latency before either unit is full: a wave's block is a chain of LDS
// reads, MFMAs, the max, the exponentials and MFMAs again (vector unit busy a
// third, matrix cores a sixth of the cycles at 8 x 12 heads of 1024 x 64).  So the
// row fragments of a step are read together ahead of its MFMAs, whose two
// chains alternate, the transposed ones ahead of the exponentials where
// registers allow, and masked and whole blocks run in loops of their own.
// Forward / backward, before and after: 1 x 8 heads of 1359 x 64 causal 25 / 68 and
// 17.6 / 52 us; 2 x 12 of 2048 x 80 causal 45 / 128 and 37 / 104; 8 x 12 of 1024 x 64
// causal 31 / 84 and 28 / 76.
//
// 128-wide heads have twice the MFMA work per score of 64-wide ones, in twice the
// registers: the row fragments are read four k-steps at a time, and the dK/dV kernel,
// with 256 registers of operands and accumulators, runs one wave per SIMD whose two
// sub-tiles of a block the compiler overlaps instead.  Against the kernels
// that stage V and dO^T through register transposes (attention.hip), forward /
// backward: 2 x 16 heads of 2048 causal 218 / 723 and 53 / 155 us; 32 x 12 of 512
// causal 186 / 653 and 56 / 200; 7 x 16 of 1500 502 / 1617 and 151 / 517; 1 x 8 of 100
// causal 10.6 / 34 and 8.9 / 18.
//
// Workgroup = 2 to 4 waves x 32 rows (queries for the forward and dQ kernels,
// keys for the dK/dV kernel) of one (batch, head); the other operand streams
// through LDS in blocks of 64 rows, two stages, copied HBM -> LDS with
// buffer_load ... lds (no VGPR staging).
//
// Tile layout in LDS (R rows of a [rows][dh] bf16 block):
//  * each 64 dims (0..63; of 128-wide heads also 64..127): R rows of 128 B, eight 16-byte chunks, chunk c of row r
//    stored at c ^ swz(r).  Row-fragment reads (16 lanes = 16 consecutive
//    rows at one chunk) and transposing reads ds_read_b64_tr_b16 (32 lanes
//    = 4 consecutive rows x 4 chunks) then both touch 16 distinct 16-byte
//    bank groups per 256 bytes.
//  * dims 64..79 (80-wide heads): two chunks per row stored chunk-major,
//    [2][R] with row r of chunk t at slot r ^ 4t, after the 64-dim part.
// Products whose output rows are head dims (O^T, dV^T, dK^T, dQ^T) use
// 32-row MFMA tiles; for 80-wide heads the third tile's rows 80..95 read
// dims 64..79 again and are discarded at the store.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace {

constexpr int WR = 32;         // rows owned by a wave
constexpr int KB = 64;         // rows per staged block
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float RESCALE_SLACK = 8.f;
constexpr uint32_t OOB = 0x80000000u;

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

// The CDNA4 transposing LDS read through a restrict-qualified pointer: once
// inlined, the read carries alias-scope information, so the compiler does not
// make it wait for every LDS copy still in flight (the next block's, which
// land in another stage); the current stage's copies are waited for, and
// published by a barrier, before any wave reads it.
__device__ __forceinline__ bf16x4 ds_read_tr(const lds_bf16x4* __restrict__ p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(const_cast<lds_bf16x4*>(p));
}
__device__ __forceinline__ lds_void* lds(const bf16* p) { return (lds_void*)(const_cast<bf16*>(p)); }

template <int DH>
struct Cfg {
  static_assert(DH == 64 || DH == 80 || DH == 128, "64-, 80- or 128-wide heads");
  static constexpr bool TAIL = DH == 80;
  static constexpr int PARTS = DH / 64;      // 64-dim parts of a staged tile
  static constexpr int KS = DH / 16;         // k-steps over the head dims
  static constexpr int RS = DH == 128 ? 4 : KS;  // k-steps whose row fragments are read together
  static constexpr int OT = (DH + 31) / 32;  // 32-dim output tiles
};

// chunk swizzle of the 64-dim part
__device__ __forceinline__ int swz(int r) { return (((r >> 1) & 1) << 2) | ((r >> 2) & 3); }

__device__ __forceinline__ floatx16 zero16() {
  floatx16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
// Row (within a 32 x 32 tile) held by accumulator register r of lane group g.
__device__ __forceinline__ int acc_row(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }
// Maximum over the two half-waves, exchanged on the vector unit (a shuffle goes
// through the LDS unit).
__device__ __forceinline__ float halves_max(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float halves_sum(float x) { return x + __shfl_xor(x, 32, 64); }

// Maximum of three.  fmaxf first quiets each operand (v_max x, x), since the
// compiler cannot know that an MFMA result is no signaling NaN; the maximum that hands
// NaN on does not, and becomes one v_maximum3.  (As inline asm the same
// instruction read its operands 2 wait states after the MFMA that writes them, which
// needs 12: the compiler keeps them apart only for instructions that it knows.)
// A NaN score leaves its query's maximum where it was; that query's sum, output and
// log-sum-exp are NaN whatever the maximum.
__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// Which head and which block of its rows a workgroup takes.  Workgroups are dealt
// round-robin over the 8 XCDs, each with its own 4 MB L2.  With at least 64
// heads, each XCD takes a contiguous eighth of them, in groups whose staged
// operands (K and V, or Q and dO: 4 S dh bytes per head) fit its L2 together, and
// within a group all first (with a causal mask: heaviest) blocks, then all second
// ones.  So a head's blocks read the staged operand from HBM once, and
// neighbouring 80-wide heads, whose rows share 128-byte lines, share the L2.
// 64 x 16 heads of 257 x 80, blocks outermost over all heads: the forward read K and V
// three times (forward 79 us, backward 229), now 53 and 175.  Fewer heads are dealt out one by one.
__device__ __forceinline__ bool wg_item(int BH, int nb, int group, int& blk, int& bh) {
  const int id = blockIdx.x;
  if (BH < 64) {
    blk = id / BH;
    bh = id % BH;
    return true;
  }
  const int hx = (BH + 7) >> 3, slot = id >> 3;
  const int g = slot / (group * nb), r = slot - g * group * nb;
  const int gh = min(group, hx - g * group);
  blk = r / gh;
  bh = (id & 7) * hx + g * group + r % gh;
  return bh < BH;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const void* base, long byte_off) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)base + byte_off), (short)0, 0x7FFFFFFF,
                                           0x00020000);
}

// Copies of R rows (a block of K, V, Q or dO) into an LDS tile; rows >=
// nvalid read zero.  rs addresses row 0 of the block, rows ld elements apart.
template <int DH, int R, int NW>
__device__ __forceinline__ void copy_tile(__amdgpu_buffer_rsrc_t rs, long ld, int nvalid, bf16* dst,
                                          int wave) {
  const int lane = threadIdx.x & 63;
  constexpr int NM = R / 8 * Cfg<DH>::PARTS;  // 1 KB instructions of the 64-dim parts
#pragma unroll
  for (int i = 0; i < (NM + NW - 1) / NW; ++i) {
    const int j = NW * i + wave;
    if (NM % NW == 0 || j < NM) {
      const int row = 8 * (j % (R / 8)) + (lane >> 3);
      const int c = 8 * (j / (R / 8)) + ((lane & 7) ^ swz(row));
      const uint32_t o = row < nvalid ? (uint32_t)(((long)row * ld + 8 * c) * 2) : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, lds(dst + j * 512), 16, o, 0, 0, 0);
    }
  }
  if constexpr (Cfg<DH>::TAIL) {
    if (wave < R / 32) {  // 2 R slots of 16 bytes
      const int slot = 64 * wave + lane;
      const int t = slot / R;
      const int row = (slot % R) ^ (4 * t);
      const uint32_t o = row < nvalid ? (uint32_t)(((long)row * ld + 64 + 8 * t) * 2) : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, lds(dst + R * 64 + 512 * wave), 16, o, 0, 0, 0);
    }
  }
}

// Lane-dependent LDS offsets of the two kinds of tile read.
template <int DH, int R>
struct TileOfs {
  int rf[4];   // row fragment, k-step c % 4 of a 64-dim part: row lane % 32, dims 16 c + 8 g .. + 7
  int rft;     // row fragment of k-step 4 (80-wide heads)
  int tr[2];   // transposed read, output tile ot % 2 of a 64-dim part, 16-row step 0, low half
  int trt;     // transposed read of output tile 2 (80-wide heads)
  __device__ __forceinline__ void init(int lane) {
    const int g = lane >> 5, l31 = lane & 31;
#pragma unroll
    for (int c = 0; c < 4; ++c) rf[c] = l31 * 64 + 8 * ((2 * c + g) ^ swz(l31));
    rft = R * 64 + 8 * (g * R + (l31 ^ (4 * g)));
    // lane group G = lane / 16 reads rows 4 (G >> 1) + {0..3} (lo; +8 hi) of
    // dims 32 ot + 16 (G & 1) + 0..15; lane 4 e + q: row e, dims 4 q .. 4 q + 3
    const int G = lane >> 4, ll = lane & 15;
    const int r = 4 * (G >> 1) + (ll >> 2);
#pragma unroll
    for (int ot = 0; ot < 2; ++ot) {
      const int c = 4 * ot + 2 * (G & 1) + ((ll >> 1) & 1);
      tr[ot] = r * 64 + 8 * (c ^ swz(r)) + 4 * (ll & 1);
    }
    const int t = (ll >> 1) & 1;
    trt = R * 64 + 8 * (t * R + (r ^ (4 * t))) + 4 * (ll & 1);
  }
  // Row fragment of k-step c for rows 32 u + lane % 32.
  __device__ __forceinline__ bf16x8 row(const bf16* tile, int u, int c) const {
    const int o = c < 4 * Cfg<DH>::PARTS ? rf[c & 3] + (c >> 2) * R * 64 + 32 * u * 64 : rft + 32 * u * 8;
    return *reinterpret_cast<const bf16x8*>(tile + o);
  }
  // Transposed operand (rows = head dims 32 ot + lane % 32, k = 16 tile rows
  // 16 kk .. + 15 in the accumulator permutation) of output tile ot.
  __device__ __forceinline__ bf16x8 trans(const bf16* tile, int kk, int ot) const {
    bf16x4 lo, hi;
    if (ot < 2 * Cfg<DH>::PARTS) {
      const int part = (ot >> 1) * R * 64 + 16 * kk * 64;
      const int o = tr[ot & 1];
      lo = ds_read_tr((const lds_bf16x4*)lds(tile + o + part));
      // rows + 8 flip bit 1 of swz, i.e. chunk bit 1
      hi = ds_read_tr((const lds_bf16x4*)lds(tile + (o ^ 16) + 8 * 64 + part));
    } else {
      const int o = trt + 16 * kk * 8;
      lo = ds_read_tr((const lds_bf16x4*)lds(tile + o));
      hi = ds_read_tr((const lds_bf16x4*)lds(tile + o + 8 * 8));
    }
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

// Row fragments (dims 16 c + 8 g .. + 7) of one row per lane, from global;
// rows >= nvalid read zero.
template <int DH>
__device__ __forceinline__ void load_rows(const bf16* base, long ld, int r0, int nvalid, int lane,
                                          bf16x8 (&f)[Cfg<DH>::KS]) {
  const __amdgpu_buffer_rsrc_t rs = rows_rsrc(base, (long)r0 * ld * 2);
  const int r = lane & 31, g = lane >> 5;
  const uint32_t o = r < nvalid ? (uint32_t)(((long)r * ld + 8 * g) * 2) : OOB;
#pragma unroll
  for (int c = 0; c < Cfg<DH>::KS; ++c)
    f[c] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, o, 32 * c, 0));
}

// Store a transposed accumulator set (rows = head dims, column = this lane's
// row) times f as bf16 into out[0 .. DH).
template <int DH>
__device__ __forceinline__ void store_rowT(bf16* out, const floatx16 (&acc)[Cfg<DH>::OT], float f, int g) {
#pragma unroll
  for (int ot = 0; ot < Cfg<DH>::OT; ++ot)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      if (32 * ot + acc_row(4 * r4, g) >= DH) continue;
      bf16x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = f2bf(acc[ot][4 * r4 + e] * f);
      *reinterpret_cast<bf16x4*>(out + 32 * ot + acc_row(4 * r4, g)) = y;
    }
}

// ================================================================ forward
// The score tile is computed transposed, S^T = K Q^T: each lane owns one
// query (two lanes per query, 16 keys each per 32-key tile), so the running
// max and sum are per-lane scalars and the probabilities are directly the B
// operand of O^T += V^T P^T.

template <int DH>
struct FwdState {
  bf16x8 qf[Cfg<DH>::KS];
  floatx16 o[Cfg<DH>::OT];
  float m, l;  // running max (base 2, scaled, lazily raised); sum over this lane's keys
};

// One block of up to 64 keys.  MASK: some score of the block is masked (key >=
// lim, lim_rel = first excluded key of this lane's query relative to the block start
// and 4 g); two: keys 32..63 of the block hold a valid key for some query of
// the wave (always the case without MASK).
// PF: 16-key steps whose V fragments are read ahead of the exponentials (80-wide
// heads: one keeps three waves per SIMD, two make it two: 53 -> 60 us at 64 x 16 x 257).
template <int DH, bool MASK, int PF = DH == 64 ? 4 : 1>
__device__ __forceinline__ void fwd_block(FwdState<DH>& st, const TileOfs<DH, KB>& to, const bf16* Ks,
                                          const bf16* Vs, float sc, bool two, int lim_rel) {
  using C = Cfg<DH>;
  floatx16 s0 = zero16(), s1 = zero16();
#pragma unroll
  for (int c0 = 0; c0 < C::KS; c0 += C::RS) {
    bf16x8 k0[C::RS], k1[C::RS];
#pragma unroll
    for (int c = 0; c < C::RS; ++c) {
      k0[c] = to.row(Ks, 0, c0 + c);
      k1[c] = to.row(Ks, 1, c0 + c);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < C::RS; ++c) {
      s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0[c], st.qf[c0 + c], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1[c], st.qf[c0 + c], s1, 0, 0, 0);
    }
  }
  bf16x8 vf[PF ? PF : 1][C::OT];
#pragma unroll
  for (int kk = 0; kk < PF; ++kk)
#pragma unroll
    for (int ot = 0; ot < C::OT; ++ot) vf[kk][ot] = to.trans(Vs, kk, ot);
  __builtin_amdgcn_sched_barrier(0);
  float x[32];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    x[r] = s0[r];
    x[16 + r] = s1[r];
  }
  if (MASK) {
#pragma unroll
    for (int r = 0; r < 32; ++r) {
      const int kr = 32 * (r >> 4) + 8 * ((r & 15) >> 2) + (r & 3);
      x[r] = kr < lim_rel ? x[r] : -INFINITY;
    }
  }
  float mx4[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    mx4[i] = max3(x[i], x[4 + i], x[8 + i]);
    mx4[i] = max3(mx4[i], x[12 + i], x[16 + i]);
    mx4[i] = max3(mx4[i], x[20 + i], x[24 + i]);
  }
  mx4[0] = max3(mx4[0], x[28], x[29]);
  mx4[1] = max3(mx4[1], x[30], x[31]);
  const float mx = max3(mx4[0], mx4[1], max3(mx4[2], mx4[3], mx4[0]));
  const float mloc = halves_max(mx) * sc;
  const bool raise = mloc > st.m + RESCALE_SLACK;
  if (__builtin_amdgcn_ballot_w64(raise) != 0) {
    const float alpha = (raise && st.m != -INFINITY) ? __builtin_amdgcn_exp2f(st.m - mloc)
                                                     : (raise ? 0.f : 1.f);
    st.l *= alpha;
#pragma unroll
    for (int ot = 0; ot < C::OT; ++ot)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[ot][r] *= alpha;
    st.m = raise ? mloc : st.m;
  }
  const float nm = (st.m == -INFINITY) ? 0.f : -st.m;
  float lsum = 0.f;
  bf16x8 pb[4];
#pragma unroll
  for (int r = 0; r < 32; ++r) {
    const float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], sc, nm));
    lsum += pr;
    pb[r >> 3][r & 7] = f2bf(pr);
  }
  st.l += lsum;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    if (MASK && kk >= 2 && !two) break;
#pragma unroll
    for (int ot = 0; ot < C::OT; ++ot)
      st.o[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk < PF ? vf[kk < PF ? kk : 0][ot] : to.trans(Vs, kk, ot),
                                                         pb[kk], st.o[ot], 0, 0, 0);
  }
}

template <int DH, int NW>
__global__ __launch_bounds__(64 * NW, 2) void attn_small_fwd_kernel(AttnArgs a, int group) {
  using C = Cfg<DH>;
  constexpr int TILE = KB * DH, WGR = NW * WR;
  __shared__ __attribute__((aligned(1024))) bf16 smem[2 * 2 * TILE];  // 2 stages x (K, V)
  const int S = a.S;
  const int nqb = (S + WGR - 1) / WGR;
  // causal: heaviest block of every head first
  const int BH = a.B * a.H;
  int xb, bh;
  if (!wg_item(BH, nqb, group, xb, bh)) return;
  const int qb = a.causal ? (nqb - 1 - xb) : xb;
  const int b = bh / a.H, h = bh % a.H;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5;
  const int q0 = qb * WGR, wq0 = q0 + wave * WR, q = wq0 + (lane & 31);
  const bf16* Qb = a.q + (long)b * S * a.ldq + (long)h * DH;
  const bf16* Kb = a.k + (long)b * S * a.ldk + (long)h * DH;
  const bf16* Vb = a.v + (long)b * S * a.ldv + (long)h * DH;

  FwdState<DH> st;
  load_rows<DH>(Qb, a.ldq, wq0, S - wq0, lane, st.qf);
#pragma unroll
  for (int t = 0; t < C::OT; ++t) st.o[t] = zero16();
  st.m = -INFINITY;
  st.l = 0.f;
  TileOfs<DH, KB> to;
  to.init(lane);
  const float sc = a.scale * LOG2E;
  const int kv_end = a.causal ? min(S, q0 + WGR) : S;
  const int nblk = (kv_end + KB - 1) / KB;
  // keys this wave's queries may see: [0, wk_end); this lane's: [0, lim)
  const int wk_end = wq0 >= S ? 0 : a.causal ? min(S, wq0 + WR) : S;
  const int lim = a.causal ? min(S, q + 1) : S;
  // blocks that every query of the wave sees whole; the rest run the masked variant (two
  // loops, not a branch in one: where the variants join, the accumulators
  // would be copied on every block)
  const int nfull = (wq0 >= S ? 0 : a.causal ? min(S, wq0 + 1) : S) / KB;

  auto copy = [&](int j) {
    bf16* dst = smem + (j & 1) * 2 * TILE;
    copy_tile<DH, KB, NW>(rows_rsrc(Kb, (long)j * KB * a.ldk * 2), a.ldk, S - j * KB, dst, wave);
    copy_tile<DH, KB, NW>(rows_rsrc(Vb, (long)j * KB * a.ldv * 2), a.ldv, S - j * KB, dst + TILE, wave);
  };
  copy(0);
  wait_vm_lgkm0<0>();
  cta_barrier();
  int j = 0;
  for (; j < nfull; ++j) {
    const bf16* Ks = smem + (j & 1) * 2 * TILE;
    if (j + 1 < nblk) copy(j + 1);
    fwd_block<DH, false>(st, to, Ks, Ks + TILE, sc, true, 0);
    wait_vm_lgkm0<0>();
    cta_barrier();
  }
  for (; j < nblk; ++j) {
    const int kv0 = j * KB;
    const bf16* Ks = smem + (j & 1) * 2 * TILE;
    if (j + 1 < nblk) copy(j + 1);
    if (kv0 < wk_end) fwd_block<DH, true>(st, to, Ks, Ks + TILE, sc, wk_end - kv0 > 32, lim - kv0 - 4 * g);
    wait_vm_lgkm0<0>();
    cta_barrier();
  }
  st.l = halves_sum(st.l);
  if (q < S) {
    const float inv = (st.l > 0.f) ? 1.f / st.l : 0.f;
    store_rowT<DH>(a.o + ((long)b * S + q) * a.ldo + (long)h * DH, st.o, inv, g);
    if (g == 0) a.lse[((long)b * a.H + h) * S + q] = (st.m + log2f(st.l)) * LN2;
  }
}

// ================================================================ backward, dK and dV
// Each wave owns 32 keys and holds their K and V rows in registers; 64-query
// blocks of Q and dO (with lse * log2 e and delta) stream through LDS.  Per
// 32-query sub-tile: S = Q K^T and dP = dO V^T with queries as rows (lane =
// key), P = exp2(S scale log2e - lse2), dS = P (dP - delta), then
// dV^T += dO^T P and dK^T += Q^T dS with dO^T / Q^T from transposing reads.
template <int DH>
struct DkvState {
  bf16x8 kf[Cfg<DH>::KS], vf[Cfg<DH>::KS];
  floatx16 dk[Cfg<DH>::OT], dv[Cfg<DH>::OT];
};

// Sub-tile u (32 queries) of a staged block.  MASK: query rows acc_row(r, g) are
// valid when acc_row - 4 g < lim_q and >= lim_k.
template <int DH, bool MASK>
__device__ __forceinline__ void dkdv_sub(DkvState<DH>& st, const TileOfs<DH, KB>& to, const bf16* Qs,
                                         const bf16* dOs, const float* l2s, const float* dls, int u,
                                         int g, float sc, int lim_q, int lim_k) {
  using C = Cfg<DH>;
  floatx16 x = zero16(), y = zero16();
#pragma unroll
  for (int c0 = 0; c0 < C::KS; c0 += C::RS) {
    bf16x8 k0[C::RS], k1[C::RS];
#pragma unroll
    for (int c = 0; c < C::RS; ++c) {
      k0[c] = to.row(Qs, u, c0 + c);
      k1[c] = to.row(dOs, u, c0 + c);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < C::RS; ++c) {
      x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0[c], st.kf[c0 + c], x, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1[c], st.vf[c0 + c], y, 0, 0, 0);
    }
  }
  bf16x8 pb[2], db[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const floatx4 l4 = *reinterpret_cast<const floatx4*>(l2s + 32 * u + 8 * i + 4 * g);
    const floatx4 d4 = *reinterpret_cast<const floatx4*>(dls + 32 * u + 8 * i + 4 * g);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 4 * i + e;
      float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], sc, -l4[e]));
      if (MASK) {
        const int rr = 8 * i + e;  // acc_row - 4 g
        pr = (rr < lim_q && rr >= lim_k) ? pr : 0.f;
      }
      pb[r >> 3][r & 7] = f2bf(pr);
      db[r >> 3][r & 7] = f2bf(pr * (y[r] - d4[e]));
    }
  }
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int ot = 0; ot < C::OT; ++ot) {
      st.dv[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(to.trans(dOs, 2 * u + hh, ot), pb[hh], st.dv[ot], 0, 0, 0);
      st.dk[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(to.trans(Qs, 2 * u + hh, ot), db[hh], st.dk[ot], 0, 0, 0);
    }
}

template <int DH, int NW>
__global__ __launch_bounds__(64 * NW, DH == 128 ? 1 : 2) void attn_small_dkdv_kernel(AttnBwdArgs a, int group) {
  using C = Cfg<DH>;
  constexpr int BQ = KB, WGR = NW * WR;
  constexpr int QT = BQ * DH;
  constexpr int STG = 2 * QT + 2 * 2 * BQ;  // Q, dO, lse2[64], delta[64]
  __shared__ __attribute__((aligned(1024))) bf16 smem[2 * STG];
  const int S = a.f.S;
  // with a causal mask the first keys see the most queries
  const int BH = a.f.B * a.f.H;
  int kblk, bh;
  if (!wg_item(BH, (S + WGR - 1) / WGR, group, kblk, bh)) return;
  const int b = bh / a.f.H, h = bh % a.f.H;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5;
  const int k0 = kblk * WGR;
  const int kmin = k0 + wave * WR;
  const int key = kmin + (lane & 31);
  const long hs = ((long)b * a.f.H + h) * S;
  const bf16* Qb = a.f.q + (long)b * S * a.f.ldq + (long)h * DH;
  const bf16* Kb = a.f.k + (long)b * S * a.f.ldk + (long)h * DH;
  const bf16* Vb = a.f.v + (long)b * S * a.f.ldv + (long)h * DH;
  const bf16* dOb = a.dout + (long)b * S * a.lddo + (long)h * DH;
  const float sc = a.f.scale * LOG2E;

  DkvState<DH> st;
  load_rows<DH>(Kb, a.f.ldk, kmin, S - kmin, lane, st.kf);
  load_rows<DH>(Vb, a.f.ldv, kmin, S - kmin, lane, st.vf);
#pragma unroll
  for (int t = 0; t < C::OT; ++t) {
    st.dk[t] = zero16();
    st.dv[t] = zero16();
  }
  TileOfs<DH, BQ> to;
  to.init(lane);

  const int q_start = a.f.causal ? k0 : 0;
  const int nqb = (S - q_start + BQ - 1) / BQ;
  float lsd = 0.f;  // wave 0: lse of the next block's query `lane`; wave 1: its delta

  auto stage = [&](int j) { return smem + (j & 1) * STG; };
  auto fetch = [&](int j) {
    const int qs = q_start + j * BQ;
    bf16* sj = stage(j);
    copy_tile<DH, BQ, NW>(rows_rsrc(Qb, (long)qs * a.f.ldq * 2), a.f.ldq, S - qs, sj, wave);
    copy_tile<DH, BQ, NW>(rows_rsrc(dOb, (long)qs * a.lddo * 2), a.lddo, S - qs, sj + QT, wave);
    if (wave < 2) {
      const int qi = qs + lane;
      lsd = qi < S ? (wave ? a.delta[hs + qi] : a.f.lse[hs + qi]) : 0.f;
    }
  };
  auto publish = [&](int j) {
    if (wave < 2) reinterpret_cast<float*>(stage(j) + 2 * QT)[wave * BQ + lane] = wave ? lsd : lsd * LOG2E;
  };
  auto next = [&](int j) {
    if (j + 1 < nqb) {
      wait_vm_lgkm0<0>();
      publish(j + 1);
      wait_vm_lgkm0<0>();
      cta_barrier();
    }
  };
  // the masked variant of a block: sub-tiles without a valid pair are skipped
  auto masked = [&](int j) {
    const bf16* Qs = stage(j);
    const float* l2s = reinterpret_cast<const float*>(Qs + 2 * QT);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int qs = q_start + j * BQ + 32 * u;
      if (kmin >= S || qs >= S || (a.f.causal && qs + 31 < kmin)) continue;
      dkdv_sub<DH, true>(st, to, Qs, Qs + QT, l2s, l2s + BQ, u, g, sc, S - qs - 4 * g,
                         a.f.causal ? key - qs - 4 * g : -(1 << 30));
    }
  };

  fetch(0);
  wait_vm_lgkm0<0>();
  publish(0);
  wait_vm_lgkm0<0>();
  cta_barrier();

  // blocks [j1, j2) hold only valid pairs for this wave: past the diagonal, short of S
  // (loops of their own: a join of two variants would copy the accumulators)
  const int j1 = a.f.causal ? min(nqb, (kmin + 31 - q_start + BQ - 1) / BQ) : 0;
  const int j2 = kmin >= S ? j1 : max(j1, (S - q_start) / BQ);
  int j = 0;
  for (; j < j1; ++j) {
    if (j + 1 < nqb) fetch(j + 1);
    masked(j);
    next(j);
  }
  for (; j < j2; ++j) {
    const bf16* Qs = stage(j);
    const float* l2s = reinterpret_cast<const float*>(Qs + 2 * QT);
    if (j + 1 < nqb) fetch(j + 1);
#pragma unroll
    for (int u = 0; u < 2; ++u) { dkdv_sub<DH, false>(st, to, Qs, Qs + QT, l2s, l2s + BQ, u, g, sc, 0, 0); if (DH != 128) __builtin_amdgcn_sched_barrier(0); }
    next(j);
  }
  for (; j < nqb; ++j) {
    if (j + 1 < nqb) fetch(j + 1);
    masked(j);
    next(j);
  }
  if (key < S) {
    store_rowT<DH>(a.dk + ((long)b * S + key) * a.lddk + (long)h * DH, st.dk, a.f.scale, g);
    store_rowT<DH>(a.dv + ((long)b * S + key) * a.lddv + (long)h * DH, st.dv, 1.f, g);
  }
}

// ================================================================ backward, dQ
// Each wave owns 32 queries and holds their Q and dO rows, lse2 and delta in
// registers; 64-key blocks of K and V stream through LDS.  Per 32-key
// sub-tile: S^T = K Q^T and dP^T = V dO^T (lane = query),
// dS^T = P^T (dP^T - delta), dQ^T += K^T dS^T with K^T from transposing reads.
// This kernel runs first and also computes delta = rowsum(dO * O) for the
// dK / dV kernel.
template <int DH>
struct DqState {
  bf16x8 qf[Cfg<DH>::KS], of[Cfg<DH>::KS];
  floatx16 dq[Cfg<DH>::OT];
  float nl2, dlt;  // -lse * log2 e and delta of this lane's query
};

// Sub-tile u (32 keys) of a staged block.  MASK: keys with acc_row - 4 g < lim_rel are valid.
template <int DH, bool MASK>
__device__ __forceinline__ void dq_sub(DqState<DH>& st, const TileOfs<DH, KB>& to, const bf16* Ks,
                                       const bf16* Vs, int u, float sc, int lim_rel) {
  using C = Cfg<DH>;
  floatx16 x = zero16(), y = zero16();
#pragma unroll
  for (int c0 = 0; c0 < C::KS; c0 += C::RS) {
    bf16x8 k0[C::RS], k1[C::RS];
#pragma unroll
    for (int c = 0; c < C::RS; ++c) {
      k0[c] = to.row(Ks, u, c0 + c);
      k1[c] = to.row(Vs, u, c0 + c);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < C::RS; ++c) {
      x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0[c], st.qf[c0 + c], x, 0, 0, 0);
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1[c], st.of[c0 + c], y, 0, 0, 0);
    }
  }
  bf16x8 kt[2][C::OT];
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int ot = 0; ot < C::OT; ++ot) kt[hh][ot] = to.trans(Ks, 2 * u + hh, ot);
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 db[2];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], sc, st.nl2));
    if (MASK) {
      const int kr = 8 * (r >> 2) + (r & 3);
      pr = kr < lim_rel ? pr : 0.f;
    }
    db[r >> 3][r & 7] = f2bf(pr * (y[r] - st.dlt));
  }
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int ot = 0; ot < C::OT; ++ot)
      st.dq[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[hh][ot], db[hh], st.dq[ot], 0, 0, 0);
}

template <int DH, int NW>
__global__ __launch_bounds__(64 * NW, 2) void attn_small_dq_kernel(AttnBwdArgs a, int group) {
  using C = Cfg<DH>;
  constexpr int TILE = KB * DH, WGR = NW * WR;
  __shared__ __attribute__((aligned(1024))) bf16 smem[2 * 2 * TILE];  // 2 stages x (K, V)
  const int S = a.f.S;
  const int nqb = (S + WGR - 1) / WGR;
  const int BH = a.f.B * a.f.H;
  int xb, bh;
  if (!wg_item(BH, nqb, group, xb, bh)) return;
  const int qb = a.f.causal ? (nqb - 1 - xb) : xb;
  const int b = bh / a.f.H, h = bh % a.f.H;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5;
  const int q0 = qb * WGR, wq0 = q0 + wave * WR, q = wq0 + (lane & 31);
  const long hs = ((long)b * a.f.H + h) * S;
  const bf16* Qb = a.f.q + (long)b * S * a.f.ldq + (long)h * DH;
  const bf16* Kb = a.f.k + (long)b * S * a.f.ldk + (long)h * DH;
  const bf16* Vb = a.f.v + (long)b * S * a.f.ldv + (long)h * DH;
  const bf16* dOb = a.dout + (long)b * S * a.lddo + (long)h * DH;
  const float sc = a.f.scale * LOG2E;

  DqState<DH> st;
  load_rows<DH>(Qb, a.f.ldq, wq0, S - wq0, lane, st.qf);
  load_rows<DH>(dOb, a.lddo, wq0, S - wq0, lane, st.of);
  st.nl2 = q < S ? -a.f.lse[hs + q] * LOG2E : 0.f;
  // delta = rowsum(dO * O) of this lane's query, from the two halves of its row
  {
    bf16x8 ov[C::KS];
    load_rows<DH>(a.f.o + (long)b * S * a.f.ldo + (long)h * DH, a.f.ldo, wq0, S - wq0, lane, ov);
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < C::KS; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = __builtin_fmaf(bf2f(st.of[c][e]), bf2f(ov[c][e]), acc);
    st.dlt = halves_sum(acc);
    if (g == 0 && q < S) a.delta[hs + q] = st.dlt;
  }
#pragma unroll
  for (int t = 0; t < C::OT; ++t) st.dq[t] = zero16();
  TileOfs<DH, KB> to;
  to.init(lane);

  const int kv_end = a.f.causal ? min(S, q0 + WGR) : S;
  const int nkb = (kv_end + KB - 1) / KB;
  const int wk_end = wq0 >= S ? 0 : a.f.causal ? min(S, wq0 + WR) : S;
  const int lim = a.f.causal ? min(S, q + 1) : S;
  const int nfull = (wq0 >= S ? 0 : a.f.causal ? min(S, wq0 + 1) : S) / KB;  // as in the forward

  auto copy = [&](int j) {
    bf16* dst = smem + (j & 1) * 2 * TILE;
    copy_tile<DH, KB, NW>(rows_rsrc(Kb, (long)j * KB * a.f.ldk * 2), a.f.ldk, S - j * KB, dst, wave);
    copy_tile<DH, KB, NW>(rows_rsrc(Vb, (long)j * KB * a.f.ldv * 2), a.f.ldv, S - j * KB, dst + TILE, wave);
  };
  copy(0);
  wait_vm_lgkm0<0>();
  cta_barrier();
  int j = 0;
  for (; j < nfull; ++j) {
    const bf16* Ks = smem + (j & 1) * 2 * TILE;
    if (j + 1 < nkb) copy(j + 1);
#pragma unroll
    for (int u = 0; u < 2; ++u) { dq_sub<DH, false>(st, to, Ks, Ks + TILE, u, sc, 0); __builtin_amdgcn_sched_barrier(0); }
    wait_vm_lgkm0<0>();
    cta_barrier();
  }
  for (; j < nkb; ++j) {
    const bf16* Ks = smem + (j & 1) * 2 * TILE;
    if (j + 1 < nkb) copy(j + 1);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int kv = j * KB + 32 * u;
      if (kv < wk_end) dq_sub<DH, true>(st, to, Ks, Ks + TILE, u, sc, lim - kv - 4 * g);
    }
    wait_vm_lgkm0<0>();
    cta_barrier();
  }
  if (q < S) store_rowT<DH>(a.dq + ((long)b * S + q) * a.lddq + (long)h * DH, st.dq, a.f.scale, g);
}

// Staged operand bytes of the heads an XCD works on at a time, of its 4 MB L2.
// Causal blocks differ in work: a larger group balances them better (96 heads of
// 1024 x 64, 3 MB per XCD: forward 28 us as one group, 33 us as 10 + 2 heads).
inline long l2_group(bool causal) { return causal ? 9L << 19 : 3L << 19; }

// Waves (of 32 rows) per workgroup.  Four, which share the staged blocks of the
// other operand; fewer where that leaves wave slots or CUs idle: in the forward
// three when the rows then fill the last workgroup better (257 rows are 9 wave
// tiles: three workgroups either way, of 9 waves instead of 12; 64 x 16 heads 58 ->
// 56 us; the backward, at two waves per SIMD either way, took 185 -> 196), two
// when four give fewer than 192 workgroups.
int waves_per_wg(int S, long BH, bool fwd) {
  const int tiles = (S + WR - 1) / WR;
  if ((long)((tiles + 3) / 4) * BH < 192) return 2;
  return fwd && (tiles + 2) / 3 * 3 < (tiles + 3) / 4 * 4 ? 3 : 4;
}

bool ok16(const void* p, long ld) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 8 == 0; }
bool ok8(const void* p, long ld) { return (reinterpret_cast<uintptr_t>(p) & 7) == 0 && ld % 4 == 0; }
// byte offsets of a staged block and of a wave's rows stay below 2^31
bool rows_fit(long ld) { return 128 * ld * 2 < (1L << 30); }

}  // namespace

bool attn_small_fwd_eligible(const AttnArgs& a) {
  return (a.dh == 64 || a.dh == 80 || a.dh == 128) && a.scale > 0.f && ok16(a.q, a.ldq) && ok16(a.k, a.ldk) && ok16(a.v, a.ldv) &&
         ok8(a.o, a.ldo) && rows_fit(a.ldq) && rows_fit(a.ldk) && rows_fit(a.ldv);
}

bool attn_small_bwd_eligible(const AttnBwdArgs& a) {
  return attn_small_fwd_eligible(a.f) && ok16(a.dout, a.lddo) && rows_fit(a.lddo) && ok16(a.f.o, a.f.ldo) &&
         rows_fit(a.f.ldo) && a.delta != nullptr && ok8(a.dq, a.lddq) &&
         ok8(a.dk, a.lddk) && ok8(a.dv, a.lddv);
}

// One kernel of a head width: `three` also instantiates it for three waves (the forward).
#define SMALL_LAUNCH(KERNEL, DH, args, f, three)                                                   \
  do {                                                                                             \
    const int BH_ = (f).B * (f).H, hx_ = (BH_ + 7) / 8;                                            \
    const int nw_ = waves_per_wg((f).S, BH_, three);                                               \
    const long nb_ = sat_cdiv((f).S, nw_ * WR);                                                    \
    const int group_ =                                                                             \
        (int)std::max(1L, std::min((long)hx_, l2_group((f).causal) / (4L * (f).S * DH)));          \
    const dim3 grid_((unsigned)(nb_ * (BH_ < 64 ? BH_ : 8 * hx_)));                                \
    if (nw_ == 2) hipLaunchKernelGGL((KERNEL<DH, 2>), grid_, dim3(128), 0, s, args, group_);       \
    else if (three && nw_ == 3) hipLaunchKernelGGL((KERNEL<DH, three ? 3 : 4>), grid_, dim3(192), 0, s, args, group_); \
    else hipLaunchKernelGGL((KERNEL<DH, 4>), grid_, dim3(256), 0, s, args, group_);                \
  } while (0)

hipError_t launch_attn_small_fwd(const AttnArgs& a, hipStream_t s) {
  if (a.dh == 64) SMALL_LAUNCH(attn_small_fwd_kernel, 64, a, a, true);
  else if (a.dh == 80) SMALL_LAUNCH(attn_small_fwd_kernel, 80, a, a, true);
  else SMALL_LAUNCH(attn_small_fwd_kernel, 128, a, a, true);
  return hipGetLastError();
}

// dQ (which also writes delta), then dK / dV.
hipError_t launch_attn_small_bwd(const AttnBwdArgs& a, hipStream_t s) {
  if (a.f.dh == 64) SMALL_LAUNCH(attn_small_dq_kernel, 64, a, a.f, false);
  else if (a.f.dh == 80) SMALL_LAUNCH(attn_small_dq_kernel, 80, a, a.f, false);
  else SMALL_LAUNCH(attn_small_dq_kernel, 128, a, a.f, false);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.f.dh == 64) SMALL_LAUNCH(attn_small_dkdv_kernel, 64, a, a.f, false);
  else if (a.f.dh == 80) SMALL_LAUNCH(attn_small_dkdv_kernel, 80, a, a.f, false);
  else SMALL_LAUNCH(attn_small_dkdv_kernel, 128, a, a.f, false);
  return hipGetLastError();
}
