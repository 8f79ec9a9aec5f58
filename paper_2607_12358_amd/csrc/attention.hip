// Full non-causal multi-head self-attention over all video (and text) tokens.
//
// bf16 path: flash-style single pass on MFMA (v_mfma_f32_32x32x16_bf16).
//   A workgroup owns 32 queries per wave of one head (8 waves for d = 128,
//   4 for d = 64) and streams the head's keys in tiles of 64 through two LDS
//   ring buffers filled by global -> LDS DMA.  Scores are formed transposed,
//   S^T = K Q^T, so that a lane owns one query (lane % 32) and 16 keys per
//   32-key block: the row max is an in-register max plus one exchange with
//   the partner half-wave (v_permlane32_swap), and the row sum stays a
//   per-lane partial until the end.  The probabilities P^T in accumulator
//   layout are exactly the B operand of O^T = V^T P^T when the contraction
//   index is relabelled accordingly, so P never leaves registers; V is stored
//   transposed (keys contiguous) by the QKV epilogue, and keys are staged
//   into LDS in a permuted order so the matching A operand is one 16-byte
//   read from an XOR-swizzled V^T tile (no LDS bank conflicts).  Each wave
//   runs a two-stage software pipeline (exponentials of one tile under the
//   score MFMAs of the next; for d = 128 the next tile's row max under the
//   P V MFMAs, for d = 64 an optimistic softmax without a row max, checked
//   through the probability sum).
//   Work items are mapped so each XCD streams a contiguous, head-major range
//   (a head's K/V passes through few L2s).  Softmax runs in the exp2 domain
//   in fp32: with plain Q, log2(e)/sqrt(d) is folded into one FMA per score;
//   with Q stored pre-multiplied by log2(e)/sqrt(d) (as the model's QKV
//   epilogue writes it) the score MFMAs start from -m and deliver the exp2
//   arguments themselves.  The row sum adds the bf16-rounded probabilities
//   that the P V product uses.
// fp32 path: the fp32 matrix instruction, 32 queries per workgroup, the keys
//   split over its four waves (for the fp32 configuration); up to 18 tokens one
//   wave per (head, query).
#include <atomic>

#include "attn_form.h"
#include "common.h"

namespace acid {

namespace {

constexpr int BKV = 64;

template <int D>
struct AttnLds {
  static constexpr int KLD = D;         // K tile row stride (elements), XOR-swizzled
  static constexpr int VLD = BKV;       // V^T tile row stride: 128 B, XOR-swizzled
  static constexpr int K_ELEMS = BKV * KLD;
  static constexpr int V_ELEMS = D * VLD;
  static constexpr size_t BYTES = (size_t)2 * (K_ELEMS + V_ELEMS) * sizeof(bf16);
};

// Dynamic LDS of a launch: a ring per key range, reused by the merge of the
// ranges (each wave's O^T in fp32, and m and l per lane).
template <int D, int NW, int KS>
constexpr size_t attn_lds_bytes() {
  const size_t ring = KS * AttnLds<D>::BYTES, merge = (size_t)NW * 64 * (D / 2 * 4 + 8);
  return KS > 1 && merge > ring ? merge : ring;
}

// Keys are staged into the K tile in the order pi(j) = j with bits 2 and 3
// swapped (an involution).  Then the 8 probabilities a lane feeds to one
// P V^T MFMA step are 8 consecutive keys, so the matching V^T operand is one
// 16-byte LDS read.
__device__ __forceinline__ int key_perm(int j) {
  return (j & ~12) | ((j & 4) << 1) | ((j & 8) >> 1);
}

// 16-byte slot of chunk c in row r of a tile with 2^log2c chunks per row:
// 16 consecutive rows read at one chunk cover all 64 four-byte LDS banks
// (rows of 256 B start on the same bank: XOR with r % 16; rows of 128 B
// alternate halves: XOR with (r / 2) % 8).
template <int CHUNKS>
__device__ __forceinline__ int swz(int r, int c) {
  if constexpr (CHUNKS == 16) return c ^ (r & 15);
  else return c ^ ((r >> 1) & 7);
}

typedef __attribute__((address_space(3))) void lds_void_t;

// One 16-byte-per-lane global -> LDS DMA: lane l reads 16 bytes at
// base + off_bytes(l) and writes LDS bytes [lds + 16 l, +16).  base and lds
// are wave-uniform (scalar registers).  Inline assembly keeps it out of the
// compiler's wait-count bookkeeping (completion is waited for explicitly).
__device__ __forceinline__ uint64_t uniform_ptr(const void* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ void dma16(uint64_t base, uint32_t off_bytes, uint32_t lds_byte) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(off_bytes), "s"(base), "s"(lds_byte)
      : "memory");
}

// Bijection from dispatch order to (head, query-tile) work items that gives
// XCD x (workgroups bid = x, x+8, ...) a contiguous, head-major range, so a
// head's K/V is streamed through as few L2s as possible.
// The number of items is below 2^26 (checked at the entry): 32-bit divisions.
__device__ __forceinline__ uint32_t attn_xcd_remap(uint32_t bid, uint32_t T) {
  constexpr uint32_t NX = 8;
  const uint32_t x = bid % NX, local = bid / NX;
  const uint32_t q = T / NX, r = T % NX;
  return (x < r) ? x * (q + 1) + local : r * (q + 1) + (x - r) * q + local;
}

// A first softmax reference below this (exp2 domain) is looked at again: a score
// added to one of this size is rounded by 2^-14 at most, a 32nd of a
// probability's rounding to bf16.
constexpr float kLowRef = -1024.f;

// Maximum of a value over the two half-waves (lanes l and l ^ 32).
__device__ __forceinline__ float half_swap_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Software pipeline, per wave and key tile j (LDS holds K_{j+1} and V_j):
//   VALU: p = 2^(s_j - m) for tile j (scores formed one iteration earlier),
//   MFMA: S_{j+1} = K_{j+1} Q^T, then O^T += V_j^T P_j^T,
//   VALU: row max of S_{j+1} (under the P V MFMAs),
// so the softmax of one tile overlaps the score MFMAs of the next.  K runs
// one tile ahead of V in the two LDS ring buffers: iteration j streams
// K_{j+2} and V_{j+1} in while K_{j+1} and V_j are read.  Softmax does not
// depend on the order of the keys, so the ragged last tile (keys up to L)
// is processed first, staged through registers and masked in the prologue;
// every tile of the loop is full and arrives by DMA.
//
// KS > 1 (short sequences): the workgroup's NW waves form KS groups of QW =
// NW / KS, each with LDS buffers of its own.  The groups hold the same 32 QW
// queries and take KS contiguous ranges of the key tiles (the ragged tile
// belongs to the last), running the pipeline above on them; their O and l
// meet in LDS and are added in group order, weighted by 2^(m - max m).
template <int D, int NW, bool kPre, int KS = 1>
__global__ __launch_bounds__(64 * NW, 8 / NW) void attn_bf16_kernel(const bf16* Q,
                                                           const bf16* Kp,
                                                           const bf16* Vt,
                                                           int64_t L, int64_t vt_ld, int n_heads,
                                                           bf16* __restrict__ O, int64_t o_ld,
                                                           float scale_log2,
                                                           const int32_t* pred) {
  if (pred && *pred == 0) return;  // predicated off by the device gate
  using Ld = AttnLds<D>;
  constexpr int QW = NW / KS;                // waves per key range
  constexpr int BQ = 32 * QW, NT = 64 * QW;  // queries / threads per key range
  constexpr int KLD = Ld::KLD, VLD = Ld::VLD;
  constexpr int NK = D / 16;     // MFMA K-steps over the head dim
  constexpr int ND = D / 32;     // 32-row blocks of O^T
  constexpr int CPT = D / (8 * QW);  // 16-byte chunks per thread per tile (K, and V^T)
  constexpr int KCH = D / 8;     // 16-byte chunks per K row
  constexpr int KROWS_PER_KB = 1024 / (2 * D);  // K rows per 1 KB
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wave_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = KS > 1 ? wave_wg / QW : 0;  // key range
  bf16* Ks = reinterpret_cast<bf16*>(smem + grp * Ld::BYTES);
  bf16* Vs = Ks + 2 * Ld::K_ELEMS;

  const uint32_t n_qt = (uint32_t)((L + BQ - 1) / BQ);
  const uint32_t item = attn_xcd_remap(blockIdx.x, n_qt * n_heads);
  const int head = (int)(item / n_qt);
  const int64_t qt = item - head * n_qt;
  const int tid = threadIdx.x - grp * NT, lane = tid & 63;
  const int wave = wave_wg - grp * QW;
  const int lr = lane & 31, lg = lane >> 5;
  const int64_t qrow = qt * BQ + wave * 32 + lr;

  const bf16* Qh = Q + (int64_t)head * L * D;
  const bf16* Kh = Kp + (int64_t)head * L * D;
  const bf16* Vh = Vt + (int64_t)head * D * vt_ld;

  bf16x8 qf[NK];
  {
    const bf16* qsrc = Qh + (qrow < L ? qrow : L - 1) * D + lg * 8;
    const uint32_t qmask = qrow < L ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      uint4 v = *reinterpret_cast<const uint4*>(qsrc + kk * 16);
      v = make_uint4(v.x & qmask, v.y & qmask, v.z & qmask, v.w & qmask);
      qf[kk] = __builtin_bit_cast(bf16x8, v);
    }
  }

  f32x16 o[ND];
#pragma unroll
  for (int db = 0; db < ND; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -__builtin_inff(), l_run = 0.f;
  // kPre (Q stored pre-multiplied by log2(e)/sqrt(d)): the score MFMAs start
  // from C = -m instead of 0, so they deliver the exp2 arguments directly and
  // no per-score multiply-add remains.  cneg holds -m in every entry.
  f32x16 cneg;
  auto set_cneg = [&](float v) {
#pragma unroll
    for (int r = 0; r < 16; ++r) cneg[r] = v;
  };

  // Offsets are 32-bit (a head's K is L * d elements, its V^T d * vt_ld:
  // far below 2^31 bytes).
  const int Li = (int)L;
  const int vld = (int)vt_ld;
  const uint32_t ks_lds = (uint32_t)(uintptr_t)(lds_void_t*)Ks;
  const uint32_t vs_lds = (uint32_t)(uintptr_t)(lds_void_t*)Vs;

  // DMA staging of a full tile in 1 KB blocks: block b = CPT w + i is wave
  // w's share.  K tile: LDS row r (D * 2 bytes) holds key j0 + key_perm(r);
  // V^T tile: LDS row d (128 bytes) holds keys j0 .. j0+63 of head dim d;
  // chunks sit at swizzled slots (swz).  With 8 waves (two per SIMD: waves
  // w and w + 4) wave w issues the blocks of both, so wave w + 4 issues no
  // global loads in the loop.  Per-lane byte offsets relative to the tile's
  // first element, and the block each DMA fills:
  constexpr bool kPairDma = NW == 8 && KS == 1;
  constexpr int NB = kPairDma ? 2 * CPT : CPT;
  const bool dma_wave = !kPairDma || wave < 4;
  uint32_t koff[NB], voff[NB];
  int kblk[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int blk = (kPairDma ? (wave & 3) + (i / CPT) * 4 : wave) * CPT + i % CPT;
    kblk[i] = blk;
    const int r = blk * KROWS_PER_KB + lane / KCH;
    koff[i] = (uint32_t)(key_perm(r) * D + swz<KCH>(r, lane % KCH) * 8) * 2u;
    const int d = blk * 8 + (lane >> 3);
    voff[i] = (uint32_t)(d * vld + swz<8>(d, lane & 7) * 8) * 2u;
  }
  auto stage_k_dma = [&](int buf, int j0) {
    if (!dma_wave) return;
    const uint64_t base = uniform_ptr(Kh + (int64_t)j0 * D);
#pragma unroll
    for (int i = 0; i < NB; ++i)
      dma16(base, koff[i], ks_lds + buf * Ld::K_ELEMS * 2 + kblk[i] * 1024);
  };
  auto stage_v_dma = [&](int buf, int j0) {
    if (!dma_wave) return;
    const uint64_t base = uniform_ptr(Vh + j0);
#pragma unroll
    for (int i = 0; i < NB; ++i)
      dma16(base, voff[i], vs_lds + buf * Ld::V_ELEMS * 2 + kblk[i] * 1024);
  };
  // The ragged tile j0 .. L-1 through registers, keys >= L zeroed (K rows,
  // and V^T columns, whose padding past L may hold anything).
  auto stage_tail = [&](int buf, int j0) {
    u32x4 rk[CPT], rv[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = tid + NT * i;
      const int key = j0 + c / KCH;
      rk[i] = *reinterpret_cast<const u32x4*>(
          Kh + (uint32_t)((key < Li ? key : Li - 1) * D + (c % KCH) * 8));
      const int key0 = j0 + (c & 7) * 8;
      rv[i] = *reinterpret_cast<const u32x4*>(Vh + (uint32_t)((c >> 3) * vld +
                                                              (key0 < Li ? key0 : 0)));
    }
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
      const int c = tid + NT * i;
      u32x4 kv = rk[i];
      kv &= (j0 + c / KCH < Li) ? 0xFFFFFFFFu : 0u;
      const int kr = key_perm(c / KCH);
      *reinterpret_cast<u32x4*>(Ks + buf * Ld::K_ELEMS + kr * KLD + swz<KCH>(kr, c % KCH) * 8) =
          kv;
      const int key0 = j0 + (c & 7) * 8;
      const int valid = key0 < Li ? Li - key0 : 0;
      u32x4 vm;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        vm[p] = ((2 * p < valid) ? 0x0000FFFFu : 0u) | ((2 * p + 1 < valid) ? 0xFFFF0000u : 0u);
      *reinterpret_cast<u32x4*>(Vs + buf * Ld::V_ELEMS + (c >> 3) * VLD +
                                swz<8>(c >> 3, c & 7) * 8) = rv[i] & vm;
    }
  };

  // S^T (keys x queries) of the K tile in buffer kbuf, two 32-key blocks.
  auto scores = [&](f32x16(&s)[2], int kbuf) {
    if constexpr (!kPre) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
    }
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const int kr = kb * 32 + lr;
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(Ks + kbuf * Ld::K_ELEMS + kr * KLD +
                                                            swz<KCH>(kr, 2 * kk + lg) * 8);
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk],
                                                        (kPre && kk == 0) ? cneg : s[kb], 0, 0, 0);
      }
  };
  // Row max of the first (raw) score tile, shared with the partner half-wave
  // that holds the other keys of the same query: the initial reference m.
  auto first_max = [&](const f32x16(&s)[2]) {
    float mx = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
    m_run = kPre ? half_swap_max(mx) : half_swap_max(mx) * scale_log2;
  };
  // Scores to exp2 arguments in place: s log2(e)/sqrt(d) - m.
  auto shift = [&](f32x16(&s)[2]) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        s[kb][r] = kPre ? s[kb][r] - m_run : __builtin_fmaf(s[kb][r], scale_log2, -m_run);
  };
  auto sub_all = [&](f32x16(&s)[2], float v) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb][r] -= v;
  };
  // Row max of a raw score tile (scale > 0 commutes with max), shared with
  // the partner half-wave that holds the other keys of the same query, then
  // the tile is rewritten in place as s log2(e)/sqrt(d) - m (exp2 argument).
  // Lazy rescaling: the reference max m moves only when the new max exceeds
  // it by more than 2^8 in probability, so probabilities stay <= 256 (exact
  // range for bf16 and fp32) and the O / l rescale is skipped on most tiles.
  float m_nx = 0.f, a_nx = 1.f, d_nx = 0.f;
  bool g_nx = false;
  auto row_max_shift = [&](f32x16(&s)[2]) {
    float mx = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
    mx = half_swap_max(mx);
    const float m_cand = mx * scale_log2;
    g_nx = m_cand > m_run + 8.0f;
    m_nx = g_nx ? m_cand : m_run;
    a_nx = __builtin_amdgcn_exp2f(m_run - m_nx);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb][r] = __builtin_fmaf(s[kb][r], scale_log2, -m_nx);
  };
  // kPre: the tile already holds s' - m; only the lazy-rescale decision is
  // taken here (its shift by d_nx, rare, is applied at the next iteration).
  auto row_max_check = [&](const f32x16(&s)[2]) {
    float mx = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
    mx = half_swap_max(mx);
    g_nx = mx > 8.0f;
    d_nx = g_nx ? mx : 0.0f;
    m_nx = m_run + d_nx;
    a_nx = __builtin_amdgcn_exp2f(-d_nx);
  };
  // p = 2^(shifted score) for the 16 keys of one P V K-step (kb, k2), rounded
  // to bf16 as the B operand of the P V MFMAs; the row sum adds exactly those
  // bf16 values (v_dot2 with (1, 1)) into ps.
  auto probs_part = [&](const f32x16(&s)[2], int kb, int k2, bf16x8(&pf)[2][2],
                        float(&ps)[2]) {
    const bf16x2 one = {(bf16)1.0f, (bf16)1.0f};
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 8 * k2 + 2 * e;
      const bf16x2 pr = {(bf16)__builtin_amdgcn_exp2f(s[kb][r]),
                         (bf16)__builtin_amdgcn_exp2f(s[kb][r + 1])};
      ps[e & 1] = __builtin_amdgcn_fdot2_f32_bf16(pr, one, ps[e & 1], false);
      w[e] = __builtin_bit_cast(uint32_t, pr);
    }
    pf[kb][k2] = __builtin_bit_cast(bf16x8, w);
  };
  // The whole tile.
  auto probs = [&](const f32x16(&s)[2], bf16x8(&pf)[2][2], float& psum) {
    float ps[2] = {0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) probs_part(s, kb, k2, pf, ps);
    psum = ps[0] + ps[1];
  };
  // O^T (d x queries) += V^T P^T.  Contraction slot (lg, e) of K-step
  // (kb, k2) is S^T row kb*32 + 16 k2 + 8 (e/4) + 4 lg + e%4, i.e. key
  // kb*32 + 16 k2 + 8 lg + e: eight consecutive keys, one 16-byte chunk
  // (4 kb + 2 k2 + lg) of the V^T row.
  auto pv = [&](const bf16x8(&pf)[2][2], int vbuf) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int db = 0; db < ND; ++db) {
        const int kb = ks >> 1, k2 = ks & 1;
        const int vr = db * 32 + lr;
        const bf16x8 vf = *reinterpret_cast<const bf16x8*>(Vs + vbuf * Ld::V_ELEMS + vr * VLD +
                                                            swz<8>(vr, 4 * kb + 2 * k2 + lg) * 8);
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[kb][k2], o[db], 0, 0, 0);
      }
  };

  // Processing order of the key tiles: the ragged tile (if any) first, then
  // the full tiles in order.  u >= 1 maps to the full tile u - has_tail.
  const int tiles = (Li + BKV - 1) / BKV;
  const int t0 = KS > 1 ? tiles * grp / KS : 0;  // first tile of this key range
  const int nkv = KS > 1 ? tiles * (grp + 1) / KS - t0 : tiles;
  const int has_tail = grp == KS - 1 && (Li % BKV) != 0;
  // One pipeline iteration: sc holds the exp2 arguments of processed tile
  // it (against the reference m); S of tile it+1 goes to sn (on the last
  // tile this reads a stale buffer and is dropped).
  //
  // d = 128 (MFMA-bound): the row max of S_{it+1} and its shift run under
  // the P V MFMAs, and the lazy rescale is decided at the top of the next
  // iteration.  d = 64 (VALU-bound: half the MFMA work per score):
  // optimistic softmax, no row max.  The probabilities are formed against
  // the current reference; a lane whose bf16 sum stays <= 2^8 had every
  // p <= 2^8 (the lazy bound).  Otherwise (rare) the wave takes the true row
  // max of the shifted tile, moves the reference to it, rescales O and l,
  // and forms the probabilities again.
  constexpr bool kOptimistic = D == 64;
  auto iter = [&](f32x16(&sc)[2], f32x16(&sn)[2], int it) {
    if (it + 2 < nkv) stage_k_dma(it & 1, (t0 + it + 2 - has_tail) * BKV);
    if (it + 1 < nkv) stage_v_dma((it + 1) & 1, (t0 + it + 1 - has_tail) * BKV);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!kOptimistic) {
      m_run = m_nx;
      if (__any(g_nx)) {
        l_run *= a_nx;
#pragma unroll
        for (int db = 0; db < ND; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= a_nx;
        if constexpr (kPre) {
          sub_all(sc, d_nx);
          // -m_run in place: (-m) - d equals -(m + d) exactly, and updating
          // cneg's own registers spares the common path a 16-register copy.
#pragma unroll
          for (int r = 0; r < 16; ++r) cneg[r] -= d_nx;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    bf16x8 pf[2][2];
    float psum;
    if constexpr (kPre && !kOptimistic) {
      // The exponentials of the first key block under the score MFMAs of the
      // next tile, those of the second under the first half of the P V
      // MFMAs (which use only the first block), the row max of the next
      // tile under the second half; exponentials (transcendental unit) and
      // the other VALU work in separate groups, one or two of each per MFMA.
      float ps[2] = {0.f, 0.f};
      probs_part(sc, 0, 0, pf, ps);
      probs_part(sc, 0, 1, pf, ps);
      scores(sn, (it + 1) & 1);
      probs_part(sc, 1, 0, pf, ps);
      probs_part(sc, 1, 1, pf, ps);
      psum = ps[0] + ps[1];
      l_run += psum;
      pv(pf, it & 1);
      row_max_check(sn);
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
      for (int i = 0; i < 2 * NK; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, (16 + 2 * NK - 1) / (2 * NK), 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (16 + 2 * NK - 1) / (2 * NK), 0);
      }
#pragma unroll
      for (int i = 0; i < 2 * ND; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x400, (16 + 2 * ND - 1) / (2 * ND), 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (18 + 2 * ND - 1) / (2 * ND), 0);
      }
#pragma unroll
      for (int i = 0; i < 2 * ND; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (24 + 2 * ND - 1) / (2 * ND), 0);
      }
    } else {
    probs(sc, pf, psum);
    scores(sn, (it + 1) & 1);
    if constexpr (kOptimistic) {
      // Each score MFMA with one fragment read and a share of the
      // exponentials.
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
      for (int i = 0; i < 2 * NK; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (66 + 2 * NK - 1) / (2 * NK), 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (__any(!(psum <= 256.0f))) {
        float mx = sc[0][0];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[kb][r]);
        mx = half_swap_max(mx);
        const float d = mx > 0.0f ? mx : 0.0f;
        const float alpha = __builtin_amdgcn_exp2f(-d);
        m_run += d;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < ND; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        sub_all(sc, d);
        if constexpr (kPre) {
          sub_all(sn, d);  // formed against the old reference
          set_cneg(-m_run);
        }
        probs(sc, pf, psum);
      }
      __builtin_amdgcn_sched_barrier(0);
      l_run += psum;
      pv(pf, it & 1);
      if constexpr (!kPre) {
        shift(sn);
        // Each P V MFMA with one fragment read and a share of the shift.
#pragma unroll
        for (int i = 0; i < 4 * ND; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, (32 + 4 * ND - 1) / (4 * ND), 0);
        }
      }
    } else {
      l_run += psum;
      pv(pf, it & 1);
      row_max_shift(sn);
      // Four fragment reads ahead, then each score MFMA with one more read
      // and a share of the exponentials, then each P V MFMA with one read
      // and a share of the row max and shift of the next tile.
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
      for (int i = 0; i < 2 * NK; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (66 + 2 * NK - 1) / (2 * NK), 0);
      }
#pragma unroll
      for (int i = 0; i < 4 * ND; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (56 + 4 * ND - 1) / (4 * ND), 0);
      }
    }
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0);  // this iteration's staging has landed
    __builtin_amdgcn_s_barrier();
  };

  f32x16 sa[2], sb[2];
  if (has_tail) {
    stage_tail(0, (tiles - 1) * BKV);
  } else if (KS == 1 || nkv > 0) {
    stage_k_dma(0, t0 * BKV);
    stage_v_dma(0, t0 * BKV);
  }
  if (nkv > 1) stage_k_dma(1, (t0 + 1 - has_tail) * BKV);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if constexpr (kPre) set_cneg(0.0f);
  scores(sa, 0);
  // Every wave has read K tile 0 before the first iteration restages its
  // buffer (a wave running ahead would otherwise overwrite it).
  __syncthreads();
  if (has_tail) {
    // Keys past L get score -inf.  S^T row kb*32 + 8 (r/4) + 4 lg + r%4
    // holds key j0 + key_perm(row).
    const int j0 = (tiles - 1) * BKV;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = j0 + kb * 32 + 16 * (r >> 3) + 8 * lg + 4 * ((r >> 2) & 1) + (r & 3);
        if (key >= Li) sa[kb][r] = -__builtin_inff();
      }
  }
  // The first reference is the first tile's row max, unless that lies so far
  // below 0 (masked keys: scores of -inf or of the type's lowest values) that
  // scores added to it would lose their digits, or that it is no score at all.
  // Then it is the true maximum over this range's keys, from a pass of its own
  // over K in global memory: no such tile may stand for the range.
  bool no_key = false;  // no score of this range can count beside another range's
  auto first_ref = [&]() {
    first_max(sa);
    if (__any(m_run < kLowRef)) {
      float mx = -__builtin_inff();
#pragma unroll 1
      for (int b = 0; b < 2 * nkv; ++b) {
        const int key = min(t0 * BKV + b * 32 + lr, Li - 1);  // past the end: the last key again
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
          const bf16x8 kf =
              *reinterpret_cast<const bf16x8*>(Kh + (uint32_t)(key * D + (2 * kk + lg) * 8));
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk], s, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
      }
      mx = half_swap_max(mx);
      if (m_run < kLowRef) m_run = kPre ? mx : mx * scale_log2;
      // Plain Q: against a reference of 2^30 and more the shift's multiply-add
      // leaves the rounding of m itself, beyond what exp2 can hold.
      if (KS > 1 && (m_run == -__builtin_inff() || (!kPre && m_run < -0x1p30f))) {
        no_key = true;
        m_run = 0.f;
      }
    }
  };
  first_ref();
  if constexpr (kPre) {  // sa was formed with m = 0
    sub_all(sa, m_run);
    set_cneg(-m_run);
  } else {
    shift(sa);
  }
  m_nx = m_run;
  int it = 0;
  // The full-size d = 128 loop's time depends on where its code lies in the
  // 32-byte fetch windows: 12 heads of 32760 tokens take 5247-5254 us with the
  // loop's first instruction 20, 28, 0 or 4 bytes into one, 5267-5277 at 8, 12,
  // 16 or 24 (16 placements, nine runs each).  Pinned to the start of one: the
  // 15 words from here to the loop end at a 64-byte boundary.  The other
  // forms showed no such difference.
  if constexpr (D == 128 && KS == 1 && kPre) asm volatile(".p2align 6\n\ts_nop 0");
  for (; it + 1 < nkv; it += 2) {
    iter(sa, sb, it);
    iter(sb, sa, it + 1);
  }
  if (it < nkv) iter(sa, sb, it);

  if constexpr (KS > 1) {
    // The longest range's barriers, one per tile.
    const int most = (tiles + KS - 1) / KS;
    for (int i = nkv; i < most; ++i) __builtin_amdgcn_s_barrier();
    if (nkv == 0) l_run = 0.f;  // scores of a stale buffer were formed and dropped
    if (nkv == 0 || no_key) m_run = -__builtin_inff();  // weight 0
    l_run += __shfl_xor(l_run, 32, 64);
    __syncthreads();
    // [wave][block, group of four rows][lane], then (m, l) per wave and lane.
    constexpr int NCH = ND * 4;
    static_assert(NW * (NCH * 16 + 8) * 64 <= attn_lds_bytes<D, NW, KS>() && NCH % KS == 0, "");
    f32x4* po = reinterpret_cast<f32x4*>(smem);
    float2* pm = reinterpret_cast<float2*>(smem + NW * NCH * 16 * 64);
#pragma unroll
    for (int db = 0; db < ND; ++db)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg)
        po[(wave_wg * NCH + db * 4 + rg) * 64 + lane] =
            f32x4{o[db][4 * rg], o[db][4 * rg + 1], o[db][4 * rg + 2], o[db][4 * rg + 3]};
    pm[wave_wg * 64 + lane] = make_float2(m_run, l_run);
    __syncthreads();
    float w[KS], mx = -__builtin_inff(), l = 0.f;
#pragma unroll
    for (int g = 0; g < KS; ++g) {
      w[g] = pm[(g * QW + wave) * 64 + lane].x;
      mx = fmaxf(mx, w[g]);
    }
#pragma unroll
    for (int g = 0; g < KS; ++g) {
      w[g] = __builtin_amdgcn_exp2f(w[g] - mx);
      l += w[g] * pm[(g * QW + wave) * 64 + lane].y;
    }
    const float inv = 1.0f / l;
    if (qrow < L) {
      bf16* orow = O + qrow * o_ld + (int64_t)head * D;
#pragma unroll
      for (int i = 0; i < NCH / KS; ++i) {  // each group stores its share of the row blocks
        const int c = grp * (NCH / KS) + i;
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < KS; ++g) a += w[g] * po[((g * QW + wave) * NCH + c) * 64 + lane];
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)(a[e] * inv);
        *reinterpret_cast<bf16x4*>(orow + (c >> 2) * 32 + 8 * (c & 3) + 4 * lg) = v;
      }
    }
    return;
  }
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = 1.0f / l_tot;
  if (qrow < L) {
    bf16* orow = O + qrow * o_ld + (int64_t)head * D;
#pragma unroll
    for (int db = 0; db < ND; ++db)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (bf16)(o[db][rg * 4 + e] * inv);
        *reinterpret_cast<bf16x4*>(orow + db * 32 + 8 * rg + 4 * lg) = w;
      }
  }
}

// ------------------------------------------------------------------ fp32

// fp32 path: flash-style on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32: products and sums in fp32), 32 queries per
// workgroup.  The four waves hold the same queries and take every fourth
// tile of 32 keys each, so that the short sequences of the fp32
// configuration still give two waves per SIMD; their partial softmaxes meet
// in LDS and are added in wave order.  Scores are formed transposed as in the
// bf16 path: a lane owns one query and 16 of the tile's keys, and with
// contraction slot r of half-wave h standing for key 8 (r / 4) + 4 h + r % 4
// the probabilities in accumulator layout are the B operand of
// O^T = V^T P^T, and the matching V^T operand is one 16-byte load per four
// MFMAs.  K and V^T come straight from global memory (16 bytes per lane and
// four MFMAs of 64 cycles), V of a tile ahead of its scores and its softmax, K
// of the next tile under P V and the first scores; Q is read from LDS.
// Scores are added from sums of 32 products and O from sums of a tile (one
// chain of all of them was up to 1.8 times as far from 64 bits: 3.3e-7 -> 1.8e-7
// at 40 keys of 128, 4.1e-7 -> 2.4e-7 at 900 of 64).  Bound by the matrix unit
// (4 L^2 d flops a head at 157 TFLOP/s).  The one-query-per-wave kernel
// before it took 2239 us at 16 heads x 1013 x 64 (V^T read four bytes a lane
// from 64 rows), and a 1013-token fp32 block of that width 2824 us; the block
// took 609 us with this kernel and takes 282 us with the fp32 GEMM's.
template <int D>
__global__ __launch_bounds__(256, 2) void attn_f32_kernel(const float* __restrict__ Q,
                                                          const float* __restrict__ Kp,
                                                          const float* __restrict__ Vt, int64_t L,
                                                          int64_t vt_ld, int n_heads,
                                                          float* __restrict__ O, int64_t o_ld,
                                                          float scale, const int32_t* pred) {
  if (pred && *pred == 0) return;
  constexpr int BT = 32;       // queries per workgroup, keys per tile
  constexpr int NC = D / 4;    // 16-byte chunks per row
  constexpr int ND = D / 32;   // 32-row blocks of O^T
  // Q as [chunk][query] during the loop, the waves' O^T as
  // [wave][chunk][query] after it.
  __shared__ f32x4 lds[4 * NC * BT];
  __shared__ float ml[2][4][BT];
  const uint32_t n_qt = (uint32_t)((L + BT - 1) / BT);
  const uint32_t item = attn_xcd_remap(blockIdx.x, n_qt * n_heads);
  const int head = (int)(item / n_qt);
  const int64_t q0 = (int64_t)(item - head * n_qt) * BT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const float* Kh = Kp + (int64_t)head * L * D;
  const float* Vh = Vt + (int64_t)head * D * vt_ld;
  for (int i = tid; i < NC * BT; i += 256) {
    const int c = i % NC, r = i / NC;
    const int64_t row = q0 + r < L ? q0 + r : L - 1;
    lds[c * BT + r] = *reinterpret_cast<const f32x4*>(Q + ((int64_t)head * L + row) * D + 4 * c);
  }
  __syncthreads();

  f32x16 o[ND];
#pragma unroll
  for (int db = 0; db < ND; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.f;
  float m_run = -__builtin_inff(), l_run = 0.f;
  const int64_t nt = (L + BT - 1) / BT;
  f32x4 kf[NC / 2];
  auto load_k = [&](int64_t t, int j0, int j1) {
    const int64_t key = t * BT + lr;
    const float* kr = Kh + (key < L ? key : L - 1) * D + 4 * lg;
#pragma unroll
    for (int j = j0; j < j1; ++j) kf[j] = *reinterpret_cast<const f32x4*>(kr + 8 * j);
  };
  if (wave < nt) load_k(wave, 0, NC / 2);
  for (int64_t t = wave; t < nt; t += 4) {
    // V in two halves, the second once the scores have left K's registers; half
    // of the next K once the first is used, the rest after P V.
    f32x4 vf[ND][4];
    auto load_v = [&](int db0, int db1) {
#pragma unroll
      for (int db = db0; db < db1; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int64_t key0 = t * BT + 8 * g + 4 * lg;
          vf[db][g] = *reinterpret_cast<const f32x4*>(Vh + (int64_t)(db * 32 + lr) * vt_ld +
                                                   (key0 < L ? key0 : 0));
        }
    };
    load_v(0, ND / 2);
    __builtin_amdgcn_sched_barrier(0);
    // Sums of 32 products, added up: a chain of all d would round d times.
    const f32x16 zero = {};
    f32x16 s = zero;
#pragma unroll
    for (int j0 = 0; j0 < NC / 2; j0 += 4) {
      if (D == 128 && j0) __builtin_amdgcn_sched_barrier(0);  // few reads of Q held ahead
      f32x16 part = zero;
#pragma unroll
      for (int j = j0; j < j0 + 4; ++j) {
        const f32x4 qf = lds[(2 * j + lg) * BT + lr];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          part = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][i], qf[i], part, 0, 0, 0);
      }
      s += part;
    }
    __builtin_amdgcn_sched_barrier(0);
    load_v(ND / 2, ND);
    __builtin_amdgcn_sched_barrier(0);
    if (t * BT + BT > L) {  // the ragged last tile: keys past L, V^T's padding
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (t * BT + 8 * g + 4 * lg + e >= L) {
            s[4 * g + e] = -__builtin_inff();
#pragma unroll
            for (int db = 0; db < ND; ++db) vf[db][g][e] = 0.f;
          }
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    const float m_new = fmaxf(m_run, half_swap_max(mx) * scale);
    // A tile of -inf scores alone leaves no reference: its probabilities are 0.
    const float m_use = m_new == -__builtin_inff() ? 0.f : m_new;
    if (__any(m_new > m_run)) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < ND; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
    }
    m_run = m_new;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale, -m_use));
      l_run += s[r];
    }
#pragma unroll
    for (int db = 0; db < ND; ++db) {  // a tile's sum, then added to the others'
      if (db == ND / 2) {
        __builtin_amdgcn_sched_barrier(0);
        if (t + 4 < nt) load_k(t + 4, 0, NC / 4);
        __builtin_amdgcn_sched_barrier(0);
      }
      f32x16 part = zero;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[db][r >> 2][r & 3], s[r], part, 0, 0, 0);
      o[db] += part;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (t + 4 < nt) load_k(t + 4, NC / 4, NC / 2);
  }
  l_run += __shfl_xor(l_run, 32, 64);
  __syncthreads();  // every wave is done with Q
#pragma unroll
  for (int db = 0; db < ND; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      lds[(wave * NC + (db * 4 + g) * 2 + lg) * BT + lr] =
          f32x4{o[db][4 * g], o[db][4 * g + 1], o[db][4 * g + 2], o[db][4 * g + 3]};
  if (lg == 0) {
    ml[0][wave][lr] = m_run;
    ml[1][wave][lr] = l_run;
  }
  __syncthreads();
  for (int i = tid; i < NC * BT; i += 256) {
    const int r = i % BT, c = i / BT;
    if (q0 + r >= L) continue;
    float m = ml[0][0][r];
#pragma unroll
    for (int w = 1; w < 4; ++w) m = fmaxf(m, ml[0][w][r]);
    float l = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {  // a wave without keys has m = -inf, weight 0
      const float a = __builtin_amdgcn_exp2f(ml[0][w][r] - m);
      l += a * ml[1][w][r];
      acc += a * lds[(w * NC + c) * BT + r];
    }
    *reinterpret_cast<f32x4*>(O + (q0 + r) * o_ld + (int64_t)head * D + 4 * c) = acc * (1.0f / l);
  }
}

// fp32 with few keys: one wave per (head, query), lane j takes key j's score
// and the wave adds the values one key at a time, lane l for dims l, l + 64,
// ....  Bound by its loads' latency.  The matrix kernel's chain for a single
// tile of keys (64 or 128 MFMAs of 64 cycles, and the merge) takes longer there:
// 24 heads of 64 / 128, 3 tokens 3.4 / 4.6 us against 5.8 / 9.3, 12 tokens 4.6 /
// 6.9 against 5.4 / 8.5, 18 equal, 24 tokens 6.2 / 10.1 against 5.5 / 8.4.
constexpr int kFewKeys = 18;  // at most 64
template <int D>
__global__ __launch_bounds__(256) void attn_f32_few_kernel(const float* __restrict__ Q,
                                                           const float* __restrict__ Kp,
                                                           const float* __restrict__ Vt, int64_t L,
                                                           int64_t vt_ld, int n_heads,
                                                           float* __restrict__ O, int64_t o_ld,
                                                           float scale, const int32_t* pred) {
  if (pred && *pred == 0) return;
  constexpr int C = D / 64;  // output dims per lane
  const int lane = threadIdx.x & 63, Li = (int)L;
  const uint32_t wq = (blockIdx.y * gridDim.x + blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (wq >= (uint32_t)Li * n_heads) return;  // whole wave; no barriers below
  const int head = (int)(wq / (uint32_t)Li);
  const int64_t qrow = wq - (uint32_t)head * Li;
  const float* Vh = Vt + (int64_t)head * D * vt_ld;
  float s = -__builtin_inff();
  if (lane < Li) {
    const float4* q4 = reinterpret_cast<const float4*>(Q + ((int64_t)head * L + qrow) * D);
    const float4* k4 = reinterpret_cast<const float4*>(Kp + ((int64_t)head * L + lane) * D);
    float a = 0.f;
#pragma unroll
    for (int d4 = 0; d4 < D / 4; ++d4) {
      const float4 qv = q4[d4], kv = k4[d4];
      a += qv.x * kv.x + qv.y * kv.y + qv.z * kv.z + qv.w * kv.w;
    }
    s = a * scale;
  }
  float m = s;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  const float p = lane < Li ? exp2f(s - m) : 0.f;
  const float inv = 1.0f / wave_sum(p);
  float o[C];
#pragma unroll
  for (int c = 0; c < C; ++c) o[c] = 0.f;
#pragma unroll 4
  for (int j = 0; j < Li; ++j) {
    const float pj = __shfl(p, j, 64);
#pragma unroll
    for (int c = 0; c < C; ++c) o[c] += pj * Vh[(int64_t)(lane + 64 * c) * vt_ld + j];
  }
  float* orow = O + qrow * o_ld + (int64_t)head * D;
#pragma unroll
  for (int c = 0; c < C; ++c) orow[lane + 64 * c] = o[c] * inv;
}

template <int D, int NW, bool kPre, int KS>
hipError_t launch_bf16_form(int n_heads, int64_t L, const void* q, const void* k, const void* vt,
                            int64_t vt_ld, void* o, int64_t o_ld, hipStream_t s,
                            const int32_t* pred) {
  constexpr int BQ = 32 * NW / KS;
  constexpr size_t kLds = attn_lds_bytes<D, NW, KS>();
  // The dynamic-LDS attribute is set once per device (one bit each).
  static std::atomic<uint64_t> attr_set{0};
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
  if (!(attr_set.load(std::memory_order_acquire) & bit)) {
    err = hipFuncSetAttribute((const void*)attn_bf16_kernel<D, NW, kPre, KS>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (err != hipSuccess) return err;
    attr_set.fetch_or(bit, std::memory_order_release);
  }
  const float scale_log2 = attn_q_scale(D);
  dim3 grid((unsigned)(((L + BQ - 1) / BQ) * n_heads));
  hipLaunchKernelGGL((attn_bf16_kernel<D, NW, kPre, KS>), grid, dim3(64 * NW), kLds, s,
                     (const bf16*)q, (const bf16*)k, (const bf16*)vt, L, vt_ld, n_heads,
                     (bf16*)o, o_ld, scale_log2, pred);
  return hipGetLastError();
}

// Waves per workgroup: 8 for d = 128 (a staged K/V tile feeds 256 queries),
// 4 for d = 64 (finer grid for the shorter sequences of that configuration),
// 8 where the keys are split.
template <int D, bool kPre>
hipError_t launch_bf16(int n_heads, int64_t L, const void* q, const void* k, const void* vt,
                       int64_t vt_ld, void* o, int64_t o_ld, hipStream_t s,
                       const int32_t* pred) {
  const int ranges = attn_key_ranges(D, n_heads, L, device_cus());
  if constexpr (D == 64) {
    if (ranges == 4)
      return launch_bf16_form<64, 8, kPre, 4>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred);
  }
  if (ranges == 2)
    return launch_bf16_form<D, 8, kPre, 2>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred);
  return launch_bf16_form<D, D == 128 ? 8 : 4, kPre, 1>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s,
                                                        pred);
}

template <int D>
hipError_t launch_f32(int n_heads, int64_t L, const void* q, const void* k, const void* vt,
                      int64_t vt_ld, void* o, int64_t o_ld, hipStream_t s, const int32_t* pred,
                      bool q_prescaled) {
  const float scale = q_prescaled ? 1.0f : attn_q_scale(D);
  if (L <= kFewKeys) {
    // Up to 2^24 workgroups of four queries, in two dimensions beyond 2^22: a
    // dimension holds fewer than 2^32 work-items.
    const int64_t wgs = (L * n_heads + 3) / 4, gy = (wgs + (1 << 22) - 1) >> 22;
    hipLaunchKernelGGL(attn_f32_few_kernel<D>, dim3((unsigned)((wgs + gy - 1) / gy), (unsigned)gy),
                       dim3(256), 0, s, (const float*)q, (const float*)k, (const float*)vt, L,
                       vt_ld, n_heads, (float*)o, o_ld, scale, pred);
    return hipGetLastError();
  }
  // Fewer than 2^22 workgroups: seq_len * n_heads is below 2^26.
  dim3 grid((unsigned)((L + 31) / 32 * n_heads));
  hipLaunchKernelGGL(attn_f32_kernel<D>, grid, dim3(256), 0, s, (const float*)q,
                     (const float*)k, (const float*)vt, L, vt_ld, n_heads, (float*)o, o_ld, scale,
                     pred);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention(int dtype, int n_heads, int64_t L, int d, const void* q,
                            const void* k, const void* vt, int64_t vt_ld, void* o,
                            hipStream_t s, const int32_t* pred, int64_t o_ld,
                            bool q_prescaled) {
  if (L == 0) return hipSuccess;
  if (o_ld == 0) o_ld = (int64_t)n_heads * d;
  if (dtype == ACID_BF16) {
    if (d == 64)
      return q_prescaled ? launch_bf16<64, true>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred)
                         : launch_bf16<64, false>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred);
    if (d == 128)
      return q_prescaled ? launch_bf16<128, true>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred)
                         : launch_bf16<128, false>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred);
  } else {
    if (d == 64) return launch_f32<64>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred, q_prescaled);
    if (d == 128) return launch_f32<128>(n_heads, L, q, k, vt, vt_ld, o, o_ld, s, pred, q_prescaled);
  }
  return hipErrorInvalidValue;
}

}  // namespace acid
