// Fused GEMMs of the DiT block: y = a W + b with the epilogues the block
// needs (plain, tanh-GELU, gated residual add, QKV head split, Euler update).
//
// bf16 path: MFMA v_mfma_f32_32x32x16_bf16 (gfx950), fp32 accumulate.
//   Macro tile 256 (tokens) x 256 (features), K in steps of 64, 8 waves in a
//   2 x 4 grid (two per SIMD), each wave 128 x 64 = 4 x 2 MFMA blocks of
//   32 x 32.  Operands go global -> LDS directly (global_load_lds_dwordx4,
//   no staging registers) into a ring of 32 KB operand tiles (three for
//   the activations, requested about 1.75 K-steps ahead, two for the
//   weights, 1.25 ahead: 160 KB, the whole LDS), K-contiguous 128-byte rows
//   (whole cache lines, so the L2 request rate stays within budget) with an
//   XOR swizzle that is conflict-free for gfx950's 64 LDS banks.  One
//   barrier per K-step, placed before the last 16-wide sub-step so the
//   weight refill and the next stage's first fragment reads hide behind its
//   MFMAs (the activation refill runs under the first sub-step); all other
//   fragment reads are software-pipelined one sub-step ahead.  A wave that
//   issues global loads holds back its own MFMA issue, so two waves share
//   each SIMD and one of them issues the DMAs of both: the other only reads
//   fragments and issues MFMAs.  A 256 x 256 tile halves the operand bytes
//   per flop of a 256 x 128 tile (operand traffic also costs clock under
//   the power cap).  The activation tile feeds MFMA operand A and the weight
//   tile operand B, so the accumulator holds C with lanes along features:
//   every epilogue store is a run of consecutive features of one token row
//   (coalesced), and bias / gate are one value per lane.  Workgroups are
//   remapped so each XCD (8 per MI355X, own L2) works on a contiguous group
//   of tiles that share activation rows.
//   Launches whose 256 x 256 tiles would leave CUs idle (few rows) take
//   256 x 128, 128 x 128 or 64 x 64 tiles (gemm_ring_kernel), with the K range
//   split too where it is long and the tiles few: one 1560-token 30-block step
//   8.62 -> 5.82 ms, the 1024-token loop 5.47 -> 2.2 ms, a 226 x 3072 x 3072
//   product 52.5 -> 11.4 us.
// fp32 path: the fp32 matrix instruction on 64 x 64 or 32 x 32 tiles, for the
//   fp32 configuration.
#include <atomic>
#include <type_traits>

#include "common.h"
#include "gemm_form.h"

namespace acid {

namespace {

struct Epi {
  const float* bias;
  const float* gate;
  void* out;
  float* v_out;
  void* q;
  void* k;
  void* vt;
  int64_t vt_ld;
  int64_t M;
  int n_heads, head_dim, H;
  float dsigma;
  const int32_t* pred;  // device gate's decision: no work when *pred == 0
  const float* bias2;   // GATE_RESIDUAL: optional second bias
  int64_t out_ld;       // QKV_GELU: row stride of the GELU output
  int n_qkv;            // QKV_GELU: columns [0, n_qkv) are Q | K | V
  float q_mul;          // QKV kinds: factor on the Q columns (1: plain Q)
  float* split_ws;      // bf16: fp32 partial tiles of a K split (nullptr: no split)
};

// Q | K | V head-major destination of column c < 3 H (which = c / H).
template <typename T>
__device__ __forceinline__ T* qkv_dst(const Epi& e, int c, int64_t& stride) {
  const int which = c / e.H, cc = c - which * e.H;
  const int head = cc / e.head_dim, dd = cc - head * e.head_dim;
  if (which < 2) {
    stride = e.head_dim;
    return static_cast<T*>(which == 0 ? e.q : e.k) + (int64_t)head * e.M * e.head_dim + dd;
  }
  stride = 1;
  return static_cast<T*>(e.vt) + ((int64_t)head * e.head_dim + dd) * e.vt_ld;
}

// Epilogue of one output column n: bias, gate and destination are resolved
// once; put(m, acc) then stores row m.
template <int KIND, typename T>
struct ColEpi {
  float bias, gate;
  T* dst_t;
  float* dst_f;
  float* v_f;
  int64_t stride;
  float dsigma;
  bool gelu;  // QKV_GELU: this column is in the GELU part
  float qmul;  // QKV kinds: e.q_mul on the Q columns, else 1
  __device__ __forceinline__ ColEpi(const Epi& e, int n, int N) {
    bias = e.bias[n];
    if (KIND == ACID_EPI_GATE_RESIDUAL && e.bias2) bias += e.bias2[n];
    gate = (KIND == ACID_EPI_GATE_RESIDUAL) ? e.gate[n] : 0.f;
    dsigma = e.dsigma;
    dst_t = nullptr;
    dst_f = nullptr;
    v_f = nullptr;
    stride = N;
    gelu = false;
    qmul = ((KIND == ACID_EPI_QKV || KIND == ACID_EPI_QKV_GELU) && n < e.H) ? e.q_mul : 1.f;
    if constexpr (KIND == ACID_EPI_QKV) {
      dst_t = qkv_dst<T>(e, n, stride);
    } else if constexpr (KIND == ACID_EPI_QKV_GELU) {
      if (n < e.n_qkv) {
        dst_t = qkv_dst<T>(e, n, stride);
      } else {
        gelu = true;
        dst_t = static_cast<T*>(e.out) + (n - e.n_qkv);
        stride = e.out_ld;
      }
    } else if constexpr (KIND == ACID_EPI_BIAS_GELU) {
      dst_t = static_cast<T*>(e.out) + n;
    } else {
      dst_f = static_cast<float*>(e.out) + n;
      if (KIND == ACID_EPI_EULER && e.v_out) v_f = e.v_out + n;
    }
  }
  static constexpr bool kRmw = KIND == ACID_EPI_GATE_RESIDUAL || KIND == ACID_EPI_EULER;
  // Read-modify-write kinds read the old value first (batched by the caller).
  __device__ __forceinline__ float old(int64_t m) const {
    if constexpr (kRmw) return dst_f[m * stride];
    return 0.f;
  }
  __device__ __forceinline__ void put_old(int64_t m, float acc, float prev) const {
    const float y = acc + bias;
    if constexpr (KIND == ACID_EPI_GATE_RESIDUAL) {
      dst_f[m * stride] = prev + gate * y;
    } else if constexpr (KIND == ACID_EPI_EULER) {
      if (v_f) v_f[m * stride] = y;
      dst_f[m * stride] = prev + dsigma * y;
    } else {
      put(m, acc);
    }
  }
  __device__ __forceinline__ void put(int64_t m, float acc) const {
    static_assert(!kRmw, "read-modify-write kinds go through put_old");
    const float y = acc + bias;
    if constexpr (KIND == ACID_EPI_BIAS) {
      dst_f[m * stride] = y;
    } else if constexpr (KIND == ACID_EPI_BIAS_GELU) {
      if constexpr (sizeof(T) == 2)
        dst_t[m * stride] = (T)gelu_tanh_fast(y);
      else
        dst_t[m * stride] = (T)gelu_tanh(y);
    } else if constexpr (KIND == ACID_EPI_QKV) {
      dst_t[m * stride] = (T)(y * qmul);
    } else {
      float z = y * qmul;
      if (gelu) {
        if constexpr (sizeof(T) == 2)
          z = gelu_tanh_fast(y);
        else
          z = gelu_tanh(y);
      }
      dst_t[m * stride] = (T)z;
    }
  }
};

// Bijection from dispatch order to tile order giving XCD x (workgroups
// bid = x, x+8, ...) the contiguous tile range of its share.  Tile numbers
// are below 2^29 (the entry bounds the 256 x 256 tiles by 2^23) and divided in 32
// bits: the 64-bit divisions of a tile's coordinates were a chain that every
// workgroup waited for before its first load.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t bid, uint32_t T) {
  constexpr uint32_t NX = 8;
  const uint32_t x = bid % NX, local = bid / NX;
  const uint32_t q = T / NX, r = T % NX;
  return (x < r) ? x * (q + 1) + local : r * (q + 1) + (x - r) * q + local;
}

// Tile t -> (tm, tn) in groups of GM token tiles, feature tiles inner.
// The 32 tiles an XCD runs at once then share few activation row blocks
// (streamed once from HBM) and many weight column blocks (re-read by every
// row block, so they come from the on-package cache): groups of 2 measured
// 3-6% faster than 8 on the model shapes here (4 and 3 within noise of 2).
template <uint32_t GM = 2>
__device__ __forceinline__ void tile_coords(uint32_t t, int64_t tiles_m, int tiles_n, int64_t& tm,
                                            int& tn) {
  const uint32_t per_group = GM * (uint32_t)tiles_n;
  const uint32_t g = t / per_group;
  const uint32_t first = g * GM;
  const uint32_t gsize = min(GM, (uint32_t)tiles_m - first);
  const uint32_t w = t - g * per_group;
  const uint32_t col = w / gsize;
  tm = first + (w - col * gsize);
  tn = (int)col;
}

// ------------------------------------------------------------ bf16 MFMA

typedef __attribute__((address_space(3))) void lds_void_t;

constexpr int BM = kGemmTile, BN = kGemmTile, BK = kGemmStep;
constexpr int kWaves = 8;                // 2 (tokens) x 4 (features), two per SIMD
constexpr int kTileElems = 256 * BK;     // one operand tile per stage (32 KB)
constexpr int64_t kSplitItemFloats = 256 * 256;  // one K-split partial tile (256 KB)

// One 16-byte-per-lane LDS-DMA: lane l reads 16 bytes at base + off(l) and
// writes LDS bytes [lds + 16 l, +16).  base and lds are wave-uniform.
// Issued as inline assembly so the compiler's wait-count pass does not see
// it (that pass cannot order DMA completions against LDS reads and would
// drain every read); completion is waited for explicitly.  M0 (the DMA's
// LDS base) is set here and nothing else in these kernels uses M0.
__device__ __forceinline__ void dma16(uint64_t base, uint32_t off_bytes, uint32_t lds_byte) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(off_bytes), "s"(base), "s"(lds_byte)
      : "memory");
}
__device__ __forceinline__ uint64_t uniform_ptr(const void* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ void wait_all() { __builtin_amdgcn_s_waitcnt(0); }

// Epilogue of one wave's block of an output tile: 32 MB rows from mw and
// 32 NB columns from nw, out of the MFMA accumulators.  full: every row of
// the block is below M.
template <int KIND, typename T, int MB, int NB, int LOADS = 32>
__device__ __forceinline__ void tile_epilogue(const Epi& e, f32x16 (&acc)[MB][NB], int64_t M,
                                              int N, int64_t mw, int nw, bool full, int lane) {
  const int lr = lane & 31, lg = lane >> 5;
  // D[i][j] of a 32x32 block: j = lane % 32, i = 8 (r / 4) + 4 (lane / 32) + r % 4.
  // A lane owns one feature column per 32-wide block: set up its epilogue
  // once, then handle its 16 MB rows of that column.  Full tiles skip the row
  // check (a per-element branch would serialise every load behind a wait);
  // read-modify-write kinds issue up to LOADS loads before their stores.
  const int64_t mrow = mw + 4 * lg;
  if constexpr (KIND == ACID_EPI_QKV || KIND == ACID_EPI_QKV_GELU) {
    // V columns are rows of V^T, whose tokens are contiguous: a lane holds 4
    // consecutive tokens per group r / 4 and its partner lane (l ^ 32) the
    // next 4, so one permlane32 swap per dword gives each lane 8 consecutive
    // tokens: 16-byte stores instead of 2-byte ones scattered over 32 rows.
    if (full && nw >= 2 * e.H && nw + 32 * NB <= 3 * e.H) {  // all columns in V
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int n = nw + nb * 32 + lr;
        const int cc = n - 2 * e.H;
        const int head = cc / e.head_dim, dd = cc - head * e.head_dim;
        T* vrow = static_cast<T*>(e.vt) + ((int64_t)head * e.head_dim + dd) * e.vt_ld;
        const float bias = e.bias[n];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
          if constexpr (sizeof(T) == 4) {  // 4 consecutive tokens are one 16-byte store
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              f32x4 v;
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = acc[mb][nb][4 * g + i] + bias;
              *reinterpret_cast<f32x4*>(vrow + mrow + mb * 32 + 8 * g) = v;
            }
          } else {
            uint32_t w[8];  // tokens 8 (r / 4) + 4 lg + r % 4 as bf16 pairs
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
              const bf16x2 pr = {(bf16)(acc[mb][nb][r] + bias), (bf16)(acc[mb][nb][r + 1] + bias)};
              w[r / 2] = __builtin_bit_cast(uint32_t, pr);
            }
            const int64_t t0 = mw + mb * 32 + 8 * lg;
#pragma unroll
            for (int p = 0; p < 2; ++p) {  // groups 2p (tokens +0..7) and 2p + 1 (+8..15)
              uint32_t lo[2], hi[2];
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const auto sw = __builtin_amdgcn_permlane32_swap(w[4 * p + h], w[4 * p + 2 + h],
                                                                 false, false);
                lo[h] = sw[0];
                hi[h] = sw[1];
              }
              const u32x4 v = {lo[0], lo[1], hi[0], hi[1]};
              *reinterpret_cast<u32x4*>(vrow + t0 + 16 * p) = v;
            }
          }
        }
      }
      return;
    }
  }
  const int rows_left = (int)(M - mrow < 32 * MB ? M - mrow : 32 * MB);
  if constexpr (!ColEpi<KIND, T>::kRmw) {
    if (full) {
      // The 32-column blocks of a wave fill the two halves of the same
      // 128-byte line of each output row (bf16): store them back to back so
      // the line is complete in the L2 before it can be written back.
      if constexpr (NB == 2) {
        const ColEpi<KIND, T> c0(e, nw + lr, N), c1(e, nw + 32 + lr, N);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int64_t m = mrow + mb * 32 + 8 * (r >> 2) + (r & 3);
            c0.put(m, acc[mb][0][r]);
            c1.put(m, acc[mb][1][r]);
          }
      } else {
        static_assert(NB == 1, "one or two column blocks per wave");
        const ColEpi<KIND, T> c0(e, nw + lr, N);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            c0.put(mrow + mb * 32 + 8 * (r >> 2) + (r & 3), acc[mb][0][r]);
      }
      return;
    }
    // The ragged last row tile: row offsets from mrow in 32 bits (a 64-bit
    // row per element made the register allocator spill).
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const ColEpi<KIND, T> ce(e, nw + nb * 32 + lr, N);
      // The column's bias has landed before the guarded stores: a load still
      // in flight there makes every guarded block wait for all earlier stores.
      asm volatile("" ::"v"(ce.bias));
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int dr = mb * 32 + 8 * (r >> 2) + (r & 3);
          if (dr < rows_left) ce.put(mrow + dr, acc[mb][nb][r]);
        }
    }
    return;
  } else {
    constexpr int G = MB % 2 || LOADS < 32 ? 1 : 2;  // row blocks per batch of loads
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const ColEpi<KIND, T> ce(e, nw + nb * 32 + lr, N);
      if (full) {
#pragma unroll
        for (int h = 0; h < MB / G; ++h) {  // a batch of loads in flight, then the stores
          float prev[G][16];
#pragma unroll
          for (int mb = 0; mb < G; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              prev[mb][r] = ce.old(mrow + (G * h + mb) * 32 + 8 * (r >> 2) + (r & 3));
#pragma unroll
          for (int mb = 0; mb < G; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              ce.put_old(mrow + (G * h + mb) * 32 + 8 * (r >> 2) + (r & 3),
                         acc[G * h + mb][nb][r], prev[mb][r]);
        }
      } else {
        // The ragged last row tile of a read-modify-write kind: loads from rows
        // clamped to M - 1 (always valid) batched as above, stores guarded.  A
        // load under the store's guard would wait for each element in turn.
#pragma unroll
        for (int h = 0; h < MB / G; ++h) {
          float prev[G][16];
#pragma unroll
          for (int mb = 0; mb < G; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int dr = (G * h + mb) * 32 + 8 * (r >> 2) + (r & 3);
              prev[mb][r] = ce.old(dr < rows_left ? mrow + dr : M - 1);
            }
#pragma unroll
          for (int mb = 0; mb < G; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) asm volatile("" ::"v"(prev[mb][r]));  // loads land here
#pragma unroll
          for (int mb = 0; mb < G; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int dr = (G * h + mb) * 32 + 8 * (r >> 2) + (r & 3);
              if (dr < rows_left) ce.put_old(mrow + dr, acc[G * h + mb][nb][r], prev[mb][r]);
            }
        }
      }
    }
  }
}

// Operand tiles are 256 rows x 64 (K-contiguous 128-byte rows: every row
// fetch is one whole line).  DMA instruction i (0..3) of wave w fills LDS
// bytes [(4 w + i) KB, +1 KB) = rows 32 w + 8 i .. +7; lane l lands in row
// 32 w + 8 i + l / 8, slot l % 8, which holds global chunk
// (l % 8) ^ ((row / 2) % 8) (= (l % 8) ^ (l / 16) for even i, ^ 4 more for
// odd i).  With 64 four-byte LDS banks a row spans half the banks, so 16
// consecutive fragment rows read at one chunk cover all 64 banks once.
//
// Eight waves, two per SIMD (waves w and w + 4): wave w issues the DMAs of
// both (a wave that issues global loads holds back its own MFMA issue), so
// wave w + 4 keeps the MFMA unit busy while wave w stalls.  Each wave owns
// 128 x 64 of the tile (4 x 2 blocks of 32 x 32, 128 accumulator registers).
//
// K split (grids whose last round of tiles would leave most CUs idle): the
// first tiles_main work items are whole tiles in the XCD-aware order; each of
// the remaining tiles is split into `split` equal K ranges, one work item
// each, which store their raw fp32 partial sums to e.split_ws for
// gemm_split_reduce_kernel.
template <int KIND>
__global__ __launch_bounds__(64 * kWaves, 1) void gemm_bf16_kernel(const bf16* A, const bf16* Wt,
                                                                   int64_t M, int N, int K,
                                                                   Epi e, int64_t tiles_main,
                                                                   int split) {
  if (e.pred && *e.pred == 0) return;
  // Three A tiles and two B tiles, one LDS object per tile so the compiler
  // can tell the tile being read from the tile being filled.
  __shared__ __attribute__((aligned(1024))) bf16 As0[kTileElems], Bs0[kTileElems];
  __shared__ __attribute__((aligned(1024))) bf16 As1[kTileElems], Bs1[kTileElems];
  __shared__ __attribute__((aligned(1024))) bf16 As2[kTileElems];

  const int tiles_n = (N + BN - 1) / BN;
  const int64_t tiles_m = (M + BM - 1) / BM;
  int64_t tm;
  int tn;
  int64_t item = -1;  // K-split work item, or -1 for a whole tile
  int kbeg = 0, klen = K;
  if ((int64_t)blockIdx.x < tiles_main) {
    tile_coords(xcd_remap(blockIdx.x, (uint32_t)tiles_main), tiles_m, tiles_n, tm, tn);
  } else {
    item = (int64_t)blockIdx.x - tiles_main;
    klen = K / split;
    kbeg = (int)(item % split) * klen;
    tile_coords((uint32_t)(tiles_main + item / split), tiles_m, tiles_n, tm, tn);
  }
  const int64_t m0 = tm * BM;
  const int n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int lr = lane & 31, lg = lane >> 5;
  // A tile of width 128 at the right edge (N % 256 == 128): waves with
  // wn >= 2 compute on clamped rows and store nothing.
  const bool active = n0 + wn * 64 < N;

  // Load-side addressing: byte offsets from the tile's first row (rows past
  // the edge are clamped; they only feed outputs that are never stored).
  // The K offset of a stage is added to the scalar base, so the per-lane
  // offsets stay fixed and a DMA needs no vector arithmetic.  Waves w and
  // w + 4 share a SIMD: wave w (< 4) issues the DMAs of both (DMA i < 4 its
  // own rows, i >= 4 those of wave w + 4), so wave w + 4 issues MFMAs only.
  const bool dma_wave = wave < 4;
  const int chunk_even = (lane & 7) ^ (lane >> 4);
  const int chunk_odd = (lane & 7) ^ ((lane >> 4) ^ 4);
  const uint64_t a_base = uniform_ptr(A + m0 * K + kbeg);
  const uint64_t b_base = uniform_ptr(Wt + (int64_t)n0 * K + kbeg);
  uint32_t a_off[8], b_off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int ww = (wave & 3) + (i >> 2) * 4;
    const int r = ww * 32 + (i & 3) * 8 + (lane >> 3);
    const int ra = m0 + r < M ? r : (int)(M - 1 - m0);
    const int rb = n0 + r < N ? r : N - 1 - n0;
    const int ch = (i & 1) ? chunk_odd : chunk_even;
    a_off[i] = (uint32_t)(ra * K + ch * 8) * 2u;
    b_off[i] = (uint32_t)(rb * K + ch * 8) * 2u;
  }
  auto tile_lds = [&](const bf16* tile) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)tile);
  };
  auto lds_slot = [&](int i) {
    return (uint32_t)((((wave & 3) + (i >> 2) * 4) * 4 + (i & 3)) * 1024);
  };

  // Read-side addressing: fragment row rr at K-step kk (16 wide) reads chunk
  // 2 kk + lg, stored at slot (2 kk + lg) ^ ((rr / 2) % 8), and
  // (rr / 2) % 8 == (lr / 2) % 8 for every fragment row of this lane.
  const int a_rbase = (wm * 128 + lr) * BK;
  const int b_rbase = (wn * 64 + lr) * BK;
  int sl[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) sl[kk] = 8 * ((2 * kk + lg) ^ ((lr >> 1) & 7));

  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  bf16x8 fa0[4], fb0[2], fa1[4], fb1[2];
  auto read_frags = [&](const bf16* As, const bf16* Bs, int slot, bf16x8(&fa)[4],
                        bf16x8(&fb)[2]) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
      fa[mb] = *reinterpret_cast<const bf16x8*>(As + a_rbase + mb * 32 * BK + slot);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
      fb[nb] = *reinterpret_cast<const bf16x8*>(Bs + b_rbase + nb * 32 * BK + slot);
  };
  auto mma = [&](const bf16x8(&fa)[4], const bf16x8(&fb)[2]) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[mb], fb[nb], acc[mb][nb], 0, 0, 0);
  };
  auto load_stage = [&](const bf16* As, const bf16* Bs, int k0) {
    const uint32_t la = tile_lds(As), lb = tile_lds(Bs);
#pragma unroll
    for (int i = 0; i < 8; ++i) dma16(a_base + (uint32_t)(k0 * 2), a_off[i], la + lds_slot(i));
#pragma unroll
    for (int i = 0; i < 8; ++i) dma16(b_base + (uint32_t)(k0 * 2), b_off[i], lb + lds_slot(i));
  };
  // One DMA after each of the 8 MFMAs of a K-step (order pinned by
  // scheduling barriers): the 8 DMAs that fill tile T at K offset k0.
  auto mma_dma = [&](const bf16x8(&fa)[4], const bf16x8(&fb)[2], const bf16* T,
                     uint64_t base, const uint32_t(&off)[8], int k0) {
    const uint32_t lt = tile_lds(T);
    const uint64_t bk = base + (uint32_t)(k0 * 2);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[mb], fb[nb], acc[mb][nb], 0, 0, 0);
        const int i = mb * 2 + nb;
        dma16(bk, off[i], lt + lds_slot(i));
        __builtin_amdgcn_sched_barrier(0);
      }
  };

  const int KT = klen / BK;  // even: K and each split's K range are multiples of 128
  auto kc = [&](int k) { return (k < KT ? k : KT - 1) * BK; };
  // Three A stages and two B stages (160 KB).  Stage kt refills A with
  // stage kt + 2 during its first K-step (the buffer stage kt - 1 read) and
  // B with stage kt + 2 during its last (the buffer it has just read), one
  // DMA per MFMA, so the activations, streamed from HBM, are requested about
  // 1.75 stages ahead of use and the weights 1.25.  Prologue: A 0, B 0, A 1,
  // B 1 (32 DMAs in a DMA wave); stage 0 landed (vmcnt 16; a wave without
  // DMAs has nothing outstanding).
  auto main_loop = [&](auto dma_flag) {
    constexpr bool kDma = decltype(dma_flag)::value;
    if constexpr (kDma) {
      load_stage(As0, Bs0, 0);
      load_stage(As1, Bs1, kc(1));
    }
    __builtin_amdgcn_s_waitcnt((16 & 15) | (7 << 4) | (15 << 8) | ((16 >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    read_frags(As0, Bs0, sl[0], fa0, fb0);

    // Stage kt reads A[kt % 3], B[kt % 2].  At its barrier the DMAs of this
    // stage's first K-step (A of stage kt + 2) may still be in flight, those
    // of stage kt + 1 (A in stage kt - 1, B in stage kt - 1's last K-step)
    // have landed: vmcnt(8).
    int kt = 0;
#define GEMM_STAGE(AS, BS, AN, BN_, AP)                                          \
  {                                                                            \
    read_frags(AS, BS, sl[1], fa1, fb1);                                       \
    __builtin_amdgcn_sched_barrier(0);                                         \
    if constexpr (kDma)                                                        \
      mma_dma(fa0, fb0, AP, a_base, a_off, kc(kt + 2));                        \
    else                                                                       \
      mma(fa0, fb0);                                                           \
    __builtin_amdgcn_sched_barrier(0);                                         \
    read_frags(AS, BS, sl[2], fa0, fb0);                                       \
    __builtin_amdgcn_sched_barrier(0);                                         \
    mma(fa1, fb1);                                                             \
    __builtin_amdgcn_sched_barrier(0);                                         \
    read_frags(AS, BS, sl[3], fa1, fb1);                                       \
    __builtin_amdgcn_sched_barrier(0);                                         \
    mma(fa0, fb0);                                                             \
    __builtin_amdgcn_sched_barrier(0);                                         \
    __builtin_amdgcn_s_waitcnt(8 | (7 << 4) | (0 << 8));                       \
    __builtin_amdgcn_s_barrier();                                              \
    read_frags(AN, BN_, sl[0], fa0, fb0);                                      \
    __builtin_amdgcn_sched_barrier(0);                                         \
    if constexpr (kDma)                                                        \
      mma_dma(fa1, fb1, BS, b_base, b_off, kc(kt + 2));                        \
    else                                                                       \
      mma(fa1, fb1);                                                           \
    __builtin_amdgcn_sched_barrier(0);                                         \
    ++kt;                                                                      \
  }
    while (kt + 6 <= KT) {
      GEMM_STAGE(As0, Bs0, As1, Bs1, As2)
      GEMM_STAGE(As1, Bs1, As2, Bs0, As0)
      GEMM_STAGE(As2, Bs0, As0, Bs1, As1)
      GEMM_STAGE(As0, Bs1, As1, Bs0, As2)
      GEMM_STAGE(As1, Bs0, As2, Bs1, As0)
      GEMM_STAGE(As2, Bs1, As0, Bs0, As1)
    }
    if (kt + 2 <= KT) {
      GEMM_STAGE(As0, Bs0, As1, Bs1, As2)
      GEMM_STAGE(As1, Bs1, As2, Bs0, As0)
    }
    if (kt + 2 <= KT) {
      GEMM_STAGE(As2, Bs0, As0, Bs1, As1)
      GEMM_STAGE(As0, Bs1, As1, Bs0, As2)
    }
#undef GEMM_STAGE
  };
  if (dma_wave)
    main_loop(std::true_type{});
  else
    main_loop(std::false_type{});
  wait_all();  // the last refill lands before the workgroup's LDS is released
  if (!active) return;
  if (item >= 0) {
    // Partial sums of this K range: value q of thread tid at (q * 512 + tid)
    // float4s into the item's 256 KB (consecutive threads, consecutive 16 B).
    f32x4* dst = reinterpret_cast<f32x4*>(e.split_ws) + item * (kSplitItemFloats / 4);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const int q = (mb * 2 + nb) * 4 + r4;
          dst[q * 64 * kWaves + tid] = f32x4{acc[mb][nb][4 * r4], acc[mb][nb][4 * r4 + 1],
                                             acc[mb][nb][4 * r4 + 2], acc[mb][nb][4 * r4 + 3]};
        }
    return;
  }
  tile_epilogue<KIND, bf16, 4, 2>(e, acc, M, N, m0 + wm * 128, n0 + wn * 64, m0 + BM <= M, lane);
}

// The split tiles: partial sums added in split order (deterministic), then
// the tile's epilogue.  Work item b reduces tile tiles_main + b.
template <int KIND>
__global__ __launch_bounds__(64 * kWaves, 1) void gemm_split_reduce_kernel(int64_t M, int N, Epi e,
                                                                           int64_t tiles_main,
                                                                           int split) {
  if (e.pred && *e.pred == 0) return;
  const int tiles_n = (N + BN - 1) / BN;
  const int64_t tiles_m = (M + BM - 1) / BM;
  int64_t tm;
  int tn;
  tile_coords((uint32_t)tiles_main + blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int64_t m0 = tm * BM;
  const int n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  if (!(n0 + wn * 64 < N)) return;
  const f32x4* src = reinterpret_cast<const f32x4*>(e.split_ws) +
                     (int64_t)blockIdx.x * split * (kSplitItemFloats / 4);
  f32x16 acc[4][2];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int q = (mb * 2 + nb) * 4 + r4;
        f32x4 v = src[q * 64 * kWaves + tid];
        for (int sp = 1; sp < split; ++sp)
          v += src[sp * (kSplitItemFloats / 4) + q * 64 * kWaves + tid];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[mb][nb][4 * r4 + i] = v[i];
      }
  tile_epilogue<KIND, bf16, 4, 2>(e, acc, M, N, m0 + wm * 128, n0 + wn * 64, m0 + BM <= M, lane);
}

// ------------------------------------------------- MFMA, few tiles

// A DMA wave (w of four) of the ring kernels.  A stage holds SUB K-steps of
// 128 bytes of the TM x TN tile's operands; DMA i of wave w fills its 1 KB
// block b = w ND + i: 8 rows of the A tile (the first TM / 8 blocks of a
// K-step) or of the B tile, 128 bytes each, chunks at the slots of the
// 256 x 256 kernel's tiles.  Rows past M are clamped.  Stage st goes into
// buffer st % NST once the MFMA waves have read stage st - NST; barrier st
// (after the one that admits stage 0) admits stage st + 1.  NS stages from
// k0 on.
template <typename T, int TM, int TN, int SUB, int NST>
__device__ __forceinline__ void ring_feed(const T* A, const T* Wt, int64_t M, int K, int64_t m0,
                                          int n0, int k0, int NS, int w, int lane,
                                          const T* ring) {
  constexpr int kBlk = (TM + TN) / 8;           // 1 KB blocks per K-step
  constexpr int ND = SUB * kBlk / 4;            // DMAs per wave and stage
  static_assert(SUB * kBlk % 4 == 0 && NST >= 2 && ND * (NST - 1) <= 63, "ring");
  uint64_t base[ND];
  uint32_t off[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int b = w * ND + i;
    const int sub = b / kBlk, bb = b % kBlk;
    const bool is_a = bb < TM / 8;
    const int r = (is_a ? bb : bb - TM / 8) * 8 + (lane >> 3);
    const int ch = (lane & 7) ^ ((r >> 1) & 7);
    const int row = is_a && m0 + r >= M ? (int)(M - 1 - m0) : r;
    base[i] = uniform_ptr((is_a ? A + m0 * K : Wt + (int64_t)n0 * K) + k0);
    off[i] = (uint32_t)row * (uint32_t)(K * (int)sizeof(T)) + (uint32_t)(sub * 128 + ch * 16);
  }
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t*)ring) +
                        (uint32_t)(w * ND) * 1024u;
  // fp32 operands may lie at any multiple of 4 bytes (plain loads read them
  // so): those are copied through registers, complete when issue returns.
  const bool copy = sizeof(T) == 4 && (((uintptr_t)A | (uintptr_t)Wt) & 15) != 0;
  auto issue = [&](int st, uint32_t buf) {
    const uint32_t kb = (uint32_t)st * (SUB * 128);
    if (copy) {
      u32x4 v[ND];
#pragma unroll
      for (int i = 0; i < ND; ++i)
        __builtin_memcpy(&v[i], reinterpret_cast<const char*>(base[i] + kb) + off[i], 16);
      u32x4* dst = reinterpret_cast<u32x4*>(const_cast<T*>(ring)) +
                   (buf * (uint32_t)(SUB * kBlk) + (uint32_t)(w * ND)) * 64u + lane;
#pragma unroll
      for (int i = 0; i < ND; ++i) dst[i * 64] = v[i];
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0);
      return;
    }
#pragma unroll
    for (int i = 0; i < ND; ++i)
      dma16(base[i] + kb, off[i], lds0 + buf * (uint32_t)(SUB * kBlk * 1024) + i * 1024u);
  };
  // vmcnt(n), no other counter
#define RING_WAIT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))
#pragma unroll
  for (int st = 0; st < NST; ++st)
    if (st < NS) issue(st, st);
  if (NS >= NST)
    RING_WAIT(ND * (NST - 1));  // stage 0 landed
  else
    RING_WAIT(0);
  __builtin_amdgcn_s_barrier();
  uint32_t buf = 0;
  for (int st = 0; st < NS; ++st) {
    // stage st + 1 landed: NST - 2 younger stages may be in flight
    if (st + NST - 1 < NS)
      RING_WAIT(ND * (NST - 2));
    else
      RING_WAIT(0);
    __builtin_amdgcn_s_barrier();  // stage st read by all: its buffer is free
    if (st + NST < NS) issue(st + NST, buf);
    buf = buf + 1 == NST ? 0 : buf + 1;
  }
#undef RING_WAIT
}

// The bf16 product for grids that the 256 x 256 tiles leave mostly idle
// (short sequences, few rows): TM x TN tiles, WM x WN waves that only read
// fragments and issue MFMAs, and four waves that only issue the operand
// DMAs, one on each SIMD beside them.  A K-step of 64 of both operands is
// one stage of a ring of NST stages, each refilled NST - 1 stages ahead; one
// barrier per stage, before the last sub-step of 16, so the next stage's
// first fragment reads run under its MFMAs.  A tile accumulates its K-steps
// in the order of the 256 x 256 kernel with the same instruction, so results
// do not depend on the tile size, bit for bit.
// SPLIT: the K-steps of each tile are split into `split` ranges, one work item
// each, which leave fp32 partial sums in e.split_ws for
// gemm_ring_reduce_kernel.
// A 128 x 128 stage takes about 0.41 us of a CU with 156 tiles in flight
// (0.36 without the DMAs, 0.31 for one tile per XCD alone; its MFMAs need
// 0.22 us at 2.4 GHz): the MFMA waves' issue between barriers bounds it, not
// the staging.  Reading fragments three sub-steps ahead instead of one, or a
// ring one stage deeper, changes nothing (57-60 us at 1560 x 1536 x 8960);
// eight MFMA waves instead of four 2-10% faster.
template <int KIND, int TM, int TN, int WM, int WN, int NST, int OCC, bool SPLIT>
__global__ __launch_bounds__(64 * (WM * WN + 4), OCC) void gemm_ring_kernel(
    const bf16* A, const bf16* Wt, int64_t M, int N, int K, Epi e, int split) {
  if (e.pred && *e.pred == 0) return;
  constexpr int kMath = WM * WN;                       // MFMA waves
  constexpr int MB = TM / WM / 32, NB = TN / WN / 32;  // 32 x 32 blocks per wave
  constexpr int kStageElems = (TM + TN) * BK;
  __shared__ __attribute__((aligned(1024))) bf16 ring[NST * kStageElems];

  const int tiles_n = N / TN;
  const int64_t tiles_m = (M + TM - 1) / TM;
  int64_t tm;
  int tn;
  const uint32_t tiles = (uint32_t)tiles_m * tiles_n, items = SPLIT ? tiles * split : tiles;
  const uint32_t bid = blockIdx.y * gridDim.x + blockIdx.x;
  if (bid >= items) return;
  uint32_t t = xcd_remap(bid, items);
  const int part = SPLIT ? (int)(t / tiles) : 0;  // ranges outer: an XCD's tiles share operands
  if constexpr (SPLIT) t -= part * tiles;
  tile_coords<4>(t, tiles_m, tiles_n, tm, tn);
  const int64_t m0 = tm * TM;
  const int n0 = tn * TN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int steps = K / BK, s0 = SPLIT ? steps * part / split : 0;
  const int NS = SPLIT ? steps * (part + 1) / split - s0 : steps;

  if (wave >= kMath) {
    ring_feed<bf16, TM, TN, 1, NST>(A, Wt, M, K, m0, n0, s0 * BK, NS, wave - kMath, lane, ring);
    return;
  }

  const int wm = wave / WN, wn = wave % WN;
  const int lr = lane & 31, lg = lane >> 5;
  const int a_rbase = (wm * (TM / WM) + lr) * BK;
  const int b_rbase = (TM + wn * (TN / WN) + lr) * BK;
  int sl[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) sl[kk] = 8 * ((2 * kk + lg) ^ ((lr >> 1) & 7));
  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  bf16x8 fa[2][MB], fb[2][NB];
  auto read_frags = [&](const bf16* stage, int kk) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      fa[kk & 1][mb] = *reinterpret_cast<const bf16x8*>(stage + a_rbase + mb * 32 * BK + sl[kk]);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      fb[kk & 1][nb] = *reinterpret_cast<const bf16x8*>(stage + b_rbase + nb * 32 * BK + sl[kk]);
  };
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_frags(ring, 0);
  int buf = 0;
  for (int st = 0; st < NS; ++st) {
    const bf16* cur = ring + buf * kStageElems;
    buf = buf + 1 == NST ? 0 : buf + 1;
    const bf16* nxt = ring + buf * kStageElems;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      if (kk < 3) {
        read_frags(cur, kk + 1);
      } else {
        // the stage's last fragments have arrived: its buffer may be refilled
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_frags(nxt, 0);  // after the last stage: read and dropped
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1][mb], fb[kk & 1][nb],
                                                                acc[mb][nb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (SPLIT) {
    // Partial sums of this K range: value q of thread tid at (q kMath 64 + tid)
    // float4s into the work item (consecutive threads, consecutive 16 B).
    const int64_t item = ((int64_t)tm * tiles_n + tn) * split + part;
    f32x4* dst = reinterpret_cast<f32x4*>(e.split_ws) + item * (TM * TN / 4);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          dst[((mb * NB + nb) * 4 + r4) * 64 * kMath + tid] =
              f32x4{acc[mb][nb][4 * r4], acc[mb][nb][4 * r4 + 1], acc[mb][nb][4 * r4 + 2],
                    acc[mb][nb][4 * r4 + 3]};
    return;
  }
  tile_epilogue<KIND, bf16, MB, NB, OCC >= 3 ? 16 : 32>(e, acc, M, N, m0 + wm * (TM / WM),
                                                       n0 + wn * (TN / WN), m0 + TM <= M, lane);
}

// Second pass of a ring launch with a K split: each wave adds the partial
// sums of one 32 x 32 block of a tile in range order (deterministic) and runs
// the tile's epilogue.  Bound by the latency of its loads: one block a wave
// and four ranges' loads in flight, the old values of a read-modify-write
// requested first.
template <int KIND, int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(256) void gemm_ring_reduce_kernel(int64_t M, int N, Epi e,
                                                               int split) {
  if (e.pred && *e.pred == 0) return;
  constexpr int MB = TM / WM / 32, NB = TN / WN / 32, kBlocks = TM / 32 * (TN / 32);
  static_assert(kBlocks % 4 == 0, "whole workgroups per tile");
  const int lane = threadIdx.x & 63;
  const uint32_t tile = blockIdx.x / (kBlocks / 4);
  // Four neighbouring column blocks per workgroup where the tile has them.
  const int b = (int)(blockIdx.x % (kBlocks / 4)) * 4 +
                __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb = b / (TN / 32), cb = b % (TN / 32);
  const uint32_t tiles_n = N / TN;
  const int64_t m = (int64_t)(tile / tiles_n) * TM + rb * 32;
  const int n = (int)(tile % tiles_n) * TN + cb * 32;
  if (m >= M) return;
  const int wave = rb / MB * WN + cb / NB;
  const int q = (rb % MB * NB + cb % NB) * 4;
  constexpr int64_t kQ = 64 * WM * WN, kPart = TM * TN / 4;
  const f32x4* src = reinterpret_cast<const f32x4*>(e.split_ws) + (int64_t)tile * split * kPart + q * kQ +
                     wave * 64 + lane;
  const int lr = lane & 31, lg = lane >> 5;
  const ColEpi<KIND, bf16> ce(e, n + lr, N);
  const int64_t mrow = m + 4 * lg;
  float prev[16];
  if constexpr (ColEpi<KIND, bf16>::kRmw) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t row = mrow + 8 * (r >> 2) + (r & 3);
      prev[r] = ce.old(row < M ? row : M - 1);
    }
  }
  f32x4 v[4];
#pragma unroll
  for (int r4 = 0; r4 < 4; ++r4) v[r4] = src[r4 * kQ];
  // Four ranges in flight at a time; past the last: read again and dropped.
  for (int s = 1; s < split; s += 4) {
    f32x4 w[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) w[j][r4] = src[min(s + j, split - 1) * kPart + r4 * kQ];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (s + j < split)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) v[r4] += w[j][r4];
  }
  if constexpr (ColEpi<KIND, bf16>::kRmw) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t row = mrow + 8 * (r >> 2) + (r & 3);
      if (row < M) ce.put_old(row, v[r / 4][r % 4], prev[r]);
    }
  } else {
    f32x16 acc[1][1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = v[r / 4][r % 4];
    tile_epilogue<KIND, bf16, 1, 1>(e, acc, M, N, m, n, m + 32 <= M, lane);
  }
}

// ------------------------------------------------------------ fp32 MFMA

// fp32: v_mfma_f32_32x32x2_f32 (products and sums in fp32) on the same ring.
// A lane's 16-byte fragment of row r holds k = 8 kk + 4 (lane / 32) + 0..3,
// so MFMA i of a sub-step contracts k = 8 kk + i and 8 kk + 4 + i.  The
// sub-steps kk = 0..3 of the 32-wide K-steps sum into accumulators of their
// own, added as ((0 + 1) + (2 + 3)) at the end: with WK = 1 a wave holds all
// four, with WK = 4 each of four waves holds one and they meet in LDS, so
// both tiles give the same bits.  Bound by the matrix unit (157 TFLOP/s; an
// MFMA of 64 cycles per two fragment registers); one wave of the 32 x 32
// tile has a quarter of the 64 x 64 tile's serial MFMA chain, which is what a
// launch of few tiles takes.  Against the 64 x 64 VALU kernel before it: a
// 1013-token fp32 block (H 1024, F 4096) 609 -> 286 us, the 128-token loop
// (H 256) 890 -> 553 us.
template <int KIND, int TM, int TN, int WM, int WN, int WK, int SUB, int NST, int OCC>
__global__ __launch_bounds__(512, OCC) void gemm_f32_kernel(const float* A, const float* Wt,
                                                            int64_t M, int N, int K, Epi e) {
  if (e.pred && *e.pred == 0) return;
  constexpr int kRow = 32;           // floats per row and K-step
  constexpr int NCL = 4 / WK;        // sub-step classes a wave sums
  constexpr int NSTEP = SUB * NCL;   // sub-steps of a wave per stage
  constexpr int kStageElems = SUB * (TM + TN) * kRow;
  static_assert(WM * WN * WK == 4 && TM == 32 * WM && TN == 32 * WN && NSTEP >= 2, "waves");
  __shared__ __attribute__((aligned(1024))) float ring[NST * kStageElems];

  const int tiles_n = N / TN;
  const int64_t tiles_m = (M + TM - 1) / TM;
  int64_t tm;
  int tn;
  const uint32_t tiles = (uint32_t)tiles_m * tiles_n;
  const uint32_t bid = blockIdx.y * gridDim.x + blockIdx.x;
  if (bid >= tiles) return;
  tile_coords<4>(xcd_remap(bid, tiles), tiles_m, tiles_n, tm, tn);
  const int64_t m0 = tm * TM;
  const int n0 = tn * TN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NS = K / (SUB * kRow);
  if (wave >= 4) {
    ring_feed<float, TM, TN, SUB, NST>(A, Wt, M, K, m0, n0, 0, NS, wave - 4, lane, ring);
    return;
  }

  const int wk = wave % WK, wm = wave / WK / WN, wn = wave / WK % WN;
  const int lr = lane & 31, lg = lane >> 5;
  const int a_rbase = (wm * 32 + lr) * kRow;
  const int b_rbase = (TM + wn * 32 + lr) * kRow;
  f32x16 part[NCL];
#pragma unroll
  for (int c = 0; c < NCL; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[c][r] = 0.f;
  f32x4 fa[2], fb[2];
  auto read_frags = [&](const float* stage, int i) {
    const int kk = i % NCL * WK + wk;
    const float* t = stage + (i / NCL) * (TM + TN) * kRow + 4 * ((2 * kk + lg) ^ ((lr >> 1) & 7));
    fa[i & 1] = *reinterpret_cast<const f32x4*>(t + a_rbase);
    fb[i & 1] = *reinterpret_cast<const f32x4*>(t + b_rbase);
  };
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_frags(ring, 0);
  int buf = 0;
  for (int st = 0; st < NS; ++st) {
    const float* cur = ring + buf * kStageElems;
    buf = buf + 1 == NST ? 0 : buf + 1;
    const float* nxt = ring + buf * kStageElems;
#pragma unroll
    for (int i = 0; i < NSTEP; ++i) {
      if (i + 1 < NSTEP) {
        read_frags(cur, i + 1);
      } else {
        // the stage's last fragments have arrived: its buffer may be refilled
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        read_frags(nxt, 0);  // after the last stage: read and dropped
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        part[i % NCL] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i & 1][j], fb[i & 1][j],
                                                             part[i % NCL], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if constexpr (WK == 1) {
    f32x16 acc[1][1];
    acc[0][0] = (part[0] + part[1]) + (part[2] + part[3]);
    tile_epilogue<KIND, float, 1, 1>(e, acc, M, N, m0 + wm * 32, n0 + wn * 32, m0 + TM <= M, lane);
  } else {
    static_assert(WK == 4 && 4 * 16 * 64 <= NST * kStageElems, "partial sums fit the ring");
    // Every DMA has landed and every wave has its last fragments.
#pragma unroll
    for (int r = 0; r < 16; ++r) ring[(wk * 16 + r) * 64 + lane] = part[0][r];
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
    __builtin_amdgcn_s_barrier();  // the four MFMA waves: the DMA waves have ended
    asm volatile("" ::: "memory");
    // wave wk finishes accumulator entries 4 wk .. 4 wk + 3: four rows a lane
    const ColEpi<KIND, float> ce(e, n0 + lr, N);
    const int64_t m = m0 + 8 * wk + 4 * lg;
    float y[4], prev[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* p = ring + (4 * wk + r) * 64 + lane;
      y[r] = (p[0] + p[16 * 64]) + (p[32 * 64] + p[48 * 64]);
      prev[r] = ce.old(m + r < M ? m + r : M - 1);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (m + r < M) ce.put_old(m + r, y[r], prev[r]);
  }
}

// Grid of a ring kernel: one workgroup per tile, in two dimensions beyond 2^22
// (a dimension holds fewer than 2^32 work-items).
dim3 ring_grid(int64_t tiles) {
  const int64_t gy = (tiles + (1 << 22) - 1) >> 22;
  return dim3((unsigned)((tiles + gy - 1) / gy), (unsigned)gy);
}

template <int KIND, int TM, int TN, int WM, int WN, int NST, int OCC>
hipError_t launch_ring(int64_t M, int N, int K, const void* a, const void* wt, const Epi& e,
                       hipStream_t s, int split) {
  const int64_t tiles = (M + TM - 1) / TM * (N / TN), grid = tiles * split;
  if (split == 1) {
    hipLaunchKernelGGL((gemm_ring_kernel<KIND, TM, TN, WM, WN, NST, OCC, false>), ring_grid(grid),
                       dim3(64 * (WM * WN + 4)), 0, s, (const bf16*)a, (const bf16*)wt, M, N, K, e,
                       1);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((gemm_ring_kernel<KIND, TM, TN, WM, WN, NST, OCC, true>), ring_grid(grid),
                     dim3(64 * (WM * WN + 4)), 0, s, (const bf16*)a, (const bf16*)wt, M, N, K, e,
                     split);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  hipLaunchKernelGGL((gemm_ring_reduce_kernel<KIND, TM, TN, WM, WN>),
                     dim3((unsigned)(tiles * (TM / 32 * (TN / 32) / 4))), dim3(256), 0, s, M, N, e,
                     split);
  return hipGetLastError();
}

template <int KIND>
hipError_t launch_kind(int dtype, int64_t M, int N, int K, const void* a, const void* wt,
                       const Epi& e, hipStream_t s) {
  if (dtype == ACID_BF16) {
    const int64_t tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    constexpr Out kOut = KIND == ACID_EPI_BIAS        ? Out::kPlain
                         : KIND == ACID_EPI_BIAS_GELU ? Out::kGelu
                         : ColEpi<KIND, bf16>::kRmw   ? Out::kUpdate
                                                      : Out::kHeads;
    const Form f = choose_form(kOut, M, N, K, e.split_ws != nullptr, device_cus());
    const int split = f.split;
    const int64_t rem = f.rem;
    switch (f.tile) {
      case Tile::k256x128: return launch_ring<KIND, 256, 128, 4, 2, 3, 3>(M, N, K, a, wt, e, s, split);
      case Tile::k128: return launch_ring<KIND, 128, 128, 2, 4, 4, 3>(M, N, K, a, wt, e, s, split);
      case Tile::k64: return launch_ring<KIND, 64, 64, 2, 2, 4, 4>(M, N, K, a, wt, e, s, split);
      case Tile::k256: break;
    }
    const int64_t tiles_main = tiles - (split > 1 ? rem : 0);
    const int64_t grid = tiles_main + (split > 1 ? rem * split : 0);
    hipLaunchKernelGGL(gemm_bf16_kernel<KIND>, dim3((unsigned)grid), dim3(64 * kWaves), 0, s,
                       (const bf16*)a, (const bf16*)wt, M, N, K, e, tiles_main, split);
    if (split > 1) {
      const hipError_t err = hipGetLastError();
      if (err != hipSuccess) return err;
      hipLaunchKernelGGL(gemm_split_reduce_kernel<KIND>, dim3((unsigned)rem), dim3(64 * kWaves),
                         0, s, M, N, e, tiles_main, split);
    }
  } else {
    // 64 x 64 tiles, or 32 x 32 ones where those leave most CUs idle: a round
    // of 32 x 32 tiles takes a quarter of the time, and about a fifth more
    // for its shorter K ranges per wave and its reduction.
    const int64_t cus = device_cus();
    const int64_t t64 = (M + 63) / 64 * (N / 64), t32 = (M + 31) / 32 * (N / 32);
    if ((double)((t32 + cus - 1) / cus) * 0.3 < (double)((t64 + cus - 1) / cus))
      hipLaunchKernelGGL((gemm_f32_kernel<KIND, 32, 32, 1, 1, 4, 2, 4, 4>), ring_grid(t32),
                         dim3(512), 0, s, (const float*)a, (const float*)wt, M, N, K, e);
    else
      hipLaunchKernelGGL((gemm_f32_kernel<KIND, 64, 64, 2, 2, 1, 1, 4, 4>), ring_grid(t64),
                         dim3(512), 0, s, (const float*)a, (const float*)wt, M, N, K, e);
  }
  return hipGetLastError();
}

}  // namespace

// The device's CUs (256 where it cannot be asked).
int device_cus() {
  static std::atomic<int> cus{0};
  int c = cus.load(std::memory_order_relaxed);
  if (c == 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        c < 1)
      c = 256;
    cus.store(c, std::memory_order_relaxed);
  }
  return c;
}

hipError_t launch_linear(int dtype, int64_t M, int N, int K, const void* a, const void* wt,
                         const acid_epilogue_args& ea, hipStream_t s, const int32_t* pred,
                         float* split_ws) {
  if (M == 0) return hipSuccess;
  Epi e;
  e.split_ws = dtype == ACID_BF16 ? split_ws : nullptr;
  e.bias = ea.bias;
  e.gate = ea.gate;
  e.out = ea.out;
  e.v_out = ea.v_out;
  e.q = ea.q;
  e.k = ea.k;
  e.vt = ea.vt;
  e.vt_ld = ea.vt_ld;
  e.M = M;
  e.n_heads = ea.n_heads;
  e.head_dim = ea.head_dim;
  e.H = ea.n_heads * ea.head_dim;
  e.dsigma = ea.dsigma;
  e.pred = pred;
  e.bias2 = ea.bias2;
  e.out_ld = ea.out_ld;
  e.n_qkv = 3 * ea.n_heads * ea.head_dim;
  e.q_mul = ea.q_prescale ? attn_q_scale(ea.head_dim) : 1.f;
  switch (ea.kind) {
    case ACID_EPI_BIAS: return launch_kind<ACID_EPI_BIAS>(dtype, M, N, K, a, wt, e, s);
    case ACID_EPI_BIAS_GELU: return launch_kind<ACID_EPI_BIAS_GELU>(dtype, M, N, K, a, wt, e, s);
    case ACID_EPI_GATE_RESIDUAL:
      return launch_kind<ACID_EPI_GATE_RESIDUAL>(dtype, M, N, K, a, wt, e, s);
    case ACID_EPI_QKV: return launch_kind<ACID_EPI_QKV>(dtype, M, N, K, a, wt, e, s);
    case ACID_EPI_EULER: return launch_kind<ACID_EPI_EULER>(dtype, M, N, K, a, wt, e, s);
    case ACID_EPI_QKV_GELU: return launch_kind<ACID_EPI_QKV_GELU>(dtype, M, N, K, a, wt, e, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace acid
