// Timestep conditioning: sinusoidal embedding of t = 1000 sigma and the small
// fp32 matrix products that turn it into the adaLN modulation table.
//
// This runs once per denoise loop for all noise levels at once, so the
// products have few rows (the step count) and are bound by reading the
// fp32 adaLN weights (1.7 GB at the Wan-1.3B shape) once.
#include "common.h"

namespace acid {

namespace {

constexpr int kMaxSig = 128;
struct SigmaPack {
  float v[kMaxSig];
};

__global__ void sinusoid_kernel(SigmaPack sig, int n, int freq_dim, float* __restrict__ e) {
  const int i = blockIdx.x;
  if (i >= n) return;
  const int half = freq_dim / 2;
  const double t = 1000.0 * (double)sig.v[i];
  const double lnp = 9.210340371976184;  // ln(10000)
  for (int j = threadIdx.x; j < half; j += blockDim.x) {
    double f = exp(-lnp * (double)j / (double)half);
    double a = t * f;
    e[(int64_t)i * freq_dim + j] = (float)cos(a);
    e[(int64_t)i * freq_dim + half + j] = (float)sin(a);
  }
}

// Y[s][n] = act(sum_k X[s][k] W[k][n] + b[n]) for 32 RB rows s and 32 CB
// columns n per workgroup, on the fp32 matrix instruction
// (v_mfma_f32_32x32x2_f32).  Bound by reading W once (1.7 GB at the Wan-1.3B
// shape).  The NW waves split K in groups of 8 (wave w takes groups w,
// w + NW, ...): lane (half-wave h, index l) loads X[l][8 g + 4 h ..+3] and
// W[8 g + 4 h + i][n0 + CB l ..+CB-1], so MFMA i of a group contracts
// k = 8 g + i and 8 g + 4 + i, and one load of W is the operand of CB column
// blocks.  Two, three or eight groups are kept in flight per wave.  The waves'
// partial sums meet in LDS and are added in wave order (deterministic, and
// independent of RB and CB: a row's values depend neither on how many rows the
// call holds nor on how many columns a workgroup has).
// 50 rows x 30 x (1536 x 9216): the 16-rows-at-a-time VALU kernel took 1277
// us, this one 545 (MFMAs on rows padded to 64: 346; one row: 316 us, 5.4
// TB/s); the table with its three small products 1793 -> 594 us.  Two column
// blocks per workgroup ran 18% slower, an eight-way split 14%.
template <int RB, int CB, int NW>
__global__ __launch_bounds__(64 * NW, CB == 4 ? 2 : 4) void skinny_gemm_kernel(
    const float* __restrict__ X, int ldx, int S, int K, const float* __restrict__ W, int ldw,
    const float* __restrict__ bias, float* __restrict__ Y, int64_t ldy, int act_out,
    int64_t w_stride, int64_t b_stride, int64_t y_stride) {
  typedef float wvec __attribute__((ext_vector_type(CB)));
  constexpr int D = CB == 4 ? 2 : NW == 16 ? 3 : 8;  // groups in flight
  __shared__ wvec lds[NW * 16 * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lg = lane >> 5;
  const int n0 = blockIdx.x * 32 * CB, g = blockIdx.y, s0 = blockIdx.z * 32 * RB;
  const float* wp = W + g * w_stride + (int64_t)(4 * lg) * ldw + n0 + CB * lr;
  const float* xp[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {  // rows past S repeat the last and are not stored
    const int row = s0 + 32 * rb + lr;
    xp[rb] = X + (int64_t)(row < S ? row : S - 1) * ldx + 4 * lg;
  }
  struct Frag {
    f32x4 x[RB];
    wvec w[4];
  };
  f32x16 acc[RB][CB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[rb][cb][r] = 0.f;
  auto load = [&](Frag& f, int grp) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      f.w[i] = *reinterpret_cast<const wvec*>(wp + (int64_t)(8 * grp + i) * ldw);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) f.x[rb] = *reinterpret_cast<const f32x4*>(xp[rb] + 8 * grp);
  };
  auto mma = [&](const Frag& f) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.x[rb][i], f.w[i][cb], acc[rb][cb],
                                                             0, 0, 0);
  };
  const int full = K / 8;
  const int cnt = wave < full ? (full - 1 - wave) / NW + 1 : 0;  // this wave's whole groups
  if (cnt > 0) {
    Frag f[D];
    auto grp = [&](int j) { return wave + min(j, cnt - 1) * NW; };  // past the last: read again
#pragma unroll
    for (int d = 0; d < D; ++d) load(f[d], grp(d));
    int j = 0;
    // No branch between a group's MFMAs and its refill: with one, the
    // compiler waits for every load in flight at the loop's top.
    for (; j + D <= cnt; j += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        mma(f[d]);
        __builtin_amdgcn_sched_barrier(0);
        load(f[d], grp(j + d + D));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (j + d < cnt) mma(f[d]);
  }
  if (K % 8 != 0 && wave == full % NW) {  // the ragged last group, element by element
    Frag f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = 8 * full + 4 * lg + i < K;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        f.w[i][cb] = in ? wp[(int64_t)(8 * full + i) * ldw + cb] : 0.f;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) f.x[rb][i] = in ? xp[rb][8 * full + i] : 0.f;
    }
    mma(f);
  }
  const wvec bv = *reinterpret_cast<const wvec*>(bias + g * b_stride + n0 + CB * lr);
  float* Yg = Y + g * y_stride + n0 + CB * lr;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    if (rb) __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      wvec v;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) v[cb] = acc[rb][cb][r];
      lds[(wave * 16 + r) * 64 + lane] = v;
    }
    __syncthreads();
#pragma unroll
    for (int r = wave; r < 16; r += NW) {  // accumulator entry r: row 8 (r / 4) + 4 h + r % 4
      wvec y = lds[r * 64 + lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) y += lds[(w * 16 + r) * 64 + lane];
      y += bv;
      if (act_out == 1) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) y[cb] = silu(y[cb]);
      }
      const int row = s0 + 32 * rb + 8 * (r >> 2) + 4 * lg + (r & 3);
      if (row < S) *reinterpret_cast<wvec*>(Yg + (int64_t)row * ldy) = y;
    }
  }
}

}  // namespace

hipError_t launch_sinusoid(const float* sigmas_host, int n, int freq_dim, float* e,
                           hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += kMaxSig) {
    SigmaPack p;
    int cnt = n - i0 < kMaxSig ? n - i0 : kMaxSig;
    for (int i = 0; i < cnt; ++i) p.v[i] = sigmas_host[i0 + i];
    hipLaunchKernelGGL(sinusoid_kernel, dim3(cnt), dim3(128), 0, s, p, cnt, freq_dim,
                       e + (int64_t)i0 * freq_dim);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

hipError_t launch_skinny_gemm(const float* X, int ldx, int S, int K, const float* W, int ldw,
                              int N, const float* b, float* Y, int64_t ldy, int act_out,
                              int batch, int64_t w_stride, int64_t b_stride, int64_t y_stride,
                              hipStream_t s, int64_t of_columns) {
  if (S == 0 || batch == 0) return hipSuccess;
  if (N % 128 != 0 || ((uintptr_t)W % 16) != 0 || (w_stride % 4) != 0 || (ldw % 4) != 0 ||
      ((uintptr_t)b % 16) != 0 || (b_stride % 4) != 0)
    return hipErrorInvalidValue;  // 16-byte loads of W and b (Y may lie at any float)
#define SKINNY(RB, CB, NW)                                                                      \
  hipLaunchKernelGGL((skinny_gemm_kernel<RB, CB, NW>),                                          \
                     dim3((unsigned)(N / (32 * CB)), (unsigned)batch,                           \
                          (unsigned)((S + 32 * RB - 1) / (32 * RB))),                           \
                     dim3(64 * NW), 0, s, X, ldx, S, K, W, ldw, b, Y, ldy, act_out, w_stride,   \
                     b_stride, y_stride)
  // 128 columns and a four-way K split per workgroup where that gives the
  // CUs a workgroup each (then 64 rows share a read of W); otherwise 32
  // columns, 32 rows and a sixteen-way split: a 1536 x 1536 product of 50
  // rows is 12 workgroups of the one and 96 of the other.  The split does
  // not look at S, so that a row's sums do not either, and where a call forms
  // some columns of a larger product (of_columns) it is that product's, so that
  // both give the same bits: 32 columns, four waves (the pair of a drift
  // signal at the Wan-1.3B shape, 1536 x 3072 of 1536 x 276480).
  const int64_t own = (int64_t)N * batch, of = of_columns > own ? of_columns : own;
  if (of / 128 < device_cus())
    SKINNY(1, 1, 16);
  else if (own / 128 < device_cus())
    SKINNY(1, 1, 4);
  else if (S <= 32)
    SKINNY(1, 4, 4);
  else
    SKINNY(2, 4, 4);
#undef SKINNY
  return hipGetLastError();
}

}  // namespace acid
