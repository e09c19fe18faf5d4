// GEMMs of the step.
//
//  * gemm_bf16: C = A . W^T on gfx950 MFMA (v_mfma_f32_32x32x16_bf16), bf16
//    operands, fp32 accumulation, LDS double buffering, fused epilogues
//    (bias, exact GELU, fp32 residual add, conv-stem row mapping, scatter of
//    all decoder layers' cross K/V into a slot's cache).
//  * gemm_f32: the same contract on fp32 MFMA (the fp32 model path).
//  * vocab_argmax_bf16: the tied vocabulary projection fused with a per-row
//    argmax (lowest index on ties) over each 32-row tile of the table, finished by a
//    deterministic cross-tile reduction.
#include "asr_device.h"

#include <algorithm>

namespace asr {

// ---------------------------------------------------------------------------
// Epilogue
// ---------------------------------------------------------------------------
template <int KIND, typename T>
__device__ __forceinline__ void epi_apply(const Epilogue& e, int r, int n, float acc) {
  float v = acc + (e.bias ? e.bias[n] : 0.0f);
  if constexpr (KIND == EPI_STORE) {
    St<T>::st((T*)e.out, (int64_t)r * e.ldc + n, v);
  } else if constexpr (KIND == EPI_GELU) {
    St<T>::st((T*)e.out, (int64_t)r * e.ldc + n, gelu_erf(v));
  } else if constexpr (KIND == EPI_CONV1) {
    int g = r / kFrames, t = r - g * kFrames;
    int64_t base = (int64_t)g * (kFrames + 1) * e.d_model;
    St<T>::st((T*)e.out, base + (int64_t)(t + 1) * e.d_model + n, gelu_erf(v));
    if (t == 0) St<T>::st((T*)e.out, base + n, 0.0f);        // position -1 of conv2
  } else if constexpr (KIND == EPI_CONV2) {
    int t = r % kCtx;
    ((float*)e.out)[(int64_t)r * e.ldc + n] = gelu_erf(v) + e.pos[(int64_t)t * e.ldc + n];
  } else if constexpr (KIND == EPI_XKV) {
    int g = r / kCtx, t = r - g * kCtx;
    int two_d = 2 * e.d_model;
    int l = n / two_d;
    int rem = n - l * two_d;
    int kv = rem >= e.d_model;
    int hd = rem - kv * e.d_model;
    int h = hd >> 6, c = hd & 63;
    int64_t addr = (int64_t)e.slots[g] * e.slot_stride +
                   ((((int64_t)l * 2 + kv) * e.n_head + h) * kCtx + t) * kHeadDim + c;
    St<T>::st((T*)e.out, addr, v);
  } else if constexpr (KIND == EPI_QKV) {
    const int two_d = 2 * e.d_model;
    if (n < two_d) {
      St<T>::st((T*)e.out, (int64_t)r * e.ldc + n, n < e.d_model ? v * kQScaleLog2 : v);
    } else {
      int g = r / kCtx, t = r - g * kCtx;
      int hd = n - two_d;
      int64_t addr = (((int64_t)g * e.n_head + (hd >> 6)) * kHeadDim + (hd & 63)) * kVtLd + t;
      St<T>::st((T*)e.out2, addr, v);
    }
  }
}

// Epilogue stores carry the non-temporal hint: the encoder products write
// hundreds of MB that the L2 cannot keep for the next kernel anyway, and
// letting them allocate there evicts the operand panels the running GEMM
// still re-reads (measured: about a quarter of the time of a K = 1280
// product goes away).
__device__ __forceinline__ void st4_bf16(bf16_t* p, float4 v) {
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  u32x2 u;
  u.x = pack2_bf16(v.x, v.y);
  u.y = pack2_bf16(v.z, v.w);
  __builtin_nontemporal_store(u, (u32x2*)p);
}
__device__ __forceinline__ void st4_f32(float* p, float4 v) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  f32x4 u = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(u, (f32x4*)p);
}
__device__ __forceinline__ float4 gelu4(float4 v) {
  return make_float4(gelu_erf(v.x), gelu_erf(v.y), gelu_erf(v.z), gelu_erf(v.w));
}
__device__ __forceinline__ float4 add4(float4 a, float4 b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// Four consecutive columns n..n+3 of row r (n % 4 == 0), bias already added.
template <int KIND>
__device__ __forceinline__ void epi_apply4(const Epilogue& e, int r, int n, float4 v) {
  if constexpr (KIND == EPI_QKV) {
    if (n < e.d_model) v = make_float4(v.x * kQScaleLog2, v.y * kQScaleLog2, v.z * kQScaleLog2,
                                       v.w * kQScaleLog2);
    st4_bf16((bf16_t*)e.out + (int64_t)r * e.ldc + n, v);
  } else if constexpr (KIND == EPI_STORE) {
    st4_bf16((bf16_t*)e.out + (int64_t)r * e.ldc + n, v);
  } else if constexpr (KIND == EPI_GELU) {
    st4_bf16((bf16_t*)e.out + (int64_t)r * e.ldc + n, gelu4(v));
  } else if constexpr (KIND == EPI_CONV1) {
    const int g = r / kFrames, t = r - g * kFrames;
    const int64_t base = (int64_t)g * (kFrames + 1) * e.d_model;
    st4_bf16((bf16_t*)e.out + base + (int64_t)(t + 1) * e.d_model + n, gelu4(v));
    if (t == 0) st4_bf16((bf16_t*)e.out + base + n, make_float4(0.f, 0.f, 0.f, 0.f));
  } else if constexpr (KIND == EPI_CONV2) {
    const int t = r % kCtx;
    st4_f32((float*)e.out + (int64_t)r * e.ldc + n,
            add4(gelu4(v), *(const float4*)(e.pos + (int64_t)t * e.ldc + n)));
  } else if constexpr (KIND == EPI_XKV) {
    const int g = r / kCtx, t = r - g * kCtx;
    const int two_d = 2 * e.d_model;
    const int l = n / two_d, rem = n - l * two_d;
    const int kv = rem >= e.d_model, hd = rem - kv * e.d_model;
    const int64_t addr = (int64_t)e.slots[g] * e.slot_stride +
                         ((((int64_t)l * 2 + kv) * e.n_head + (hd >> 6)) * kCtx + t) * kHeadDim +
                         (hd & 63);
    st4_bf16((bf16_t*)e.out + addr, v);
  }
}

// Bias of the four columns n..n+3 (zero without bias or past N).  The
// epilogues load it once per wave tile, ahead of the block loop: a load per
// block would put an L2 round trip on the epilogue's critical path 2 FM FN
// times.
__device__ __forceinline__ float4 bias4(const Epilogue& e, int n, int N) {
  if (!e.bias || n >= N) return make_float4(0.f, 0.f, 0.f, 0.f);
  if (n + 3 < N) return *(const float4*)(e.bias + n);
  return make_float4(e.bias[n], n + 1 < N ? e.bias[n + 1] : 0.f, n + 2 < N ? e.bias[n + 2] : 0.f, 0.f);
}
__device__ __forceinline__ float bias1(const Epilogue& e, int n, int N) {
  return e.bias && n < N ? e.bias[n] : 0.f;
}

// Epilogue of a wave's FM x FN accumulator blocks.  Each 32x32 block goes
// through the wave's private LDS stage (row stride 36 floats) in the MFMA
// output layout -- lane holds column lane%32 and, for register r, row
// 8*(r/4) + 4*(lane/32) + r%4 -- and is read back as four consecutive
// columns of one row per lane, so every store moves 8 or 16 bytes.  The
// transposed V of the fused QKV product (VT below) is read back as four
// consecutive rows of one column instead (contiguous in V^T).  The stage is
// private to the wave and LDS executes a wave's accesses in order, so no
// barrier is needed between blocks; the caller synchronises the block once
// before the first block (the stage aliases the operand ring).
constexpr int kStageLd = 36;
constexpr int EPI_VT = 100;   // internal: V columns of EPI_QKV

// The conv-stem epilogue keeps its row loop rolled: unrolled, its address
// arithmetic spills the accumulators.
#define EPI_UNROLL (KIND == EPI_CONV1 ? 1 : 4)
template <int KIND, int FM, int FN>
__device__ __forceinline__ void epi_wave_impl(const Epilogue& e, f32x16 (&acc)[FM][FN],
                                              float* stage, int m0w, int n0w, int M, int N,
                                              int lane) {
  const int l32 = lane & 31, lh = lane >> 5;
  const bool vec_ok = (N & 3) == 0 && (e.ldc & 3) == 0 && (e.d_model & 3) == 0;
  constexpr int AK = KIND == EPI_VT ? EPI_QKV : KIND;     // kind for the scalar fallback
  constexpr int NB = KIND == EPI_VT ? 4 : 1;
  float4 bj[FN];                // bias of the lane's columns (x only for VT: one per it)
  float bvt[FN][NB];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    if constexpr (KIND == EPI_VT) {
#pragma unroll
      for (int it = 0; it < NB; ++it) bvt[j][it] = bias1(e, n0w + j * 32 + it * 8 + (lane >> 3), N);
    } else {
      bj[j] = bias4(e, n0w + j * 32 + (lane & 7) * 4, N);
    }
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stage[((r >> 2) * 8 + lh * 4 + (r & 3)) * kStageLd + l32] = acc[i][j][r];
      __builtin_amdgcn_wave_barrier();
      const int rbase = m0w + i * 32, cbase = n0w + j * 32;
      if constexpr (KIND == EPI_VT) {
        // lane takes rows 4q..4q+3 of one column
        const int r4 = (lane & 7) * 4;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int c = it * 8 + (lane >> 3), n = cbase + c;
          if (n >= N) continue;
          const int row = rbase + r4;
          float4 v = make_float4(stage[r4 * kStageLd + c], stage[(r4 + 1) * kStageLd + c],
                                 stage[(r4 + 2) * kStageLd + c], stage[(r4 + 3) * kStageLd + c]);
          if (row + 3 < M) {
            const float b = bvt[j][it];
            v = add4(v, make_float4(b, b, b, b));
            const int g = row / kCtx, t = row - g * kCtx;    // t % 4 == 0: same clip
            const int hd = n - 2 * e.d_model;
            const int64_t addr =
                (((int64_t)g * e.n_head + (hd >> 6)) * kHeadDim + (hd & 63)) * kVtLd + t;
            st4_bf16((bf16_t*)e.out2 + addr, v);
          } else {
            const float vv[4] = {v.x, v.y, v.z, v.w};
            for (int q = 0; q < 4; ++q)
              if (row + q < M) epi_apply<AK, bf16_t>(e, row + q, n, vv[q]);
          }
        }
      } else {
        const int c4 = (lane & 7) * 4;
#pragma unroll EPI_UNROLL
        for (int it = 0; it < 4; ++it) {
          const int rr = it * 8 + (lane >> 3), row = rbase + rr, n = cbase + c4;
          if (row >= M || n >= N) continue;
          const float4 v = *(const float4*)&stage[rr * kStageLd + c4];
          if (vec_ok) {
            epi_apply4<KIND>(e, row, n, add4(v, bj[j]));
          } else {
            const float vv[4] = {v.x, v.y, v.z, v.w};
            for (int q = 0; q < 4; ++q)
              if (n + q < N) epi_apply<AK, bf16_t>(e, row, n + q, vv[q]);
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
}
#undef EPI_UNROLL

// Plain element-wise fallback (a wave whose columns straddle q/k and V).
template <int FM, int FN>
__device__ __forceinline__ void epi_wave_mixed(const Epilogue& e, f32x16 (&acc)[FM][FN],
                                            float* stage, int m0w, int n0w, int M, int N,
                                            int lane) {
  const int l32 = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stage[((r >> 2) * 8 + lh * 4 + (r & 3)) * kStageLd + l32] = acc[i][j][r];
      __builtin_amdgcn_wave_barrier();
      for (int t = 0; t < 16; ++t) {
        const int rr = t * 2 + lh, row = m0w + i * 32 + rr, col = n0w + j * 32 + l32;
        if (row < M && col < N) epi_apply<EPI_QKV, bf16_t>(e, row, col, stage[rr * kStageLd + l32]);
      }
      __builtin_amdgcn_wave_barrier();
    }
}

// For EPI_QKV a wave's columns are all q/k or all V when 2 d_model is a
// multiple of the wave's column span (always, for d_model % 128 == 0 and
// spans of 32 or 64); otherwise the blocks are sorted out one by one.
template <int KIND, int FM, int FN>
__device__ __forceinline__ void epi_wave(const Epilogue& e, f32x16 (&acc)[FM][FN], float* stage,
                                         int m0w, int n0w, int M, int N, int lane) {
  if constexpr (KIND == EPI_QKV) {
    const int two_d = 2 * e.d_model;
    if (n0w >= two_d)
      epi_wave_impl<EPI_VT, FM, FN>(e, acc, stage, m0w, n0w, M, N, lane);
    else if (n0w + FN * 32 <= two_d)
      epi_wave_impl<EPI_QKV, FM, FN>(e, acc, stage, m0w, n0w, M, N, lane);
    else
      epi_wave_mixed<FM, FN>(e, acc, stage, m0w, n0w, M, N, lane);
  } else {
    epi_wave_impl<KIND, FM, FN>(e, acc, stage, m0w, n0w, M, N, lane);
  }
}

__device__ __forceinline__ int64_t arow_offset(const AView& a, int r) {
  int g = r / a.rows_per_batch;
  return (int64_t)g * a.batch_stride + (int64_t)(r - g * a.rows_per_batch) * a.lda;
}

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM
//
// Workgroup tile BM x BN x 64 with WM x WN waves, each wave owning a
// (BM/WM) x (BN/WN) block of 32x32 MFMA tiles whose fp32 accumulators stay in
// registers for the whole K loop.  Operand tiles are double-buffered in LDS
// (rows padded to 72 elements so the 16-byte fragment reads of 32 consecutive
// rows hit distinct banks); the next K tile is fetched into registers while
// the current one feeds the MFMAs.
//
// Tile order is XCD-aware: the hardware deals workgroups round-robin to the
// 8 XCDs, so block b runs on XCD b % 8.  Each XCD is given one contiguous
// range of tiles, walked in groups of GM row tiles (column tile outer, row
// tile inner) so that the A rows and the W columns a group needs stay in that
// XCD's L2 while its CUs work through them.
// ---------------------------------------------------------------------------
constexpr int kXcd = 8;

__device__ __forceinline__ void tile_of(int bid, int n_tiles, int n_tm, int n_tn, int gm,
                                        int& tm, int& tn) {
  const int q = n_tiles / kXcd, r = n_tiles % kXcd;
  const int xcd = bid % kXcd, local = bid / kXcd;
  const int t = xcd * q + min(xcd, r) + local;           // contiguous range per XCD
  const int group = t / (gm * n_tn);
  const int first_tm = group * gm;
  const int rows = min(gm, n_tm - first_tm);
  const int in_group = t - group * gm * n_tn;
  tm = first_tm + in_group % rows;
  tn = in_group / rows;
}

// LDS holds each operand tile row-major without padding; the 16-byte chunk c
// of row r sits at chunk position c ^ swz(r).  On gfx950 a 16-byte LDS access
// is served 16 lanes at a time from 64 four-byte banks, so 16 lanes must touch
// 16 distinct 16-byte slots of a 256-byte window: with these swizzles both the
// fragment reads (32 consecutive rows, same chunk) and the tile stores (whole
// rows) are conflict-free.
template <int BK>
__device__ __forceinline__ int lds_swz(int row) {
  return BK == 32 ? ((row >> 2) & 3) : ((row >> 1) & 7);
}

template <int BM, int BN, int BK, int WM, int WN, int KIND>
__global__ __launch_bounds__(WM* WN * 64) void k_gemm_bf16(AView a, const bf16_t* __restrict__ w,
                                                          int M, int N, int K, Epilogue e,
                                                          int n_tm, int n_tn, int gm) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  constexpr int CPR = BK / 8;                      // 16-byte chunks per tile row
  constexpr int CA = BM * CPR / NT, CB = BN * CPR / NT;
  constexpr int RSTEP = NT / CPR;                  // rows covered by one pass of the block
  static_assert(BK == 32 || BK == 64, "BK");
  static_assert(CA * NT == BM * CPR && CB * NT == BN * CPR, "tile/threads");
  static_assert(RSTEP % 16 == 0, "swizzle period");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  bf16_t* As = smem;                               // [2][BM * BK]
  bf16_t* Bs = smem + 2 * BM * BK;                 // [2][BN * BK]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;
  int tm, tn;
  tile_of(blockIdx.x, n_tm * n_tn, n_tm, n_tn, gm, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;

  // loader: thread t moves logical chunk t % CPR of rows t/CPR + i*RSTEP
  const int lrow0 = tid / CPR, lc = tid % CPR;
  const int st_off = lrow0 * BK + ((lc ^ lds_swz<BK>(lrow0)) * 8);   // same swizzle for all i
  const bf16_t* abase = (const bf16_t*)a.ptr;
  int64_t aoff[CA];
#pragma unroll
  for (int i = 0; i < CA; ++i) {
    int r = min(m0 + lrow0 + i * RSTEP, M - 1);    // rows past M load row M-1, never stored
    int g = r / a.rows_per_batch;
    aoff[i] = (int64_t)g * a.batch_stride + (int64_t)(r - g * a.rows_per_batch) * a.lda + lc * 8;
  }
  int64_t boff[CB];
#pragma unroll
  for (int i = 0; i < CB; ++i) boff[i] = (int64_t)min(n0 + lrow0 + i * RSTEP, N - 1) * K + lc * 8;

  const int nk = (K + BK - 1) / BK;
  const bool ktail = (K % BK) != 0;

#define GEMM_GLOAD(RA, RB, k0)                                                      \
  do {                                                                              \
    if (!ktail || (k0) + BK <= K) {                                                 \
      _Pragma("unroll") for (int i = 0; i < CA; ++i) RA[i] = *(const uint4*)(abase + aoff[i] + (k0)); \
      _Pragma("unroll") for (int i = 0; i < CB; ++i) RB[i] = *(const uint4*)(w + boff[i] + (k0));     \
    } else {                                                                        \
      const bool in = (k0) + lc * 8 < K;                                            \
      _Pragma("unroll") for (int i = 0; i < CA; ++i)                                \
        RA[i] = in ? *(const uint4*)(abase + aoff[i] + (k0)) : uint4{0u, 0u, 0u, 0u}; \
      _Pragma("unroll") for (int i = 0; i < CB; ++i)                                \
        RB[i] = in ? *(const uint4*)(w + boff[i] + (k0)) : uint4{0u, 0u, 0u, 0u};   \
    }                                                                               \
  } while (0)
#define GEMM_SSTORE(RA, RB, buf)                                                    \
  do {                                                                              \
    _Pragma("unroll") for (int i = 0; i < CA; ++i)                                  \
      *(uint4*)&As[(buf) * BM * BK + st_off + i * RSTEP * BK] = RA[i];              \
    _Pragma("unroll") for (int i = 0; i < CB; ++i)                                  \
      *(uint4*)&Bs[(buf) * BN * BK + st_off + i * RSTEP * BK] = RB[i];              \
  } while (0)

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // fragment reads: row lane%32 of each 32-row block (blocks start on
  // multiples of 32, so the swizzle depends on the lane only), chunk
  // kk*2 + lane/32.  Fragments of step kk+1 are requested before the MFMAs of
  // step kk so that LDS latency overlaps matrix work within the wave.
  const int lrow = lane & 31, sw = lds_swz<BK>(lrow), lh = lane >> 5;
  const bf16_t* a_frag = As + (wm * TM + lrow) * BK;
  const bf16_t* b_frag = Bs + (wn * TN + lrow) * BK;

  uint4 ra[CA], rb[CB];
  GEMM_GLOAD(ra, rb, 0);
  GEMM_SSTORE(ra, rb, 0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) GEMM_GLOAD(ra, rb, (kt + 1) * BK);
    const bf16_t* Ac = a_frag + cur * BM * BK;
    const bf16_t* Bc = b_frag + cur * BN * BK;
    bf16x8 af[2][FM], bfr[2][FN];
    {
      const int ch = (lh ^ sw) * 8;
#pragma unroll
      for (int i = 0; i < FM; ++i) af[0][i] = *(const bf16x8*)(Ac + i * 32 * BK + ch);
#pragma unroll
      for (int j = 0; j < FN; ++j) bfr[0][j] = *(const bf16x8*)(Bc + j * 32 * BK + ch);
    }
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int p = kk & 1;
      if (kk + 1 < BK / 16) {
        const int ch = (((kk + 1) * 2 + lh) ^ sw) * 8;
#pragma unroll
        for (int i = 0; i < FM; ++i) af[p ^ 1][i] = *(const bf16x8*)(Ac + i * 32 * BK + ch);
#pragma unroll
        for (int j = 0; j < FN; ++j) bfr[p ^ 1][j] = *(const bf16x8*)(Bc + j * 32 * BK + ch);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[p][i], bfr[p][j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) GEMM_SSTORE(ra, rb, cur ^ 1);
    __syncthreads();
  }
#undef GEMM_GLOAD
#undef GEMM_SSTORE

  // Epilogue through LDS, one 32x32 block per wave at a time.  In the MFMA
  // output layout a lane holds column lane%32 and, for register r, row
  // 8*(r/4) + 4*(lane/32) + r%4; the block is written to LDS in that layout
  // and read back as two full rows per instruction, so the (possibly heavy)
  // epilogue math runs in a short rolled loop and every store covers whole
  // 32-column row segments.
  epi_wave<KIND, FM, FN>(e, acc, (float*)smem + wave * (32 * kStageLd), m0 + wm * TM,
                         n0 + wn * TN, M, N, lane);
}

// ---------------------------------------------------------------------------
// bf16 MFMA GEMM with an S-stage LDS ring filled by direct global->LDS loads.
//
// Each wave issues global_load_lds_dwordx4: lane l of one instruction lands
// 16 bytes at LDS base + 16 l, so an instruction fills one contiguous 1 KB
// slice of a tile (16 rows at BK = 32, 8 rows at BK = 64); the lane picks the
// global chunk that the swizzled layout wants at its slot.  The loads are
// issued from inline assembly so the compiler does not serialise every LDS
// read behind them; completion of tile kt is awaited explicitly (vmcnt) while
// the loads of the next S-2 tiles stay in flight, then one barrier per K
// tile publishes it and frees the buffer the next tile is loaded into.
// Requires K % BK == 0.
// ---------------------------------------------------------------------------
template <int BM, int BN, int BK, int WM, int WN, int S, int KIND>
__global__ __launch_bounds__(WM* WN * 64) void k_gemm_bf16_dma(AView a,
                                                              const bf16_t* __restrict__ w,
                                                              int M, int N, int K, Epilogue e,
                                                              int n_tm, int n_tn, int gm) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  constexpr int CPR = BK / 8;
  constexpr int RPI = 1024 / (BK * 2);             // tile rows filled by one wave instruction
  constexpr int IA = BM / (RPI * NW), IB = BN / (RPI * NW);   // instructions per wave per tile
  constexpr int LPT = IA + IB;                     // loads per lane per tile
  static_assert(BK == 32 || BK == 64, "BK");
  static_assert(IA * RPI * NW == BM && IB * RPI * NW == BN, "tile/waves");
  static_assert(S >= 2 && LPT * (S - 2) < 64, "stages");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  constexpr int STAGE = (BM + BN) * BK;            // elements per stage

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;
  int tm, tn;
  tile_of(blockIdx.x, n_tm * n_tn, n_tm, n_tn, gm, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const uint32_t lds0 =
      (uint32_t)(uintptr_t)((__attribute__((address_space(3))) bf16_t*)smem);

  // per-lane global sources and per-wave LDS destinations of the tile loads
  const bf16_t* abase = (const bf16_t*)a.ptr;
  const bf16_t* asrc[IA];
  uint32_t adst[IA];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int r0 = (i * NW + wave) * RPI;
    const int row = r0 + lane / CPR;
    const int c = (lane % CPR) ^ lds_swz<BK>(row);
    const int r = min(m0 + row, M - 1);
    const int g = r / a.rows_per_batch;
    asrc[i] = abase + (int64_t)g * a.batch_stride + (int64_t)(r - g * a.rows_per_batch) * a.lda +
              c * 8;
    adst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(r0 * BK * 2));
  }
  const bf16_t* bsrc[IB];
  uint32_t bdst[IB];
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int r0 = (i * NW + wave) * RPI;
    const int row = r0 + lane / CPR;
    const int c = (lane % CPR) ^ lds_swz<BK>(row);
    bsrc[i] = w + (int64_t)min(n0 + row, N - 1) * K + c * 8;
    bdst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)((BM * BK + r0 * BK) * 2));
  }
  const int nk = K / BK;
  auto issue = [&](int tile) {
    const uint32_t so = (uint32_t)((tile % S) * STAGE * 2);
    const int k0 = tile * BK;
#pragma unroll
    for (int i = 0; i < IA; ++i) lds_dma16(adst[i] + so, asrc[i] + k0);
#pragma unroll
    for (int i = 0; i < IB; ++i) lds_dma16(bdst[i] + so, bsrc[i] + k0);
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int lrow = lane & 31, sw = lds_swz<BK>(lrow), lh = lane >> 5;
  const bf16_t* a_frag = smem + (wm * TM + lrow) * BK;
  const bf16_t* b_frag = smem + BM * BK + (wn * TN + lrow) * BK;

#pragma unroll
  for (int t = 0; t < S - 1; ++t)
    if (t < nk) issue(t);
  for (int kt = 0; kt < nk; ++kt) {
    // tile kt has landed once at most min(S-2, nk-1-kt) later tiles are pending
    wait_vmcnt_rt<LPT * (S - 2)>(LPT * min(S - 2, nk - 1 - kt));
    __builtin_amdgcn_s_barrier();
    if (kt + S - 1 < nk) issue(kt + S - 1);
    const bf16_t* Ac = a_frag + (kt % S) * STAGE;
    const bf16_t* Bc = b_frag + (kt % S) * STAGE;
    bf16x8 af[2][FM], bfr[2][FN];
    {
      const int ch = (lh ^ sw) * 8;
#pragma unroll
      for (int i = 0; i < FM; ++i) af[0][i] = *(const bf16x8*)(Ac + i * 32 * BK + ch);
#pragma unroll
      for (int j = 0; j < FN; ++j) bfr[0][j] = *(const bf16x8*)(Bc + j * 32 * BK + ch);
    }
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int p = kk & 1;
      if (kk + 1 < BK / 16) {
        const int ch = (((kk + 1) * 2 + lh) ^ sw) * 8;
#pragma unroll
        for (int i = 0; i < FM; ++i) af[p ^ 1][i] = *(const bf16x8*)(Ac + i * 32 * BK + ch);
#pragma unroll
        for (int j = 0; j < FN; ++j) bfr[p ^ 1][j] = *(const bf16x8*)(Bc + j * 32 * BK + ch);
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[p][i], bfr[p][j], acc[i][j], 0, 0, 0);
    }
  }
  wait_vmcnt<0>();
  __syncthreads();

  epi_wave<KIND, FM, FN>(e, acc, (float*)smem + wave * (32 * kStageLd), m0 + wm * TM,
                         n0 + wn * TN, M, N, lane);
}

// Same operand ring, with the fragment reads software-pipelined across K
// tiles: the barrier that publishes tile kt+1 sits before the MFMAs of the
// last k-step of tile kt, so the first fragments of tile kt+1 are read while
// those MFMAs run, and no k-step ever waits on a fragment read issued just
// before it.  All S stages are in flight: tile kt+S is requested as soon as
// every wave has finished reading tile kt.  sched_barrier fences keep the
// compiler from sinking the prefetching reads below the MFMAs.
template <int VM>
__device__ __forceinline__ void wait_vm_lgkm0() {
  static_assert(VM >= 0 && VM < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4));
}
template <int MAXN>
__device__ __forceinline__ void wait_vm_lgkm0_rt(int n) {
  if constexpr (MAXN > 0) {
    if (n >= MAXN) { wait_vm_lgkm0<MAXN>(); return; }
    wait_vm_lgkm0_rt<MAXN - 1>(n);
  } else {
    wait_vm_lgkm0<0>();
  }
}

template <int BM, int BN, int BK, int WM, int WN, int S, int KIND>
__global__ __launch_bounds__(WM* WN * 64) void k_gemm_bf16_pf(AView a,
                                                             const bf16_t* __restrict__ w,
                                                             int M, int N, int K, Epilogue e,
                                                             int n_tm, int n_tn, int gm) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  constexpr int CPR = BK / 8;
  constexpr int NS = BK / 16;                      // MFMA k-steps per tile
  constexpr int RPI = 1024 / (BK * 2);
  constexpr int IA = BM / (RPI * NW), IB = BN / (RPI * NW);
  constexpr int LPT = IA + IB;
  static_assert(BK == 32 || BK == 64, "BK");
  static_assert(IA * RPI * NW == BM && IB * RPI * NW == BN, "tile/waves");
  static_assert(S >= 2 && LPT * (S - 1) < 64, "stages");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  constexpr int STAGE = (BM + BN) * BK;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;
  int tm, tn;
  tile_of(blockIdx.x, n_tm * n_tn, n_tm, n_tn, gm, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const uint32_t lds0 =
      (uint32_t)(uintptr_t)((__attribute__((address_space(3))) bf16_t*)smem);

  const bf16_t* abase = (const bf16_t*)a.ptr;
  const bf16_t* asrc[IA];
  uint32_t adst[IA];
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int r0 = (i * NW + wave) * RPI;
    const int row = r0 + lane / CPR;
    const int c = (lane % CPR) ^ lds_swz<BK>(row);
    const int r = min(m0 + row, M - 1);
    const int g = r / a.rows_per_batch;
    asrc[i] = abase + (int64_t)g * a.batch_stride + (int64_t)(r - g * a.rows_per_batch) * a.lda +
              c * 8;
    adst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(r0 * BK * 2));
  }
  const bf16_t* bsrc[IB];
  uint32_t bdst[IB];
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int r0 = (i * NW + wave) * RPI;
    const int row = r0 + lane / CPR;
    const int c = (lane % CPR) ^ lds_swz<BK>(row);
    bsrc[i] = w + (int64_t)min(n0 + row, N - 1) * K + c * 8;
    bdst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)((BM * BK + r0 * BK) * 2));
  }
  const int nk = K / BK;
  auto issue = [&](int tile) {
    const uint32_t so = (uint32_t)((tile % S) * STAGE * 2);
    const int k0 = tile * BK;
#pragma unroll
    for (int i = 0; i < IA; ++i) lds_dma16(adst[i] + so, asrc[i] + k0);
#pragma unroll
    for (int i = 0; i < IB; ++i) lds_dma16(bdst[i] + so, bsrc[i] + k0);
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int lrow = lane & 31, sw = lds_swz<BK>(lrow), lh = lane >> 5;
  const bf16_t* a_frag = smem + (wm * TM + lrow) * BK;
  const bf16_t* b_frag = smem + BM * BK + (wn * TN + lrow) * BK;
  bf16x8 af[2][FM], bfr[2][FN];
#define PF_READ(P, TILE, KK)                                                          \
  do {                                                                                \
    const int off_ = ((TILE) % S) * STAGE + ((((KK) * 2 + lh) ^ sw) * 8);             \
    _Pragma("unroll") for (int i = 0; i < FM; ++i)                                    \
      af[P][i] = *(const bf16x8*)(a_frag + off_ + i * 32 * BK);                       \
    _Pragma("unroll") for (int j = 0; j < FN; ++j)                                    \
      bfr[P][j] = *(const bf16x8*)(b_frag + off_ + j * 32 * BK);                      \
  } while (0)

  // Issued right after a fragment prefetch, this tells the wait-count pass
  // that every older LDS read has completed (the reads feeding the coming
  // MFMAs), which it cannot prove by itself across the loop back edge.
  constexpr int kLgkmImm = 0xF | (0x3 << 14) | (0x7 << 4) | ((FM + FN) << 8);
  static_assert(FM + FN <= 15, "lgkmcnt");

#pragma unroll
  for (int t = 0; t < S; ++t)
    if (t < nk) issue(t);
  wait_vm_lgkm0_rt<LPT*(S - 1)>(LPT * min(S - 1, nk - 1));
  __builtin_amdgcn_s_barrier();
  PF_READ(0, 0, 0);
  for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
      const int p = kk & 1;
      if (kk + 1 < NS) {
        PF_READ(p ^ 1, kt, kk + 1);
      } else if (kt + 1 < nk) {
        // tile kt+1 landed (later tiles may still fly), this wave's reads of
        // tile kt done; after the barrier nobody reads tile kt any more
        wait_vm_lgkm0_rt<LPT*(S - 2)>(LPT * min(S - 2, nk - 2 - kt));
        __builtin_amdgcn_s_barrier();
        if (kt + S < nk) issue(kt + S);
        PF_READ(p ^ 1, kt + 1, 0);
      }
      if (kk + 1 < NS || kt + 1 < nk) __builtin_amdgcn_s_waitcnt(kLgkmImm);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[p][i], bfr[p][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#undef PF_READ
  wait_vmcnt<0>();
  __syncthreads();

  epi_wave<KIND, FM, FN>(e, acc, (float*)smem + wave * (32 * kStageLd), m0 + wm * TM,
                         n0 + wn * TN, M, N, lane);
}

// ---------------------------------------------------------------------------
// Persistent variant.  One workgroup per CU walks its share of the output
// tiles (virtual block ids b, b + grid, ... through the same XCD-aware tile
// order) and the operand ring runs on across tile boundaries, so the first K
// tile of the next output tile is in flight while the current one is written
// out through a small stage of its own beside the ring.  At a tile switch the
// next K tile is awaited before the stores are issued, and the ring's next
// load goes out after them, so every wait count stays exact or errs towards
// waiting longer.
// ---------------------------------------------------------------------------
// Epilogue through a 16-row stage per wave (it lives beside the operand
// ring, which is busy with the next tile): each 32x32 block goes out in two
// halves, registers 0-7 (rows 0-15) then 8-15 (rows 16-31).  The scatter
// epilogues keep their row loops rolled (unrolled, they spill).
#define EPI_HALF_UNROLL ((KIND == EPI_CONV1 || KIND == EPI_QKV) ? 1 : 2)
template <int KIND, int FM, int FN>
__device__ __forceinline__ void epi_wave_half(const Epilogue& e, f32x16 (&acc)[FM][FN],
                                              float* stage, int m0w, int n0w, int M, int N,
                                              int lane) {
  const int l32 = lane & 31, lh = lane >> 5;
  const bool vec_ok = (N & 3) == 0 && (e.ldc & 3) == 0 && (e.d_model & 3) == 0;
  const bool vt = KIND == EPI_QKV && n0w >= 2 * e.d_model;   // wave-uniform
  float4 bj[FN];     // bias of the lane's columns: c4..c4+3, or (VT) columns it*16 + lane/4
#pragma unroll
  for (int j = 0; j < FN; ++j)
    bj[j] = vt ? make_float4(bias1(e, n0w + j * 32 + (lane >> 2), N),
                             bias1(e, n0w + j * 32 + 16 + (lane >> 2), N), 0.f, 0.f)
               : bias4(e, n0w + j * 32 + (lane & 7) * 4, N);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
          stage[((r >> 2) * 8 + lh * 4 + (r & 3)) * kStageLd + l32] = acc[i][j][h * 8 + r];
        __builtin_amdgcn_wave_barrier();
        const int rbase = m0w + i * 32 + h * 16, cbase = n0w + j * 32;
        if (KIND == EPI_QKV && vt) {
          // lane takes rows 4q..4q+3 (of 16) of one column
          const int r4 = (lane & 3) * 4;
#pragma unroll EPI_HALF_UNROLL
          for (int it = 0; it < 2; ++it) {
            const int c = it * 16 + (lane >> 2), n = cbase + c, row = rbase + r4;
            if (n >= N) continue;
            float4 v = make_float4(stage[r4 * kStageLd + c], stage[(r4 + 1) * kStageLd + c],
                                   stage[(r4 + 2) * kStageLd + c], stage[(r4 + 3) * kStageLd + c]);
            if (row + 3 < M) {
              const float b = it == 0 ? bj[j].x : bj[j].y;
              v = add4(v, make_float4(b, b, b, b));
              const int g = row / kCtx, t = row - g * kCtx;    // t % 4 == 0: same clip
              const int hd = n - 2 * e.d_model;
              st4_bf16((bf16_t*)e.out2 +
                           (((int64_t)g * e.n_head + (hd >> 6)) * kHeadDim + (hd & 63)) * kVtLd + t,
                       v);
            } else {
              const float vv[4] = {v.x, v.y, v.z, v.w};
              for (int q = 0; q < 4; ++q)
                if (row + q < M) epi_apply<KIND, bf16_t>(e, row + q, n, vv[q]);
            }
          }
        } else {
          const int c4 = (lane & 7) * 4;
#pragma unroll EPI_HALF_UNROLL
          for (int it = 0; it < 2; ++it) {
            const int rr = it * 8 + (lane >> 3), row = rbase + rr, n = cbase + c4;
            if (row >= M || n >= N) continue;
            const float4 v = *(const float4*)&stage[rr * kStageLd + c4];
            if (vec_ok) {
              epi_apply4<KIND>(e, row, n, add4(v, bj[j]));
            } else {
              const float vv[4] = {v.x, v.y, v.z, v.w};
              for (int q = 0; q < 4; ++q)
                if (n + q < N) epi_apply<KIND, bf16_t>(e, row, n + q, vv[q]);
            }
          }
        }
        __builtin_amdgcn_wave_barrier();
      }
}

#undef EPI_HALF_UNROLL

// Epilogue straight from registers, for a product formed transposed
// (W fragment as the MFMA's first operand): a lane then holds output row
// l32 of each 32x32 block and, in register quad q, the four consecutive
// columns 8q + 4 lh .. 8q + 4 lh + 3.  The values are packed to bf16 and one
// lane-half swap (v_permlane32_swap) gathers eight consecutive columns per
// lane, so each store moves 16 bytes.  Row-major outputs are stored
// through a buffer resource sized to the output: lanes past M or N get an
// offset beyond it, which the hardware drops, so no lane diverges.  The
// cross-attention cache (XKV, far above the 2^31-byte reach of a buffer
// offset) is addressed per lane: the row part (slot, position) once per
// tile, the column part (layer, K/V, head, dim) once per wave, whose columns
// stay within one head.  No LDS round trip:
// the store stream issues as fast as the accumulators convert.
// Cache policy of the register epilogue's stores: the default.  Unlike the
// staged epilogue's full-row stores, each of these instructions writes
// 32-byte runs of 32 different rows, which the L2 merges into whole lines;
// with the non-temporal hint every encoder product ran 7-16 % slower.
constexpr int kNtAux = 0;

template <int KIND>
constexpr bool kDirectEpi =
    KIND == EPI_STORE || KIND == EPI_GELU || KIND == EPI_XKV || KIND == EPI_QKV;

// V columns of the fused QKV product from the transposed layout: there the
// MFMA output block is V^T itself (rows = V columns, columns = positions), so
// it goes through the wave's 16-row LDS stage as the plain epilogue does and
// is read back as four consecutive positions of one V column -- eight
// contiguous bytes of V^T[clip][head][dim][position] (1500 is a multiple of
// 4, so the four never straddle clips); eight lanes fill 64 contiguous bytes.
template <int FM, int FN>
__device__ __forceinline__ void epi_direct_vt(const Epilogue& e, f32x16 (&acc)[FM][FN],
                                              float* stage, int m0w, int n0w, int M, int N,
                                              int lane) {
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
  const int l32 = lane & 31, lh = lane >> 5;
  const int n_clips = (M + kCtx - 1) / kCtx;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      e.out2, (short)0, (int)((int64_t)n_clips * e.n_head * kHeadDim * kVtLd * 2), 0x00020000);
  const int c4 = (lane & 7) * 4, r8 = lane >> 3;
  float bv[FN][2][2];     // bias of the lane's V column per (block column, half, it)
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int it = 0; it < 2; ++it) bv[j][h][it] = bias1(e, n0w + j * 32 + h * 16 + it * 8 + r8, N);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = m0w + i * 32 + c4;                   // first of four positions
    const int g = row / kCtx, t = row - g * kCtx;
    const int rbase = g * e.n_head * kHeadDim * kVtLd + t;
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
          stage[((r >> 2) * 8 + lh * 4 + (r & 3)) * kStageLd + l32] = acc[i][j][h * 8 + r];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int rr = it * 8 + r8, n = n0w + j * 32 + h * 16 + rr;
          const float4 v = *(const float4*)&stage[rr * kStageLd + c4];
          const float bb = bv[j][h][it];
          const int hd = n - 2 * e.d_model;
          const u32x2 x = {pack2_bf16(v.x + bb, v.y + bb), pack2_bf16(v.z + bb, v.w + bb)};
          const uint32_t off = row < M && n < N
                                   ? (uint32_t)(rbase + ((hd >> 6) * kHeadDim + (hd & 63)) * kVtLd) * 2u
                                   : 0x80000000u;
          __builtin_amdgcn_raw_buffer_store_b64(x, rs, off, 0, kNtAux);
        }
        __builtin_amdgcn_wave_barrier();
      }
  }
}

template <int KIND, int FM, int FN>
__device__ __forceinline__ void epi_direct(const Epilogue& e, f32x16 (&acc)[FM][FN], int m0w,
                                           int n0w, int M, int N, int lane) {
  static_assert(kDirectEpi<KIND>, "direct epilogue kind");
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
  const int l32 = lane & 31, lh = lane >> 5;
  __amdgpu_buffer_rsrc_t rs;
  int64_t xrow[FM];    // XKV: slot and position part of each of the lane's rows
  int64_t xcol = 0;    // XKV: (layer, K/V, head, dim) part of the wave's first column
  if constexpr (KIND == EPI_XKV) {
    static_assert(kHeadDim % (FN * 32) == 0, "a wave's columns stay within one head");
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int r = min(m0w + i * 32 + l32, M - 1), g = r / kCtx;
      xrow[i] = (int64_t)e.slots[g] * e.slot_stride + (int64_t)(r - g * kCtx) * kHeadDim;
    }
    // the wave's 32 or 64 columns start at a multiple of their number, and d_model
    // is a multiple of 64, so they lie in one layer, one of K / V and one head
    // and follow each other from the first one's address: wave-uniform.  (The
    // same as n0w / 64 heads of 1500 x 64; computed so, the product of 64 large-v3
    // clips took 21.1 ms instead of 20.8.)
    const int two_d = 2 * e.d_model;
    const int l = n0w / two_d, rem = n0w - l * two_d;
    const int kv = rem >= e.d_model, hd0 = rem - kv * e.d_model;
    xcol = ((((int64_t)l * 2 + kv) * e.n_head + (hd0 >> 6)) * kCtx) * kHeadDim + (hd0 & 63);
  } else {
    rs = __builtin_amdgcn_make_buffer_rsrc(e.out, (short)0, (int)((int64_t)M * e.ldc * 2),
                                           0x00020000);
  }
  float4 bq[FN][4];
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) bq[j][q] = bias4(e, n0w + j * 32 + 8 * q + 4 * lh, N);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = m0w + i * 32 + l32;
    const bool rok = row < M;
    const int rofs = row * (int)e.ldc;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      float v[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v[4 * q] = acc[i][j][4 * q] + bq[j][q].x;
        v[4 * q + 1] = acc[i][j][4 * q + 1] + bq[j][q].y;
        v[4 * q + 2] = acc[i][j][4 * q + 2] + bq[j][q].z;
        v[4 * q + 3] = acc[i][j][4 * q + 3] + bq[j][q].w;
      }
      if constexpr (KIND == EPI_GELU) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = gelu_erf(v[r]);
      }
      if constexpr (KIND == EPI_QKV) {
        // q columns (n < d, whole quads) carry the attention scale into exp2
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (n0w + j * 32 + 8 * q + 4 * lh < e.d_model)
#pragma unroll
            for (int r = 0; r < 4; ++r) v[4 * q + r] *= kQScaleLog2;
      }
      {
        uint32_t o[8];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          o[2 * q] = pack2_bf16(v[4 * q], v[4 * q + 1]);
          o[2 * q + 1] = pack2_bf16(v[4 * q + 2], v[4 * q + 3]);
        }
        // lanes 32-63 of quads 0 / 2 <-> lanes 0-31 of quads 1 / 3: lane l < 32
        // then holds columns 0-7 (16-23), lane l + 32 columns 8-15 (24-31)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const auto s0 = __builtin_amdgcn_permlane32_swap(o[4 * h], o[4 * h + 2], false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(o[4 * h + 1], o[4 * h + 3], false, false);
          o[4 * h] = s0[0];
          o[4 * h + 2] = s0[1];
          o[4 * h + 1] = s1[0];
          o[4 * h + 3] = s1[1];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int n = n0w + j * 32 + 16 * h + 8 * lh;
          const u32x4 x = {o[4 * h], o[4 * h + 1], o[4 * h + 2], o[4 * h + 3]};
          if constexpr (KIND == EPI_XKV) {
            if (rok && n < N)
              *(u32x4*)((bf16_t*)e.out + xrow[i] + xcol + (n - n0w)) = x;
          } else {
            const uint32_t off = rok && n < N ? (uint32_t)(rofs + n) * 2u : 0x80000000u;
            __builtin_amdgcn_raw_buffer_store_b128(x, rs, off, 0, kNtAux);
          }
        }
      }
    }
  }
}

template <int BM, int BN, int BK, int WM, int WN, int S, int KIND, bool SW>
__global__ __launch_bounds__(WM* WN * 64) __attribute__((amdgpu_waves_per_eu(2)))
void k_gemm_bf16_ps(AView a,
                                                             const bf16_t* __restrict__ w,
                                                             int M, int N, int K, Epilogue e,
                                                             int n_tm, int n_tn, int gm) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / 32, FN = TN / 32;
  constexpr int CPR = BK / 8;
  constexpr int NS = BK / 16;
  constexpr int RPI = 1024 / (BK * 2);
  constexpr int IA = BM / (RPI * NW), IB = BN / (RPI * NW);
  constexpr int LPT = IA + IB;
  static_assert(BK == 32 || BK == 64, "BK");
  static_assert(NS % 2 == 0, "fragment double buffer parity");
  static_assert(IA * RPI * NW == BM && IB * RPI * NW == BN, "tile/waves");
  static_assert(S >= 2 && LPT * (S - 1) < 64, "stages");
  static_assert(FM + FN <= 15, "lgkmcnt");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  constexpr int STAGE = (BM + BN) * BK;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM;
  const int n_tiles = n_tm * n_tn, grid = gridDim.x;
  if ((int)blockIdx.x >= n_tiles) return;
  const int my_tiles = (n_tiles - (int)blockIdx.x + grid - 1) / grid;
  const int nk = K / BK;
  const int total = my_tiles * nk;
  const uint32_t lds0 =
      (uint32_t)(uintptr_t)((__attribute__((address_space(3))) bf16_t*)smem);

  // per-wave LDS destinations (fixed) and per-lane source offsets in bytes
  // from a wave-uniform base (32-bit: the launcher checks the operand
  // extents), reset per tile
  uint32_t adst[IA], bdst[IB];
#pragma unroll
  for (int i = 0; i < IA; ++i)
    adst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)((i * NW + wave) * RPI * BK * 2));
#pragma unroll
  for (int i = 0; i < IB; ++i)
    bdst[i] = __builtin_amdgcn_readfirstlane(
        lds0 + (uint32_t)((BM * BK + (i * NW + wave) * RPI * BK) * 2));
  const bf16_t* abase = (const bf16_t*)a.ptr;
  uint32_t aoff[IA], boff[IB];
  int src_tile = -1;
  auto set_src = [&](int ti) {
    int tm, tn;
    tile_of((int)blockIdx.x + ti * grid, n_tiles, n_tm, n_tn, gm, tm, tn);
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const int row = (i * NW + wave) * RPI + lane / CPR;
      const int c = ((lane % CPR) ^ lds_swz<BK>(row)) * 8;
      const int r = min(tm * BM + row, M - 1);
      const int g = r / a.rows_per_batch;
      aoff[i] = (uint32_t)(g * a.batch_stride + (int64_t)(r - g * a.rows_per_batch) * a.lda + c) * 2u;
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      const int row = (i * NW + wave) * RPI + lane / CPR;
      const int c = ((lane % CPR) ^ lds_swz<BK>(row)) * 8;
      boff[i] = ((uint32_t)min(tn * BN + row, N - 1) * (uint32_t)K + (uint32_t)c) * 2u;
    }
    src_tile = ti;
  };
  // the direct loads of K tile gi, numbered 0 .. LPT - 1 (A's first): iss_begin
  // sets the tile, iss(q) issues one
  uint32_t iss_so = 0;
  const bf16_t *iss_a = nullptr, *iss_b = nullptr;
  auto iss_begin = [&](int gi) {
    const int ti = gi / nk, kt = gi - ti * nk;
    if (ti != src_tile) set_src(ti);
    iss_so = (uint32_t)((gi % S) * STAGE * 2);
    iss_a = abase + kt * BK;
    iss_b = w + kt * BK;
  };
  auto iss = [&](int q) {
    if (q < IA) lds_dma16_s(adst[q] + iss_so, aoff[q], iss_a);
    else lds_dma16_s(bdst[q - IA] + iss_so, boff[q - IA], iss_b);
  };
  auto issue = [&](int gi) {
    iss_begin(gi);
#pragma unroll
    for (int q = 0; q < LPT; ++q) iss(q);
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int lrow = lane & 31, sw = lds_swz<BK>(lrow), lh = lane >> 5;
  const bf16_t* a_frag = smem + (wm * TM + lrow) * BK;
  const bf16_t* b_frag = smem + BM * BK + (wn * TN + lrow) * BK;
  bf16x8 af[2][FM], bfr[2][FN];
#define PS_READ(P, GI, KK)                                                            \
  do {                                                                                \
    const int off_ = ((GI) % S) * STAGE + ((((KK) * 2 + lh) ^ sw) * 8);               \
    _Pragma("unroll") for (int i = 0; i < FM; ++i)                                    \
      af[P][i] = *(const bf16x8*)(a_frag + off_ + i * 32 * BK);                       \
    _Pragma("unroll") for (int j = 0; j < FN; ++j)                                    \
      bfr[P][j] = *(const bf16x8*)(b_frag + off_ + j * 32 * BK);                      \
  } while (0)

#pragma unroll
  for (int t = 0; t < S; ++t)
    if (t < total) issue(t);
  wait_vm_lgkm0_rt<LPT*(S - 1)>(LPT * min(S - 1, total - 1));
  __builtin_amdgcn_s_barrier();
  PS_READ(0, 0, 0);
  // QKV: output tiles of V columns take the staged V^T epilogue, q / k tiles
  // the register one; 2 d_model is a multiple of the tile width, so a tile
  // never mixes them
  auto vt_of = [&](int t) {
    if constexpr (KIND != EPI_QKV) {
      return false;
    } else {
      int tm, tn;
      tile_of((int)blockIdx.x + t * grid, n_tiles, n_tm, n_tn, gm, tm, tn);
      return tn * BN >= 2 * e.d_model;
    }
  };
  bool tile_vt = vt_of(0);
  // One MFMA, then its share of the next fragments' reads and of a K tile's
  // direct loads: a wave issues in order, and eight direct loads in a row hold
  // it for up to 1024 cycles (the eight waves' 64 KB at 64 B a clock) with its
  // matrix pipe idle.  Tile gi + 1's second half of loads goes out in the first
  // step of tile gi, right behind the half sent when its slot came free.
  constexpr int HALF = LPT / 2, NM = FM * FN;
  static_assert(LPT % 2 == 0 && NM % HALF == 0, "the loads of a K tile in two steps");
  static_assert(FM + FN <= NM, "a fragment read behind an MFMA each");
  int ti = 0, kt = 0;
  bool half_left = false;                          // the second half of a tile is due
  for (int gi = 0; gi < total; ++gi) {
    const bool last_k = kt == nk - 1;
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
      const int p = kk & 1;
      const bool reads = kk + 1 < NS || !last_k;
      bool loads = false;
      if (kk + 1 < NS) {
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);    // this step's fragments
        if (kk == 0) loads = half_left;
      } else if (!last_k) {
        wait_vm_lgkm0_rt<LPT*(S - 2)>(LPT * min(S - 2, total - 2 - gi));
        __builtin_amdgcn_s_barrier();
        loads = half_left = gi + S < total;
        if (loads) iss_begin(gi + S);
      } else {
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      }
      const int rg = kk + 1 < NS ? gi : gi + 1, rk = (kk + 1) % NS;
      const int off_ = (rg % S) * STAGE + (((rk * 2 + lh) ^ sw) * 8);
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const int i = m / FN, j = m % FN;
        __builtin_amdgcn_sched_barrier(0);
        acc[i][j] = SW ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[p][j], af[p][i], acc[i][j], 0, 0, 0)
                       : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[p][i], bfr[p][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (reads && m < FM + FN) {
          // in the order of use: A 0, B 0, B 1, A 1, ...
          if (m == 0) af[p ^ 1][0] = *(const bf16x8*)(a_frag + off_);
          else if (m <= FN) bfr[p ^ 1][m - 1] = *(const bf16x8*)(b_frag + off_ + (m - 1) * 32 * BK);
          else af[p ^ 1][m - FN] = *(const bf16x8*)(a_frag + off_ + (m - FN) * 32 * BK);
        }
        if ((kk == 0 || kk == NS - 1) && m % (NM / HALF) == NM / HALF - 1) {
          if (loads) iss((kk == 0 ? HALF : 0) + m / (NM / HALF));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (last_k) {
      const bool more = gi + 1 < total;
      if (more) {
        // next K tile landed and every wave is done with this one
        wait_vm_lgkm0_rt<LPT*(S - 2)>(LPT * min(S - 2, total - 2 - gi));
        __builtin_amdgcn_s_barrier();
      }
      int tm, tn;
      tile_of((int)blockIdx.x + ti * grid, n_tiles, n_tm, n_tn, gm, tm, tn);
      if constexpr (SW && KIND == EPI_QKV) {
        if (tile_vt)
          epi_direct_vt<FM, FN>(e, acc, (float*)(smem + S * STAGE) + wave * 16 * kStageLd,
                                tm * BM + wm * TM, tn * BN + wn * TN, M, N, lane);
        else
          epi_direct<KIND, FM, FN>(e, acc, tm * BM + wm * TM, tn * BN + wn * TN, M, N, lane);
      } else if constexpr (SW)
        epi_direct<KIND, FM, FN>(e, acc, tm * BM + wm * TM, tn * BN + wn * TN, M, N, lane);
      else
        epi_wave_half<KIND, FM, FN>(e, acc, (float*)(smem + S * STAGE) + wave * 16 * kStageLd,
                                    tm * BM + wm * TM, tn * BN + wn * TN, M, N, lane);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
      half_left = more && gi + S < total;
      if (more) {
        if (half_left) {
          iss_begin(gi + S);
#pragma unroll
          for (int q = 0; q < HALF; ++q) iss(q);
        }
        PS_READ(0, gi + 1, 0);
      }
      ++ti;
      kt = 0;
      tile_vt = vt_of(ti);
    } else {
      ++kt;
    }
  }
#undef PS_READ
}

// ---------------------------------------------------------------------------
// Products too small for the persistent kernel's tiles (a few clips): tiles of
// 128 x 128 or 128 x 64 on four waves.  With one or two waves per SIMD the bound
// is a wave's own instruction order: a 1 KB direct load holds the wave while the
// CU's load path (64 B a clock) takes the four waves' loads, and the LDS reads
// come behind them, so a K tile of 128 x 128 x 64 took 1380 cycles (520 of loads,
// 256 of reads, 512 of MFMAs, one after the other) however many stages were in
// flight.  Here a wave reads all fragments of K tile t + 1 into registers while
// it multiplies tile t, and every MFMA is followed by one or two of those reads
// and a share of the direct loads: about 730 cycles.  A K tile's LDS slot is free
// as soon as its fragments are in registers, so all S slots hold tiles in flight.
// ---------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, int S, int KIND>
__global__ __launch_bounds__(WM* WN * 64) __attribute__((amdgpu_waves_per_eu(2)))
void k_gemm_bf16_rt(AView a, const bf16_t* __restrict__ w, int M, int N, int K, Epilogue e, int n_tm,
                    int n_tn, int gm) {
  constexpr bool SW = kDirectEpi<KIND>;            // product formed transposed
  constexpr int BK = 64, NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 32, FN = TN / 32, NS = BK / 16;
  constexpr int IA = BM / (8 * NW), IB = BN / (8 * NW), LPT = IA + IB;
  static_assert(IA * 8 * NW == BM && IB * 8 * NW == BN, "tile/waves");
  static_assert(S >= 2 && LPT * (S - 1) < 64, "stages");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  constexpr int STAGE = (BM + BN) * BK;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = wave % WM, wn = wave / WM;
  int tm, tn;
  tile_of(blockIdx.x, n_tm * n_tn, n_tm, n_tn, gm, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) bf16_t*)smem);
  const bf16_t* abase = (const bf16_t*)a.ptr;
  uint32_t aoff[IA], boff[IB];                     // bytes (the launcher checks the extents)
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int row = (i * NW + wave) * 8 + lane / 8;
    const int r = min(m0 + row, M - 1), c = ((lane % 8) ^ lds_swz<BK>(row)) * 8;
    const int g = a.rows_per_batch >= M ? 0 : r / a.rows_per_batch;
    aoff[i] = (uint32_t)(g * a.batch_stride + (int64_t)(r - g * a.rows_per_batch) * a.lda + c) * 2u;
  }
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int row = (i * NW + wave) * 8 + lane / 8;
    const int c = ((lane % 8) ^ lds_swz<BK>(row)) * 8;
    boff[i] = ((uint32_t)min(n0 + row, N - 1) * (uint32_t)K + (uint32_t)c) * 2u;
  }
  const int nk = K / BK;
  auto issue = [&](int t) {
    const uint32_t d = lds0 + (uint32_t)((t % S) * STAGE * 2 + wave * 1024);
#pragma unroll
    for (int i = 0; i < IA; ++i) lds_dma16_s(d + i * NW * 1024, aoff[i], abase + t * BK);
#pragma unroll
    for (int i = 0; i < IB; ++i) lds_dma16_s(d + BM * BK * 2 + i * NW * 1024, boff[i], w + t * BK);
  };
  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int lrow = lane & 31, sw = lds_swz<BK>(lrow), lh = lane >> 5;
  const bf16_t* a_frag = smem + (wm * TM + lrow) * BK;
  const bf16_t* b_frag = smem + BM * BK + (wn * TN + lrow) * BK;
  bf16x8 af[2][NS][FM], bfr[2][NS][FN];
  auto read = [&](int t, bf16x8 (&x)[NS][FM], bf16x8 (&y)[NS][FN]) {
    const int base = (t % S) * STAGE;
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
      const int off = base + (((kk * 2 + lh) ^ sw) * 8);
#pragma unroll
      for (int i = 0; i < FM; ++i) x[kk][i] = *(const bf16x8*)(a_frag + off + i * 32 * BK);
#pragma unroll
      for (int j = 0; j < FN; ++j) y[kk][j] = *(const bf16x8*)(b_frag + off + j * 32 * BK);
    }
  };
#pragma unroll
  for (int t = 0; t < S; ++t)
    if (t < nk) issue(t);
  wait_vm_lgkm0_rt<LPT*(S - 1)>(LPT * (min(S, nk) - 1));
  __builtin_amdgcn_s_barrier();
  read(0, af[0], bfr[0]);
  // While S more tiles follow: every MFMA is followed by its share of the next
  // tile's fragment reads (first) and of the direct loads, so the wave's one
  // instruction stream keeps the matrix, LDS and load pipes busy together.
  constexpr int NM = NS * FM * FN, NR = NS * (FM + FN);
  int t0 = 0;
  for (; t0 + 1 + S < nk; t0 += 2) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int t = t0 + p;
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      wait_vmcnt<LPT*(S - 2)>();
      __builtin_amdgcn_s_barrier();
      const int rb = ((t + 1) % S) * STAGE;
      const uint32_t dst = lds0 + (uint32_t)((t % S) * STAGE * 2 + wave * 1024);
      const bf16_t* an = abase + (t + S) * BK;
      const bf16_t* wn_ = w + (t + S) * BK;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        __builtin_amdgcn_sched_barrier(0);
        {
          const int kk = m / (FM * FN), i = m / FN % FM, j = m % FN;
          acc[i][j] = SW ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[p][kk][j], af[p][kk][i],
                                                                   acc[i][j], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[p][kk][i], bfr[p][kk][j],
                                                                   acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // reads over the first three quarters of the MFMAs, loads over all
#pragma unroll
        for (int q = 0; q < NR; ++q) {
          if (q * NM * 3 / (NR * 4) != m) continue;
          const int kk = q / (FM + FN), f = q % (FM + FN);
          const int off = rb + (((kk * 2 + lh) ^ sw) * 8);
          if (f < FM) af[p ^ 1][kk][f] = *(const bf16x8*)(a_frag + off + f * 32 * BK);
          else bfr[p ^ 1][kk][f - FM] = *(const bf16x8*)(b_frag + off + (f - FM) * 32 * BK);
        }
#pragma unroll
        for (int q = 0; q < LPT; ++q) {
          if (q * NM / LPT != m) continue;
          if (q < IA) lds_dma16_s(dst + q * NW * 1024, aoff[q], an);
          else lds_dma16_s(dst + BM * BK * 2 + (q - IA) * NW * 1024, boff[q - IA], wn_);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  for (; t0 < nk; t0 += 2) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int t = t0 + p;
      if (t < nk) {
        // this wave holds tile t (waited for on every path, so that the compiler
        // need not wait for tile t + 1's reads before the MFMAs); tile t + 1 has
        // landed once at most the tiles after it are pending; after the barrier
        // nobody reads tile t's slot
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        if (t + 1 < nk) {
          wait_vmcnt_rt<LPT*(S - 2)>(LPT * (min(S, nk - t) - 2));
          __builtin_amdgcn_s_barrier();
          if (t + S < nk) issue(t + S);
          read(t + 1, af[p ^ 1], bfr[p ^ 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < NS; ++kk)
#pragma unroll
          for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
              acc[i][j] = SW ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[p][kk][j], af[p][kk][i],
                                                                       acc[i][j], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[p][kk][i], bfr[p][kk][j],
                                                                       acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __syncthreads();                                 // the ring is free (every load has landed)
  if constexpr (SW) {
    if constexpr (KIND == EPI_QKV) {
      if (n0 >= 2 * e.d_model) {
        epi_direct_vt<FM, FN>(e, acc, (float*)smem + wave * 16 * kStageLd, m0 + wm * TM,
                              n0 + wn * TN, M, N, lane);
        return;
      }
    }
    epi_direct<KIND, FM, FN>(e, acc, m0 + wm * TM, n0 + wn * TN, M, N, lane);
  } else {
    epi_wave<KIND, FM, FN>(e, acc, (float*)smem + wave * (32 * kStageLd), m0 + wm * TM,
                           n0 + wn * TN, M, N, lane);
  }
}

// CUs the persistent GEMM leaves free (0 by default); set while a prefill
// runs beside decode work on another stream, so that work finds CUs.
static int g_ps_reserve = 0;
void gemm_set_cu_reserve(int n) { g_ps_reserve = n < 0 ? 0 : n; }

template <int BM, int BN, int BK, int WM, int WN, int S, int KIND, int OCC = 1, bool SW = false>
static void launch_gemm_ps(const AView& a, const bf16_t* w, int M, int N, int K,
                           const Epilogue& e, hipStream_t s, int gm) {
  constexpr size_t lds = (size_t)S * (BM + BN) * BK * sizeof(bf16_t) +
                        (SW && KIND != EPI_QKV ? 0 : (size_t)WM * WN * 16 * kStageLd * sizeof(float));
  auto kfn = k_gemm_bf16_ps<BM, BN, BK, WM, WN, S, KIND, SW>;
  static bool attr = false;
  static int n_cu = 0;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    int dev = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (n_cu <= 0) n_cu = 256;
    attr = true;
  }
  const int n_tm = (M + BM - 1) / BM, n_tn = (N + BN - 1) / BN;
  // keep the grid a multiple of 8 (one share per XCD) when CUs are reserved
  const int avail = g_ps_reserve > 0 ? std::max(8, (n_cu - g_ps_reserve) / 8 * 8) : n_cu;
  const int grid = std::min(n_tm * n_tn, OCC * avail);
  kfn<<<grid, WM * WN * 64, lds, s>>>(a, w, M, N, K, e, n_tm, n_tn, gm);
}

// The register epilogue stores 16-byte runs of eight columns through a
// buffer resource that spans the output (byte size below 2^31).
static bool direct_epi_ok(const Epilogue& e, int M, int N) {
  if (N % 8 != 0 || ((uintptr_t)e.out & 15) != 0) return false;
  if (e.kind == EPI_XKV) return e.d_model % 64 == 0 && e.slot_stride % 8 == 0;
  if (e.kind == EPI_QKV) {
    // tiles of up to 256 columns never mix q / k with V; V^T fits a buffer resource
    const int64_t vt_bytes = (int64_t)((M + kCtx - 1) / kCtx) * e.n_head * kHeadDim * kVtLd * 2;
    if (e.d_model % 128 != 0 || N != 3 * e.d_model || ((uintptr_t)e.out2 & 7) != 0 ||
        vt_bytes >= (int64_t)INT32_MAX)
      return false;
  }
  return e.ldc % 8 == 0 && e.ldc >= N && (int64_t)M * e.ldc * 2 < (int64_t)INT32_MAX;
}

// Operand extents that the persistent kernel's 32-bit byte offsets can
// address.
static bool fits_u32_offsets(const AView& a, int M, int N, int K) {
  const int64_t r = M - 1, g = r / a.rows_per_batch;
  const int64_t a_end = g * a.batch_stride + (r - g * a.rows_per_batch) * a.lda + K;
  return 2 * a_end < (int64_t)UINT32_MAX && 2 * (int64_t)N * K < (int64_t)UINT32_MAX;
}

template <int BM, int BN, int BK, int WM, int WN, int S, int KIND>
static void launch_gemm_pf(const AView& a, const bf16_t* w, int M, int N, int K,
                           const Epilogue& e, hipStream_t s, int gm) {
  constexpr size_t lds0 = (size_t)S * (BM + BN) * BK * sizeof(bf16_t);
  constexpr size_t lds_epi = (size_t)WM * WN * 32 * kStageLd * sizeof(float);
  constexpr size_t lds = lds0 > lds_epi ? lds0 : lds_epi;
  auto kfn = k_gemm_bf16_pf<BM, BN, BK, WM, WN, S, KIND>;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    attr = true;
  }
  int n_tm = (M + BM - 1) / BM, n_tn = (N + BN - 1) / BN;
  kfn<<<n_tm * n_tn, WM * WN * 64, lds, s>>>(a, w, M, N, K, e, n_tm, n_tn, gm);
}

template <int BM, int BN, int WM, int WN, int S, int KIND>
static void launch_gemm_rt(const AView& a, const bf16_t* w, int M, int N, int K,
                           const Epilogue& e, hipStream_t s, int gm) {
  constexpr size_t lds0 = (size_t)S * (BM + BN) * 64 * sizeof(bf16_t);
  constexpr size_t lds_epi = (size_t)WM * WN * 32 * kStageLd * sizeof(float);
  constexpr size_t lds = lds0 > lds_epi ? lds0 : lds_epi;
  static_assert(lds <= 160 * 1024, "LDS");
  auto kfn = k_gemm_bf16_rt<BM, BN, WM, WN, S, KIND>;
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)attr;
  const int n_tm = (M + BM - 1) / BM, n_tn = (N + BN - 1) / BN;
  kfn<<<n_tm * n_tn, WM * WN * 64, lds, s>>>(a, w, M, N, K, e, n_tm, n_tn, gm);
}

template <int BM, int BN, int BK, int WM, int WN, int S, int KIND>
static void launch_gemm_dma(const AView& a, const bf16_t* w, int M, int N, int K,
                            const Epilogue& e, hipStream_t s, int gm) {
  constexpr size_t lds0 = (size_t)S * (BM + BN) * BK * sizeof(bf16_t);
  constexpr size_t lds_epi = (size_t)WM * WN * 32 * kStageLd * sizeof(float);
  constexpr size_t lds = lds0 > lds_epi ? lds0 : lds_epi;
  auto kfn = k_gemm_bf16_dma<BM, BN, BK, WM, WN, S, KIND>;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    attr = true;
  }
  int n_tm = (M + BM - 1) / BM, n_tn = (N + BN - 1) / BN;
  kfn<<<n_tm * n_tn, WM * WN * 64, lds, s>>>(a, w, M, N, K, e, n_tm, n_tn, gm);
}

template <int BM, int BN, int BK, int WM, int WN, int KIND>
static void launch_gemm_cfg(const AView& a, const bf16_t* w, int M, int N, int K,
                            const Epilogue& e, hipStream_t s, int gm) {
  constexpr size_t lds0 = (size_t)2 * (BM + BN) * BK * sizeof(bf16_t);
  constexpr size_t lds_epi = (size_t)WM * WN * 32 * kStageLd * sizeof(float);
  constexpr size_t lds = lds0 > lds_epi ? lds0 : lds_epi;
  auto kfn = k_gemm_bf16<BM, BN, BK, WM, WN, KIND>;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    attr = true;
  }
  int n_tm = (M + BM - 1) / BM, n_tn = (N + BN - 1) / BN;
  kfn<<<n_tm * n_tn, WM * WN * 64, lds, s>>>(a, w, M, N, K, e, n_tm, n_tn, gm);
}

// Tile choice by shape (measured on MI355X with the encoder's products; M x N x
// K, us as here / as the other):
//  * K a multiple of 64 and at least two rounds of 256x256 tiles: persistent
//    256x256x64 kernel, 8 waves of 128x64 (24000 x 2304 x 768, 846 tiles: 112 /
//    about 137 in 128x128 tiles), except the first convolution, whose scatter
//    epilogue runs slower from the persistent kernel's half-block stage than
//    from the plain kernel's full-block one;
//  * fewer: 128x128 tiles, two blocks of two LDS stages a CU (4500 x 5120 x
//    1280: 77 / 83 in the unpipelined 256x128; 24000 x 768 x 3072: 136 / 159);
//    when they are at most one round, one block of four stages (6000 x 512 x
//    2048, 188 tiles: 17.6 / 24.6); when at most half a round, 128x64 tiles of
//    three stages (1500 x 1280 x 5120: 30 / 54, as 120 tiles of 128x128 37).
//    The sums are the same in all of these (one chain over K), so a clip's
//    result does not depend on how many clips share a product.
//  * K a multiple of 32 only (the first convolution of 32 or 96 filters): two
//    rounds of 256x128x32 tiles or more with three stages (96000 x 1280 x 288:
//    153 / 186 in 128x128x32, 24000 rows 47 / 55, 15000 rows, 590 tiles, 34.5 /
//    35.7), 128x128x32 with four stages below; K not even that (the 80-mel first
//    convolution): the register-path kernel, which zero-fills the K tail.
template <int KIND>
static void launch_gemm_bf16(const AView& a, const bf16_t* w, int M, int N, int K,
                             const Epilogue& e, hipStream_t s) {
  const int64_t t256x256 = (int64_t)((M + 255) / 256) * ((N + 255) / 256);
  const int64_t t256x128 = (int64_t)((M + 255) / 256) * ((N + 127) / 128);
  const int64_t t128x128 = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
  const bool direct = kDirectEpi<KIND> && direct_epi_ok(e, M, N);
  if (K % 32 != 0) {
    if (t256x128 >= 1024)
      launch_gemm_cfg<256, 128, 32, 4, 2, KIND>(a, w, M, N, K, e, s, 4);
    else
      launch_gemm_cfg<128, 128, 32, 2, 2, KIND>(a, w, M, N, K, e, s, 8);
  } else if (K % 64 == 0 && t256x256 >= 512) {
    // (the fused QKV product goes persistent only with its register epilogue)
    if (KIND != EPI_CONV1 && fits_u32_offsets(a, M, N, K) && (KIND != EPI_QKV || direct)) {
      const int gm = N >= 3072 ? 8 : 4;
      if constexpr (kDirectEpi<KIND>) {
        if (direct) {
          launch_gemm_ps<256, 256, 64, 2, 4, 2, KIND, 1, true>(a, w, M, N, K, e, s, gm);
          return;
        }
      }
      launch_gemm_ps<256, 256, 64, 2, 4, 2, KIND>(a, w, M, N, K, e, s, gm);
    } else
      launch_gemm_pf<256, 256, 64, 2, 4, 2, KIND>(a, w, M, N, K, e, s, 4);
  } else if (K % 64 == 0 && fits_u32_offsets(a, M, N, K) && (direct || !kDirectEpi<KIND>)) {
    if (t128x128 <= 128)
      launch_gemm_rt<128, 64, 2, 2, 3, KIND>(a, w, M, N, K, e, s, 8);
    else if (t128x128 <= 256)
      launch_gemm_rt<128, 128, 2, 2, 4, KIND>(a, w, M, N, K, e, s, 8);
    else
      launch_gemm_rt<128, 128, 2, 2, 2, KIND>(a, w, M, N, K, e, s, 8);
  } else if (KIND == EPI_CONV1 && t256x128 >= 512) {
    launch_gemm_pf<256, 128, 32, 4, 2, 3, KIND>(a, w, M, N, K, e, s, 4);
  } else {
    launch_gemm_dma<128, 128, 32, 2, 2, 4, KIND>(a, w, M, N, K, e, s, 8);
  }
}

void gemm_bf16(const AView& a, const bf16_t* w, int M, int N, int K, const Epilogue& e,
               hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  switch (e.kind) {
    case EPI_STORE: launch_gemm_bf16<EPI_STORE>(a, w, M, N, K, e, s); break;
    case EPI_GELU: launch_gemm_bf16<EPI_GELU>(a, w, M, N, K, e, s); break;
    case EPI_CONV1: launch_gemm_bf16<EPI_CONV1>(a, w, M, N, K, e, s); break;
    case EPI_CONV2: launch_gemm_bf16<EPI_CONV2>(a, w, M, N, K, e, s); break;
    case EPI_XKV: launch_gemm_bf16<EPI_XKV>(a, w, M, N, K, e, s); break;
    case EPI_QKV: launch_gemm_bf16<EPI_QKV>(a, w, M, N, K, e, s); break;
  }
}

// ---------------------------------------------------------------------------
// fp32 GEMM on v_mfma_f32_32x32x2_f32: bound by the fp32 matrix rate (148
// TFLOP/s for a large product) and, at one clip's sizes, by each block's start
// and end.  Four waves hold one 32x32 block of the output between them: K goes
// in chunks of 16 floats (16-byte pieces XOR-swizzled as in the bf16 kernels),
// chunk c belongs to wave c % 4, and the four chains are added as (0 + 1) +
// (2 + 3) at the end.  So even a product of 1500 x 384 puts several waves on
// every SIMD, and the sums of an element are the same in every tile shape:
// they do not depend on how many rows a product has.
// Measured (M x N x K): 1500 x 1536 x 384 30 us, 12000 x 1536 x 384 (as two
// halves beside each other) 164 us each; 42 us and about 1 ms as 64x64 tiles
// of scalar fp32.  32-float chunks 34 us (too few blocks a CU), a wave per
// output block with all four chains 35 us, operands read from global memory
// into registers without LDS 39 us.
// ---------------------------------------------------------------------------
constexpr int GF_KC = 16, GF_PR = GF_KC / 4;   // floats, 16-byte pieces a row

template <int KIND, int WM, int WN>
__global__ __launch_bounds__(WM* WN * 256) void k_gemm_f32(AView a, const float* __restrict__ w,
                                                           int M, int N, int K, Epilogue e,
                                                           int n_tm, int n_tn, int gm) {
  constexpr int NT = WM * WN * 256, BM = 32 * WM, BN = 32 * WN, ST = 4 * GF_KC;
  constexpr int PA = BM * 4 * GF_PR / NT, PB = BN * 4 * GF_PR / NT;   // pieces per thread
  static_assert(PA * NT == BM * 4 * GF_PR && PB * NT == BN * 4 * GF_PR, "tile/threads");
  extern __shared__ __attribute__((aligned(16))) float fsmem[];
  float (*As)[BM * ST] = (float (*)[BM * ST])fsmem;                   // [2 stages][4 chunks][BM][16]
  float (*Bs)[BN * ST] = (float (*)[BN * ST])(fsmem + 2 * BM * ST);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lh = lane >> 5;
  const int wk = wave & 3, wm = (wave >> 2) % WM, wn = (wave >> 2) / WM;
  int tm, tn;
  tile_of(blockIdx.x, n_tm * n_tn, n_tm, n_tn, gm, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  // piece p of a stage: row p / 16, chunk p / 4 % 4, 16 bytes p % 4
  const float* ap[PA];
  const float* bp[PB];
  int ao[PA], bo[PB], ak[PA], bk[PB];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int p = tid + i * NT, row = p / (4 * GF_PR), ck = p / GF_PR % 4, c = p % GF_PR;
    ak[i] = ck * GF_KC + c * 4;
    // (plain matrices skip the clip division)
    const int r = min(m0 + row, M - 1);
    ap[i] = (const float*)a.ptr + (a.rows_per_batch >= M ? r * a.lda : arow_offset(a, r)) + ak[i];
    ao[i] = (ck * BM + row) * GF_KC + ((c ^ lds_swz<2 * GF_KC>(row)) * 4);
  }
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int p = tid + i * NT, row = p / (4 * GF_PR), ck = p / GF_PR % 4, c = p % GF_PR;
    bk[i] = ck * GF_KC + c * 4;
    bp[i] = w + (int64_t)min(n0 + row, N - 1) * K + bk[i];
    bo[i] = (ck * BN + row) * GF_KC + ((c ^ lds_swz<2 * GF_KC>(row)) * 4);
  }
  f32x4 ra[PA], rb[PB];
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  auto load = [&](int k0) {
    if (k0 + ST <= K) {
#pragma unroll
      for (int i = 0; i < PA; ++i) ra[i] = *(const f32x4*)(ap[i] + k0);
#pragma unroll
      for (int i = 0; i < PB; ++i) rb[i] = *(const f32x4*)(bp[i] + k0);
    } else {                                       // K is a multiple of 4
#pragma unroll
      for (int i = 0; i < PA; ++i) ra[i] = k0 + ak[i] < K ? *(const f32x4*)(ap[i] + k0) : zero;
#pragma unroll
      for (int i = 0; i < PB; ++i) rb[i] = k0 + bk[i] < K ? *(const f32x4*)(bp[i] + k0) : zero;
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PA; ++i) *(f32x4*)&As[buf][ao[i]] = ra[i];
#pragma unroll
    for (int i = 0; i < PB; ++i) *(f32x4*)&Bs[buf][bo[i]] = rb[i];
  };
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const int sw = lds_swz<2 * GF_KC>(l32);
  const int arow = (wk * BM + wm * 32 + l32) * GF_KC, brow = (wk * BN + wn * 32 + l32) * GF_KC;
  const int nst = (K + ST - 1) / ST;
  load(0);
  store(0);
  __syncthreads();
  for (int t = 0; t < nst; ++t) {
    if (t + 1 < nst) load((t + 1) * ST);
    const float* as = As[t & 1] + arow;
    const float* bs = Bs[t & 1] + brow;
    f32x4 af[GF_KC / 8], bf[GF_KC / 8];
#pragma unroll
    for (int s = 0; s < GF_KC / 8; ++s) {
      const int c = ((2 * s + lh) ^ sw) * 4;
      af[s] = *(const f32x4*)(as + c);
      bf[s] = *(const f32x4*)(bs + c);
    }
#pragma unroll
    for (int s = 0; s < GF_KC / 8; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[s][q], bf[s][q], acc, 0, 0, 0);
    if (t + 1 < nst) store((t + 1) & 1);
    __syncthreads();
  }
  // the chains meet in LDS (the stages are free); a lane holds column l32
  // and, for register r, row 8 (r / 4) + 4 lh + r % 4 of the 32x32 block
  static_assert(2 * ST * (BM + BN) >= WM * WN * 4096, "reduction space");
  float* red = fsmem + (wn * WM + wm) * 4096;      // [4 chains][16][64]
#pragma unroll
  for (int r = 0; r < 16; ++r) red[(wk * 16 + r) * 64 + lane] = acc[r];
  __syncthreads();
  const int row0 = m0 + wm * 32 + 4 * lh + 8 * wk, col = n0 + wn * 32 + l32;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float* c = red + (wk * 4 + i) * 64 + lane;
    if (row0 + i < M && col < N)
      epi_apply<KIND, float>(e, row0 + i, col, (c[0] + c[1024]) + (c[2048] + c[3072]));
  }
}

template <int KIND, int WM, int WN>
static void launch_gemm_f32_cfg(const AView& a, const float* w, int M, int N, int K,
                                const Epilogue& e, hipStream_t s) {
  constexpr size_t lds = (size_t)2 * 4 * GF_KC * 32 * (WM + WN) * sizeof(float);
  static_assert(lds <= 64 * 1024, "LDS");
  const int n_tm = (M + 32 * WM - 1) / (32 * WM), n_tn = (N + 32 * WN - 1) / (32 * WN);
  k_gemm_f32<KIND, WM, WN><<<n_tm * n_tn, WM * WN * 256, lds, s>>>(a, w, M, N, K, e, n_tm, n_tn, 4);
}

// 64x64 tiles (16 waves) halve the operand traffic.  They take over from 577 of
// them on, past two rounds of one block a CU: 12000 x 1536 x 384 in halves 164 us
// against 190 in 32x32, 4500 rows of the same (1704 tiles; the encode of three
// tiny clips) 1672 against 1720; at 576 (1500 x 1536 x 384) the 32x32 ones still
// take 30.2 against 31.6.  Not where one 32-row tile holds all rows (the
// vocabulary product of a few decode rows): half of the tile would be padding, a
// tiny step of one row 235 us in 32x32 tiles, 245 in 64x64, of 32 rows 389 and
// 397; of 33 rows 415 and 410.
template <int KIND>
static void launch_gemm_f32(const AView& a, const float* w, int M, int N, int K,
                            const Epilogue& e, hipStream_t s) {
  if (M > 32 && (int64_t)((M + 63) / 64) * ((N + 63) / 64) > 576)
    launch_gemm_f32_cfg<KIND, 2, 2>(a, w, M, N, K, e, s);
  else
    launch_gemm_f32_cfg<KIND, 1, 1>(a, w, M, N, K, e, s);
}

void gemm_f32(const AView& a, const float* w, int M, int N, int K, const Epilogue& e,
              hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  switch (e.kind) {
    case EPI_STORE: launch_gemm_f32<EPI_STORE>(a, w, M, N, K, e, s); break;
    case EPI_GELU: launch_gemm_f32<EPI_GELU>(a, w, M, N, K, e, s); break;
    case EPI_CONV1: launch_gemm_f32<EPI_CONV1>(a, w, M, N, K, e, s); break;
    case EPI_CONV2: launch_gemm_f32<EPI_CONV2>(a, w, M, N, K, e, s); break;
    case EPI_XKV: launch_gemm_f32<EPI_XKV>(a, w, M, N, K, e, s); break;
  }
}

// ---------------------------------------------------------------------------
// Vocabulary projection (a skinny product)
// ---------------------------------------------------------------------------
// A decode step multiplies at most 128 rows by the token embedding once, so
// the product streams the table from HBM (128 flops per byte, far below the
// MFMA ridge) and the rows ride along from L2.  A block owns a strip of 32 WN
// table rows and all 128 row slots, in 64-deep chunks of K: each chunk's table
// tile and activation tile go global -> LDS with global_load_lds_dwordx4, eight
// lanes per 128-byte row segment (whole cache lines per instruction), with the
// round-robin XOR swizzle of the encoder GEMM (16-byte slot c of row r holds
// chunk c ^ ((r >> 1) & 7): conflict-free fragment reads).  The two operands
// have rings of their own, NW and NX chunks deep.  Wave w computes strip w % WN
// against 32 WN activation rows with v_mfma_f32_32x32x16_bf16: table rows are
// the "A" operand, activation rows the "B" operand.
constexpr int SK_BK = 64;          // K per chunk

__device__ __forceinline__ int sk_swz(int row) { return (row >> 1) & 7; }

// Larger key = larger value, then lower index.  Any NaN gets the largest
// value key so that it always wins and the finishing pass reports it.
__device__ __forceinline__ uint64_t argmax_key(float v, int n) {
  uint32_t o = (v != v) ? 0xffffffffu : ordered_u32(v);
  return ((uint64_t)o << 32) | (uint64_t)(0xffffffffu - (uint32_t)n);
}

struct SkOut {
  uint64_t* keys;       // [D][N / 32] best key per 32-row tile
  float* logits;        // optional float [D][N]
};

// Loads issued after chunk c's activation tile (which follows every earlier
// load in issue order): the prologue issues weight chunks 0 .. NW-2, then
// activation chunks 0 .. NX-2; iteration c' issues weight chunk c' + NW - 1,
// then activation chunk c' + NX - 1 (each only when it exists).
template <int NW, int NX>
__device__ __forceinline__ int sk_after(int c, int nck, int lpw, int lpx) {
  int n = 0;
  int first = c - NX + 2;                 // iterations that issued after X(c)
  if (c <= NX - 2) {
    n += lpx * max(0, min(NX - 2, nck - 1) - c);
    first = 0;
  }
  for (int i = first; i < c; ++i)
    n += (i + NW - 1 < nck ? lpw : 0) + (i + NX - 1 < nck ? lpx : 0);
  return n;
}

template <int WN, int NW, int NX>
__global__ __launch_bounds__(256) void k_skinny_bf16(const bf16_t* __restrict__ x,
                                                     const bf16_t* __restrict__ w, int D, int N,
                                                     int K, SkOut o) {
  constexpr int RB = WN;                         // row blocks of 32 per wave
  constexpr int WR = 32 * WN;                    // weight rows per block
  constexpr int WSTAGE = WR * SK_BK, XSTAGE = 128 * SK_BK;   // elements per ring stage
  constexpr int LPW = WN, LPX = 4;               // DMA instructions per wave per chunk
  constexpr int MAXOUT = (NW - 1) * LPW + (NX - 1) * LPX;
  static_assert(MAXOUT < 64, "vmcnt");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  bf16_t* wring = smem;
  bf16_t* xring = smem + NW * WSTAGE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, lh = lane >> 5;
  const int n0 = blockIdx.x * WR, nck = K / SK_BK;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) bf16_t*)smem);
  const uint32_t xlds0 = lds0 + (uint32_t)(NW * WSTAGE * 2);
  // DMA: instruction i of a wave fills rows 8 i .. 8 i + 7 of its share; lane
  // l lands at slot l % 8 of row l / 8 and fetches chunk (l % 8) ^ swz(row)
  uint32_t xdst[4], wdst[WN], xoff[4], woff[WN];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = wave * 32 + i * 8;                               // activation rows
    xdst[i] = __builtin_amdgcn_readfirstlane(xlds0 + (uint32_t)(row * SK_BK * 2));
    const int r = row + (lane >> 3);
    xoff[i] = (uint32_t)(((int64_t)min(r, D - 1) * K + (((lane & 7) ^ sk_swz(r)) * 8)) * 2);
  }
#pragma unroll
  for (int i = 0; i < WN; ++i) {
    const int row = wave * 8 * WN + i * 8;                           // weight rows
    wdst[i] = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(row * SK_BK * 2));
    const int r = row + (lane >> 3);
    woff[i] = (uint32_t)(((int64_t)min(n0 + r, N - 1) * K + (((lane & 7) ^ sk_swz(r)) * 8)) * 2);
  }
  auto issue_w = [&](int c) {
    const uint32_t so = (uint32_t)((c % NW) * WSTAGE * 2);
    const bf16_t* wk = w + c * SK_BK;
#pragma unroll
    for (int i = 0; i < WN; ++i) lds_dma16_s(wdst[i] + so, woff[i], wk);
  };
  auto issue_x = [&](int c) {
    const uint32_t so = (uint32_t)((c % NX) * XSTAGE * 2);
    const bf16_t* xk = x + c * SK_BK;
#pragma unroll
    for (int i = 0; i < 4; ++i) lds_dma16_s(xdst[i] + so, xoff[i], xk);
  };
  const int strip = wave % WN, rg = wave / WN;                      // this wave's strip, row group
  const int wrow = strip * 32 + l32, sww = sk_swz(wrow);
  int xrow[RB], swx[RB];
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    xrow[j] = (rg * RB + j) * 32 + l32;
    swx[j] = sk_swz(xrow[j]);
  }
  f32x16 acc[RB];
#pragma unroll
  for (int j = 0; j < RB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

  for (int c = 0; c < NW - 1 && c < nck; ++c) issue_w(c);
  for (int c = 0; c < NX - 1 && c < nck; ++c) issue_x(c);
  for (int c = 0; c < nck; ++c) {
    // this wave's tiles of chunk c have landed once at most the loads issued
    // after them are outstanding; the barrier then publishes every wave's
    // share and frees the stages of chunk c - 1 for the next issues
    wait_vmcnt_rt<MAXOUT>(sk_after<NW, NX>(c, nck, LPW, LPX));
    __builtin_amdgcn_s_barrier();
    if (c + NW - 1 < nck) issue_w(c + NW - 1);
    if (c + NX - 1 < nck) issue_x(c + NX - 1);
    const bf16_t* wt = wring + (c % NW) * WSTAGE;
    const bf16_t* xt = xring + (c % NX) * XSTAGE;
    bf16x8 wf[4], xf[4][RB];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int ch = kk * 2 + lh;
      wf[kk] = *(const bf16x8*)(wt + wrow * SK_BK + ((ch ^ sww) * 8));
#pragma unroll
      for (int j = 0; j < RB; ++j)
        xf[kk][j] = *(const bf16x8*)(xt + xrow[j] * SK_BK + ((ch ^ swx[j]) * 8));
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int j = 0; j < RB; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[kk], xf[kk][j], acc[j], 0, 0, 0);
  }
  // lane holds activation row xrow[j] and weight rows (output columns)
  // n0 + strip 32 + 8 (r / 4) + 4 (lane / 32) + r % 4
  const int nb = n0 + strip * 32;
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    const int row = xrow[j];
    uint64_t best = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int n = nb + (r >> 2) * 8 + lh * 4 + (r & 3);
      if (n < N) {
        const uint64_t kk = argmax_key(acc[j][r], n);
        best = kk > best ? kk : best;
        if (o.logits && row < D) o.logits[(int64_t)row * N + n] = acc[j][r];
      }
    }
    const uint32_t plo = __shfl_xor((uint32_t)best, 32, 64);
    const uint32_t phi = __shfl_xor((uint32_t)(best >> 32), 32, 64);
    const uint64_t other = ((uint64_t)phi << 32) | plo;
    best = other > best ? other : best;
    const int n_tiles = (N + 31) / 32;
    if (lane < 32 && row < D && nb < N) o.keys[(int64_t)row * n_tiles + nb / 32] = best;
  }
}

template <int WN, int NW, int NX>
static void launch_skinny(const bf16_t* x, const bf16_t* w, int D, int N, int K, const SkOut& o,
                          hipStream_t s) {
  constexpr size_t lds = ((size_t)NW * 32 * WN + (size_t)NX * 128) * SK_BK * sizeof(bf16_t);
  static_assert(lds <= 160 * 1024, "LDS");
  auto kfn = k_skinny_bf16<WN, NW, NX>;
  static bool attr = false;
  if (!attr) {
    (void)hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
    attr = true;
  }
  kfn<<<(N + 32 * WN - 1) / (32 * WN), 256, lds, s>>>(x, w, D, N, K, o);
}

// ---------------------------------------------------------------------------
// Vocabulary projection + argmax
// ---------------------------------------------------------------------------
int vocab_tiles(int V) { return (V + 31) / 32; }

// The vocabulary projection is the skinny product with 128 vocabulary rows per
// block (each wave one 32-row strip against all 128 row slots, so the
// activations are read once per 128 vocabulary rows); each wave leaves, for
// each decode row, the best key over its 32-row vocabulary tile.
void vocab_argmax_bf16(const bf16_t* x, const bf16_t* emb, int D, int V, int K, uint64_t* keys,
                       int n_tiles, float* logits, hipStream_t s) {
  if (D <= 0) return;
  (void)n_tiles;   // = vocab_tiles(V): the kernel derives it from V
  SkOut o{keys, logits};
  // 128 vocabulary rows per block with a 3-chunk weight and 2-chunk
  // activation ring (80 KB of LDS): two blocks per CU, so the 406 blocks of
  // the 51866-row table are all resident at once instead of running in a
  // full round and a partial one
  launch_skinny<4, 3, 2>(x, emb, D, V, K, o, s);
}

void vocab_logits_f32(const float* x, const float* emb, int D, int V, int K, float* logits,
                      hipStream_t s) {
  AView a{x, K, 0, 1 << 30};
  Epilogue e{};
  e.kind = EPI_STORE;
  e.out = logits;
  e.ldc = V;
  gemm_f32(a, emb, D, V, K, e, s);
}

__global__ __launch_bounds__(256) void k_logits_keys(const float* logits, int D, int V,
                                                     uint64_t* keys, int n_tiles) {
  const int tile = blockIdx.x * 8 + (threadIdx.x >> 5), b = blockIdx.y;
  const int n = tile * 32 + (threadIdx.x & 31);    // a half-wave per 32-entry tile
  uint64_t best = 0;
  if (n < V) best = argmax_key(logits[(int64_t)b * V + n], n);
  for (int o = 16; o > 0; o >>= 1) {
    uint32_t lo = __shfl_xor((uint32_t)best, o, 64), hi = __shfl_xor((uint32_t)(best >> 32), o, 64);
    uint64_t other = ((uint64_t)hi << 32) | lo;
    best = other > best ? other : best;
  }
  if ((threadIdx.x & 31) == 0 && tile < n_tiles) keys[(int64_t)b * n_tiles + tile] = best;
}
void logits_argmax_keys(const float* logits, int D, int V, uint64_t* keys, int n_tiles,
                        hipStream_t s) {
  if (D > 0) k_logits_keys<<<dim3((n_tiles + 7) / 8, D), 256, 0, s>>>(logits, D, V, keys, n_tiles);
}

// One block per row: the largest key of the row's tiles, whose index is the
// argmax; -1 - index where its logit is a NaN.  A latency chain, not a stream:
// eight keys a thread in flight take the 1621 tiles of a 51866-entry table in
// one pass (8.0 us with one wave, 3.9 with four).
__global__ __launch_bounds__(256) void k_argmax_finish(const uint64_t* keys, int n_tiles,
                                                       int32_t* out) {
  __shared__ uint64_t wave_best[4];
  const int b = blockIdx.x;
  uint64_t best = 0;
  for (int t = threadIdx.x; t < n_tiles; t += 256 * 8) {
    uint64_t k[8];                                 // (past the end: the last tile again)
#pragma unroll
    for (int i = 0; i < 8; ++i) k[i] = keys[(int64_t)b * n_tiles + min(t + 256 * i, n_tiles - 1)];
#pragma unroll
    for (int i = 0; i < 8; ++i) best = k[i] > best ? k[i] : best;
  }
  for (int o = 32; o > 0; o >>= 1) {
    uint32_t lo = __shfl_xor((uint32_t)best, o, 64), hi = __shfl_xor((uint32_t)(best >> 32), o, 64);
    uint64_t other = ((uint64_t)hi << 32) | lo;
    best = other > best ? other : best;
  }
  if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 1; i < 4; ++i) best = wave_best[i] > best ? wave_best[i] : best;
    const float v = from_ordered_u32((uint32_t)(best >> 32));
    const int32_t idx = (int32_t)(0xffffffffu - (uint32_t)best);
    out[b] = v != v ? -1 - idx : idx;
  }
}
void argmax_finish(const uint64_t* keys, int D, int n_tiles, int32_t* out, hipStream_t s) {
  if (D > 0) k_argmax_finish<<<D, 256, 0, s>>>(keys, n_tiles, out);
}

}  // namespace asr
