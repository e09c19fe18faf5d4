// Products of a decode step's rows: out[b] = epilogue(x[b] . W^T) for at most
// 128 rows b, bf16 and float32.
//
// Bound by reading the weights once (3 to 13 MB a product at d = 1280, 0.5 to
// 2 us at the rate of a plain read) and, for few rows, by the fixed time of a
// launch (about 3 us between dependent kernels): a product therefore takes its
// operand's preparation into its own start where that is short -- the LayerNorm
// of the residual stream, or the merge of the cross attention's key chunks --
// and its whole sum, bias and GELU or residual add into its end.
//
// The sum of an output element is fixed by K and S alone: the 128-byte chunks
// of K are dealt to S slices in turn (chunk c: slice c % S), each slice is one
// MFMA accumulation in ascending order, and the slices are added as a balanced
// tree.  Both kernels below do that, whatever blocks they use, so a row's
// result is the same whatever batch it is in.
#include "asr_device.h"

#include <algorithm>

namespace asr {

constexpr int RL_LW = 8;             // waves that prepare x, and the most rows that are prepared
constexpr int RL_RB = 32;            // decode rows of a block at most
constexpr size_t RL_LDS = 160 * 1024;

struct RowsArgs {
  const void* w;        // [N][K]
  const float* bias;    // [N]
  const void* x;        // RX_MEM: [D][K]; RX_LN: float h [D][K]; RX_MERGE: float records
  const float* g;       // RX_LN
  const float* beta;    // RX_LN
  void* out;            // RE_F32: float [D][N]; RE_GELU: T [D][N]; RE_RESID: float [D][N] (added to)
  int D, N, K;
  int rb;               // decode rows of a block
  int ring;             // chunks of a wave's ring
};

__device__ __forceinline__ int rl_swz(int row) { return (row >> 1) & 7; }

// Few rows: a block owns 8 WR8 weight rows and up to 32 decode rows, and wave s
// of S holds slice s.  Each wave sends its chunks global -> LDS
// (global_load_lds_dwordx4, eight lanes to a 128-byte row segment) into a ring
// of its own as soon as the block starts, so all of a block's weights are
// usually in flight before any arithmetic, and needs no barrier to use them: x
// comes either through the same ring or from LDS rows that RL_LW further waves
// prepare meanwhile (waves of their own, as waiting for the loads of the row
// would wait for the weights too).  The products are v_mfma_f32_32x32x16_bf16 /
// v_mfma_f32_32x32x2_f32 with the weight rows as first operand (repeated when
// there are fewer than 32); the slices meet in LDS.
// Measured at d = 1280 in the kernel trace of a graph-replayed step (us), as split-K
// partial sums, which a kernel of residual and LayerNorm (4.2 for one row, 4.8 for
// 128) or the attention added up, and now.  One row (the launch's fixed part is
// near 3): QKV 7.4, now 5.5 with its LayerNorm; out-projection 4.2, now 3.7; cross
// query 3.6, now 4.4 with its LayerNorm; FC1 11.7, now 7.2 with its LayerNorm; FC2
// 9.3, now 7.1.  128 rows: QKV 8.4, now 8.7; out-projection 5.2, 5.5; cross query
// 5.8, 5.2; FC1 12.1, 11.9; the LayerNorms apart 4.7 each.
template <typename T, int X, int EPI, int S, int WR8, int NV>
__global__ __launch_bounds__((S + (X == RX_MEM ? 0 : RL_LW)) * 64) void k_rows(RowsArgs a) {
  constexpr int ES = sizeof(T), WR = 8 * WR8;
  extern __shared__ __attribute__((aligned(16))) char rsm[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const int row0 = (int)blockIdx.y * a.rb, rows = min(a.rb, a.D - row0);
  const int n0 = (int)blockIdx.x * WR;
  const int kb = a.K * ES;                             // bytes of a row, a multiple of 128
  const int nx = X == RX_MEM ? (rows + 7) / 8 : 0;     // x instructions of a chunk
  const int slot = (WR8 + nx) * 1024;
  const int xld = kb + 16;                             // row stride of prepared x (conflict-free)
  char* xs = rsm + S * a.ring * slot;

  if (X != RX_MEM && wave >= S) {
    const int lw = wave - S;
    if constexpr (X == RX_LN) {
      if (lw < rows) {
        RowLN<NV> ln;
        ln.row((const float*)a.x + (int64_t)(row0 + lw) * a.K, a.K, lane);
        ln.params(a.g, a.beta, a.K, lane);
        ln.template write<T>((T*)(xs + lw * xld), a.K, lane);
      }
    } else {
      const int n_head = a.K / kHeadDim;
      for (int p = lw; p < rows * n_head; p += RL_LW) {
        const int r = p / n_head, h = p - r * n_head;
        const float v = cross_merge<T>((const float*)a.x, (int64_t)(row0 + r) * n_head + h, lane);
        St<T>::st((T*)(xs + r * xld), h * kHeadDim + lane, v);
      }
    }
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    __builtin_amdgcn_s_barrier();                      // x is ready
    __builtin_amdgcn_s_barrier();                      // (the sums)
    return;
  }

  const int nck = kb / 128, mine = (nck - wave + S - 1) / S;   // chunks wave, wave + S, ...
  char* ring = rsm + wave * a.ring * slot;
  const uint32_t lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)ring));
  const char* wb = (const char*)a.w + (int64_t)n0 * kb;
  const char* xb = (const char*)a.x + (int64_t)row0 * kb;
  // lane l of an instruction lands at slot l % 8 of row l / 8 and fetches the
  // piece that the swizzle puts there
  const int lr = lane >> 3;
  uint32_t woff[WR8];
#pragma unroll
  for (int j = 0; j < WR8; ++j) {
    const int r = 8 * j + lr;
    woff[j] = (uint32_t)(r * kb + (((lane & 7) ^ rl_swz(r)) * 16));
  }
  auto issue = [&](int i) {
    const uint32_t d = lds + (uint32_t)((i % a.ring) * slot);
    const int c = (wave + i * S) * 128;
#pragma unroll
    for (int j = 0; j < WR8; ++j) lds_dma16_s(d + j * 1024, woff[j], wb + c);
    if constexpr (X == RX_MEM) {
      for (int j = 0; j < nx; ++j) {
        const int r = 8 * j + lr;
        lds_dma16_s(d + (WR8 + j) * 1024,
                    (uint32_t)(min(r, rows - 1) * kb + (((lane & 7) ^ rl_swz(r)) * 16)), xb + c);
      }
    }
  };
  // the epilogue's operands, ahead of everything (one memory round trip less)
  const int n = n0 + 8 * wave + 4 * lh;
  const int64_t o = (int64_t)(row0 + l32) * a.N + n;
  const bool mine_out = wave < WR8 && l32 < rows;
  f32x4 old = {0.f, 0.f, 0.f, 0.f}, bias = old;
  if (mine_out) {
    bias = *(const f32x4*)(a.bias + n);
    if constexpr (EPI == RE_RESID) old = *(const f32x4*)((const float*)a.out + o);
  }
  const int ahead = min(a.ring, mine);
  for (int i = 0; i < ahead; ++i) issue(i);

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const int wrow = l32 & (WR - 1), sww = rl_swz(wrow);
  const int xrow = X == RX_MEM ? min(l32, nx * 8 - 1) : min(l32, rows - 1);
  const int swx = X == RX_MEM ? rl_swz(xrow) : 0;
  if constexpr (X != RX_MEM) __builtin_amdgcn_s_barrier();   // x is ready
  for (int i = 0; i < mine; ++i) {
    // chunk i has landed once at most the later ones are outstanding
    wait_vmcnt_rt<24>((min(mine, i + a.ring) - 1 - i) * (WR8 + nx));
    const char* wt = ring + (i % a.ring) * slot + wrow * 128;
    const char* xt = X == RX_MEM ? ring + (i % a.ring) * slot + WR8 * 1024 + xrow * 128
                                 : xs + xrow * xld + (wave + i * S) * 128;
    uint4 wf[4], xf[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      wf[s] = *(const uint4*)(wt + (((2 * s + lh) ^ sww) * 16));
      xf[s] = *(const uint4*)(xt + (((2 * s + lh) ^ swx) * 16));
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if constexpr (ES == 2) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[s]),
                                                      __builtin_bit_cast(bf16x8, xf[s]), acc, 0, 0, 0);
      } else {
        const f32x4 wv = __builtin_bit_cast(f32x4, wf[s]), xv = __builtin_bit_cast(f32x4, xf[s]);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[q], xv[q], acc, 0, 0, 0);
      }
    }
    if (i + a.ring < mine) {
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);          // the stage's reads are done
      issue(i + a.ring);
    }
  }
  // a lane holds decode row l32 and, in registers 4 j .. 4 j + 3, weight rows
  // 8 j + 4 lh .. + 3; the wave's sums go to the front of its own ring
#pragma unroll
  for (int j = 0; j < WR8; ++j)
    *(f32x4*)(ring + (j * 64 + lane) * 16) =
        f32x4{acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]};
  __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
  __builtin_amdgcn_s_barrier();
  if (!mine_out) return;
  f32x4 v = tree_sum<S>(0, [&](int s) {
    return *(const f32x4*)(rsm + s * a.ring * slot + (wave * 64 + lane) * 16);
  });
  v += bias;
  if constexpr (EPI == RE_GELU) {
    St<T>::st4((T*)a.out, o, make_float4(gelu_erf(v[0]), gelu_erf(v[1]), gelu_erf(v[2]), gelu_erf(v[3])));
  } else {
    if constexpr (EPI == RE_RESID) v += old;
    *(f32x4*)((float*)a.out + o) = v;
  }
}

// Decode rows of a block at most.
template <int X>
constexpr int kBlockRows = X == RX_MEM ? RL_RB : RL_LW;

template <typename T, int X, int EPI, int S, int WR8, int NV>
static void launch_rows(RowsArgs a, hipStream_t s) {
  const int kb = a.K * (int)sizeof(T);
  a.rb = std::min(a.D, kBlockRows<X>);
  // LDS: the prepared rows, and as many ring stages as a wave has chunks or fit
  constexpr int kWidest = 2048;                        // K of prepared rows at most
  static_assert((X == RX_MEM ? 0 : (size_t)RL_LW * (kWidest * sizeof(T) + 16)) +
                        (size_t)S * (WR8 + (X == RX_MEM ? RL_RB / 8 : 0)) * 1024 <= RL_LDS,
                "one ring stage fits");
  const size_t xbytes = X == RX_MEM ? 0 : (size_t)a.rb * (kb + 16);
  const size_t stage = (size_t)S * (WR8 + (X == RX_MEM ? (a.rb + 7) / 8 : 0)) * 1024;
  a.ring = (int)std::min<size_t>((kb / 128 + S - 1) / S, (RL_LDS - xbytes) / stage);
  auto kfn = k_rows<T, X, EPI, S, WR8, NV>;
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)RL_LDS);
  (void)attr;
  constexpr int NT = (S + (X == RX_MEM ? 0 : RL_LW)) * 64;
  kfn<<<dim3(a.N / (8 * WR8), (a.D + a.rb - 1) / a.rb), NT, xbytes + a.ring * stage, s>>>(a);
}

// Weight rows of a block: the fewest that keep the grid within one block a CU
// (FC1 of one row at d = 1280: 320 blocks of 16 rows 8.8 us, 160 of 32 7.6; QKV:
// 240 of 16 6.2 us, 120 of 32 7.2, 480 of 8 7.7).  The kernels lie in the code
// object in the order of these branches: the other way round, the same code, steps
// of 9 to 32 large-v3 rows took 0.5 % longer (3210 -> 3225 us).
template <typename T, int X, int EPI, int S, int NV = 1>
static void launch_rows_any(const RowsArgs& a, hipStream_t s) {
  const int ny = (a.D + kBlockRows<X> - 1) / kBlockRows<X>;
  if ((int64_t)(a.N / 16) * ny > 256) launch_rows<T, X, EPI, S, 4, NV>(a, s);
  else if ((int64_t)(a.N / 8) * ny > 256) launch_rows<T, X, EPI, S, 2, NV>(a, s);
  else launch_rows<T, X, EPI, S, 1, NV>(a, s);
}

// ---------------------------------------------------------------------------
// Many rows, bf16, long K (FC2): a block owns 32 weight rows and all 128 row
// slots (wave w rows 32 w .. 32 w + 31) over `ns` consecutive slices, so the
// weights are read once; per block of 32 rows, as above, K = 5120 would not fit
// LDS more than one chunk deep.  Chunks go through two LDS rings shared by the
// waves: the weights, which come cold from HBM, NW - 1 chunks ahead, x, an L2
// hit, NX - 1 ahead.  The time is that of a chain of chunks (load, barrier,
// read, MFMA), so two blocks a CU and short chains: N = 1280, K = 5120, 128 rows
// 11.7 us in 8 parts with 72 KB of LDS, 14.1 in 4 parts with 152 KB (9.9 in 5 parts
// that added their chunks in another order, so not the sums of a row alone).
// ---------------------------------------------------------------------------
struct WideArgs {
  const bf16_t* x;      // [D][K]
  const bf16_t* w;      // [N][K]
  float* out;           // [S / ns][D][N] partial sums
  int D, N, K;
  int S, ns;            // slices of the product, slices of a block
};
constexpr int RW_NW = 6, RW_NX = 3;        // 24 + 48 KB: two blocks a CU

// The chunks of slices [first, first + ns) in order.
struct ChunkWalk {
  int c, sl;
  __device__ __forceinline__ void next(int S, int nck) {
    c += S;
    if (c >= nck) c = ++sl;
  }
};

__global__ __launch_bounds__(256) void k_rows_wide(WideArgs a) {
  extern __shared__ __attribute__((aligned(16))) char rsm[];
  char* wring = rsm;                       // [NW][32 rows][128 B]
  char* xring = rsm + RW_NW * 4096;        // [NX][128 rows][128 B]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const int n0 = (int)blockIdx.x * 32, first = (int)blockIdx.y * a.ns;
  const int kb = a.K * 2, nck = kb / 128;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)rsm);
  // wave w fills weight rows 8 w .. 8 w + 7 and x rows 32 w .. 32 w + 31 of a
  // chunk; lane l lands at slot l % 8 of row l / 8 and fetches the piece that
  // the swizzle puts there
  const int lr = lane >> 3;
  const uint32_t wdst = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(wave * 1024));
  const uint32_t xdst = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(RW_NW * 4096 + wave * 4096));
  const char* wb = (const char*)a.w + (int64_t)n0 * kb;
  uint32_t woff, xoff[4];
  {
    const int r = wave * 8 + lr;
    woff = (uint32_t)(r * kb + (((lane & 7) ^ rl_swz(r)) * 16));
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = wave * 32 + j * 8 + lr;
    xoff[j] = (uint32_t)(min(r, a.D - 1) * kb + (((lane & 7) ^ rl_swz(r)) * 16));
  }
  int n = 0;                               // chunks of the block
  for (int s = first; s < first + a.ns; ++s) n += max(0, (nck - s + a.S - 1) / a.S);
  ChunkWalk ww{first, first}, wx{first, first};
  int iw = 0, ix = 0;
  auto issue_w = [&]() {
    lds_dma16_s(wdst + (uint32_t)((iw % RW_NW) * 4096), woff, wb + ww.c * 128);
    ww.next(a.S, nck);
    ++iw;
  };
  auto issue_x = [&]() {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      lds_dma16_s(xdst + (uint32_t)((ix % RW_NX) * 16384 + j * 1024), xoff[j],
                  (const char*)a.x + wx.c * 128);
    wx.next(a.S, nck);
    ++ix;
  };
  while (iw < RW_NW - 1 && iw < n) issue_w();
  while (ix < RW_NX - 1 && ix < n) issue_x();

  const int sw = rl_swz(l32);              // of weight row l32 and x row 32 w + l32
  f32x16 t0, t1, t2, t3, acc;              // tree levels: sums of 1, 2, 4, 8 slices
#pragma unroll
  for (int r = 0; r < 16; ++r) t0[r] = t1[r] = t2[r] = t3[r] = 0.f;
  int i = 0;
  for (int s = 0; s < a.ns; ++s) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    for (int c = first + s; c < nck; c += a.S, ++i) {
      // chunk number i has landed once at most the loads issued after its x
      // tile are outstanding: later x tiles, and the weight tiles past the
      // w_then that were issued by then (in the prologue, or up to and with
      // iteration i - NX + 1); the barrier then publishes every wave's share and frees
      // the stages of chunk i - 1 for the next issues
      const int w_then = i < RW_NX - 1 ? min(RW_NW - 1, n) : min(n, RW_NW + i - RW_NX + 1);
      wait_vmcnt_rt<(RW_NW - 1) + 4 * (RW_NX - 1)>(4 * (ix - 1 - i) + iw - w_then);
      __builtin_amdgcn_s_barrier();
      if (iw < n) issue_w();
      if (ix < n) issue_x();
      const char* wt = wring + (i % RW_NW) * 4096 + l32 * 128;
      const char* xt = xring + (i % RW_NX) * 16384 + (wave * 32 + l32) * 128;
      bf16x8 wf[4], xf[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int off = ((2 * q + lh) ^ sw) * 16;
        wf[q] = *(const bf16x8*)(wt + off);
        xf[q] = *(const bf16x8*)(xt + off);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q], xf[q], acc, 0, 0, 0);
    }
    // slice s joins the tree: it completes the pairs that its trailing one
    // bits stand for (ns <= 16)
    if (s & 1) {
      acc = t0 + acc;
      if (s & 2) {
        acc = t1 + acc;
        if (s & 4) {
          acc = t2 + acc;
          if (s & 8) acc = t3 + acc;
          else t3 = acc;
        } else {
          t2 = acc;
        }
      } else {
        t1 = acc;
      }
    } else {
      t0 = acc;
    }
  }
  const int row = wave * 32 + l32;
  if (row >= a.D) return;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int col = n0 + 8 * j + 4 * lh;
    *(f32x4*)(a.out + ((int64_t)blockIdx.y * a.D + row) * a.N + col) =
        f32x4{acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]};
  }
}

static void launch_wide(const WideArgs& a, hipStream_t s) {
  constexpr int lds = RW_NW * 4096 + RW_NX * 16384;
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)k_rows_wide, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  (void)attr;
  k_rows_wide<<<dim3(a.N / 32, a.S / a.ns), 256, lds, s>>>(a);
}

// h[b] += bias + the tree of the partial sums of row b, xn[b] = LayerNorm(h[b]):
// one block a row.
constexpr int RW_SPLITS = 8;
__global__ __launch_bounds__(256) void k_rows_reduce_norm(const float* __restrict__ part, int D,
                                                          int d, const float* __restrict__ bias,
                                                          float* __restrict__ h,
                                                          const float* __restrict__ g,
                                                          const float* __restrict__ beta,
                                                          bf16_t* __restrict__ xn) {
  __shared__ __attribute__((aligned(16))) float row[2048];
  const int b = blockIdx.x, tid = threadIdx.x;
  RowLN<8> ln;
  if (tid < 64) ln.params(g, beta, d, tid);
  for (int e = tid * 4; e < d; e += 1024) {
    const int64_t o = (int64_t)b * d + e;
    f32x4 v = tree_sum<RW_SPLITS>(
        0, [&](int s) { return *(const f32x4*)(part + (int64_t)s * D * d + o); });
    v += *(const f32x4*)(bias + e);
    v += *(const f32x4*)(h + o);
    *(f32x4*)(h + o) = v;
    *(f32x4*)(row + e) = v;
  }
  __syncthreads();
  if (tid >= 64) return;
  ln.row(row, d, tid);
  ln.write<bf16_t>(xn + (int64_t)b * d, d, tid);
}

// ---------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------
// Slices: 8 for K = d, 16 for the longer K of FC2 (a property of the product,
// never of the batch).
static int slices(int N, int K) { return K > N ? 16 : 8; }

template <typename T>
void rows_ln(const float* h, const float* g, const float* beta, const T* w, const float* bias, int D,
             int N, int K, bool gelu, void* out, hipStream_t s) {
  if (D <= 0) return;
  RowsArgs a{w, bias, h, g, beta, out, D, N, K, 0, 0};
  if (gelu) {
    if (K <= 1280) launch_rows_any<T, RX_LN, RE_GELU, 8, 5>(a, s);
    else launch_rows_any<T, RX_LN, RE_GELU, 8, 8>(a, s);
  } else {
    if (K <= 1280) launch_rows_any<T, RX_LN, RE_F32, 8, 5>(a, s);
    else launch_rows_any<T, RX_LN, RE_F32, 8, 8>(a, s);
  }
}
template <typename T>
void rows_mem(const T* x, const T* w, const float* bias, int D, int N, int K, bool gelu, void* out,
             hipStream_t s) {
  if (D <= 0) return;
  RowsArgs a{w, bias, x, nullptr, nullptr, out, D, N, K, 0, 0};
  if (gelu) launch_rows_any<T, RX_MEM, RE_GELU, 8>(a, s);
  else launch_rows_any<T, RX_MEM, RE_F32, 8>(a, s);
}
template <typename T>
void rows_resid(const T* x, const T* w, const float* bias, int D, int N, int K, float* h,
                hipStream_t s) {
  if (D <= 0) return;
  RowsArgs a{w, bias, x, nullptr, nullptr, h, D, N, K, 0, 0};
  if (slices(N, K) == 16) launch_rows_any<T, RX_MEM, RE_RESID, 16>(a, s);
  else launch_rows_any<T, RX_MEM, RE_RESID, 8>(a, s);
}
template <typename T>
void rows_merge_resid(const float* rec, const T* w, const float* bias, int D, int d, float* h,
                      hipStream_t s) {
  if (D <= 0) return;
  RowsArgs a{w, bias, rec, nullptr, nullptr, h, D, d, d, 0, 0};
  launch_rows_any<T, RX_MERGE, RE_RESID, 8>(a, s);
}

// The LayerNorm alone, one wave a row.
template <typename T>
__global__ __launch_bounds__(64) void k_rows_norm(const float* __restrict__ h, int d,
                                                  const float* __restrict__ g,
                                                  const float* __restrict__ beta,
                                                  T* __restrict__ out) {
  RowLN<8> ln;
  const int64_t o = (int64_t)blockIdx.x * d;
  ln.row(h + o, d, threadIdx.x);
  ln.params(g, beta, d, threadIdx.x);
  ln.template write<T>(out + o, d, threadIdx.x);
}
template <typename T>
void rows_norm(const float* h, int D, int d, const float* g, const float* beta, T* out,
               hipStream_t s) {
  if (D > 0) k_rows_norm<T><<<D, 64, 0, s>>>(h, d, g, beta, out);
}

void rows_resid_norm(const bf16_t* x, const bf16_t* w, const float* bias, int D, int d, int K,
                     float* h, const float* g, const float* beta, bf16_t* xn, float* part,
                     hipStream_t s) {
  if (D <= 0) return;
  const int S = slices(d, K);
  launch_wide(WideArgs{x, w, part, D, d, K, S, S / RW_SPLITS}, s);
  k_rows_reduce_norm<<<D, 256, 0, s>>>(part, D, d, bias, h, g, beta, xn);
}
size_t rows_part_floats(int D, int d) { return (size_t)RW_SPLITS * D * d; }

#define ROWS_INST(T)                                                                              \
  template void rows_ln<T>(const float*, const float*, const float*, const T*, const float*, int, \
                           int, int, bool, void*, hipStream_t);                                   \
  template void rows_mem<T>(const T*, const T*, const float*, int, int, int, bool, void*,         \
                            hipStream_t);                                                         \
  template void rows_resid<T>(const T*, const T*, const float*, int, int, int, float*,            \
                              hipStream_t);                                                       \
  template void rows_merge_resid<T>(const float*, const T*, const float*, int, int, float*,       \
                                    hipStream_t);                                                 \
  template void rows_norm<T>(const float*, int, int, const float*, const float*, T*, hipStream_t);
ROWS_INST(float)
ROWS_INST(bf16_t)
#undef ROWS_INST

}  // namespace asr
