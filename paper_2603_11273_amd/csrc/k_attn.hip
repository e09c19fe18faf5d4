// Attention kernels.
//
//  * flash_attn_bf16: encoder self-attention over the 1500 positions of a
//    30-s segment (no mask), MFMA-based.  Each wave owns 32 queries; K and
//    V^T tiles of 64 keys are staged in LDS and shared by the block's
//    waves.  The kernel computes S^T = K Q^T so that, in the MFMA output
//    layout, each lane holds one query's scores for 32 keys: the row max
//    needs a single cross-lane exchange, the probabilities feed the
//    O^T = V^T P^T product directly as its B operand, and the per-query
//    rescale is a per-lane multiply.  Softmax runs in fp32 with exp2.
//  * flash_attn_f32: the same result in fp32 MFMA, keys split over a block's waves.
//  * decode self attention: one block per (row, head) over the row's cached keys
//    in parts joined by an online softmax; this step's key and value go into
//    the cache at the slot's position.
//  * decode cross attention: one block per (row, head, chunk of the 1500 keys),
//    each leaving a record (max, sum, weighted values) that is merged later.
#include "asr_device.h"

#include <algorithm>

namespace asr {

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 u) {
  bf16x8 r;
  __builtin_memcpy(&r, &u, 16);
  return r;
}

// ---------------------------------------------------------------------------
// Encoder flash attention (bf16)
//
// Block = NW (8 or 4) waves x 32 queries of one (clip, head); tiles of 64 keys.
// K comes from the fused QKV buffer, V from the per-head transposed copy the
// QKV GEMM writes (V^T[dim][position], zero past 1500).  S^T = K Q^T is
// computed per 32-key x 32-query block, so in the MFMA output layout a lane
// owns one query: the row max needs one cross-lane exchange (lane ^ 32) and
// the online-softmax rescale is per lane.
//  * The K rows of each 32-key block enter the MFMA in the order that swaps
//    bits 2 and 3 of the row index.  A lane then holds its query's scores
//    for 8 consecutive keys per 16-key group, which, packed to bf16, are
//    directly the B operand of O^T += V^T P^T; the matching A operand is one
//    16-byte chunk of a V^T row.  Both tiles are plain [row][64] bf16 tiles
//    with 16-byte chunks XOR-swizzled by (row / 2) % 8 (conflict-free
//    fragment reads), double-buffered in LDS and filled by direct
//    global-to-LDS loads (8 / NW 1 KB instructions per wave per operand): tile
//    kt+1 is in flight while tile kt is consumed, one barrier per tile.
//  * The probability sum uses v_dot2 on the packed bf16 probabilities (the
//    same rounded values the P V product uses), two per instruction.
//  * Q arrives scaled by 1/sqrt(64) log2(e) (the QKV epilogue folds the
//    factor in before its one bf16 rounding), so scores are in the exp2
//    domain; softmax in fp32 with exp2 and a lazy reference (below).
// The kernel keeps to 128 VGPRs (four waves per SIMD, two blocks per CU):
// the exp2 work on the VALU and the MFMAs of other waves then overlap.
// ---------------------------------------------------------------------------
constexpr int FP_KT = 64;

__device__ __forceinline__ void fp_dma16(uint32_t lds_addr, uint32_t voff, const void* sbase) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void fp_wait_vmcnt() {
  static_assert(N >= 0 && N < 16, "vmcnt");
  __builtin_amdgcn_s_waitcnt(N | (0x7 << 4) | (0xF << 8));
}
// row index of the K tile that feeds MFMA row i (bits 2 and 3 swapped)
__device__ __forceinline__ int fp_perm(int i) {
  return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1);
}

template <int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(4)))
void k_flash_bf16(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ vt,
                       bf16_t* __restrict__ out, int n_head) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  constexpr int S = 2;                             // LDS stages
  __shared__ __attribute__((aligned(16))) bf16_t Ks[S][FP_KT * 64];   // [key][dim]
  __shared__ __attribute__((aligned(16))) bf16_t Vs[S][64 * FP_KT];   // [dim][key]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // XCD-aware work order: the hardware deals blocks round-robin to the 8
  // XCDs in dispatch order (x fastest), so block i runs on XCD i % 8.  Each
  // XCD takes a contiguous range of (query block, head, clip) work items,
  // query block fastest, so the query blocks of one (clip, head) share an
  // L2 and its K and V^T tiles are fetched from beyond it about once.
  int qb, h, b;
  {
    const int nqb = gridDim.x, nh = gridDim.y;
    const int total = nqb * nh * (int)gridDim.z;
    const int lin = (int)blockIdx.x + nqb * ((int)blockIdx.y + nh * (int)blockIdx.z);
    const int per = total / 8, rem = total % 8, xcd = lin % 8;
    const int w = xcd * per + min(xcd, rem) + lin / 8;
    qb = w % nqb;
    h = (w / nqb) % nh;
    b = w / (nqb * nh);
  }
  const int d = n_head * 64, ld3 = 3 * d;
  const bf16_t* base = qkv + (int64_t)b * kCtx * ld3;
  const int half = lane >> 5, l32 = lane & 31;
  const int q = qb * (NW * 32) + wave * 32 + l32;   // this lane's query
  constexpr int NT = (kCtx + FP_KT - 1) / FP_KT;

  // Q fragments (B operand of S^T): dims kk*16 + half*8 .. +8 of query q
  bf16x8 qf[4];
  {
    const bf16_t* qp = base + (int64_t)(q < kCtx ? q : 0) * ld3 + h * 64 + half * 8;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      uint4 v = {0u, 0u, 0u, 0u};
      if (q < kCtx) v = *(const uint4*)(qp + kk * 16);
      qf[kk] = as_bf16x8(v);
    }
  }

  // Direct loads: wave w fills rows 8w .. 8w+7 of both tiles (and, of four waves,
  // rows 32 + 8w .. as well); lane l lands 16 bytes at slot l % 8 of row 8w + l / 8
  // and fetches the chunk that the swizzle (the same 32 rows on) puts there.  K
  // rows past position 1499 re-read row 1499 (their scores are masked); V^T rows
  // are padded to kVtLd >= 64 NT positions.
  const int lrow = wave * 8 + (lane >> 3);
  const int lch = (lane & 7) ^ ((lrow >> 1) & 7);
  const uint32_t k_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)&Ks[0][0] + (uint32_t)(wave * 1024));
  const uint32_t v_lds = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)&Vs[0][0] + (uint32_t)(wave * 1024));
  const bf16_t* kbase = base + d + h * 64;                          // K columns of head h
  const bf16_t* vbase = vt + ((int64_t)b * n_head + h) * 64 * kVtLd;
  const uint32_t v_off = (uint32_t)((lrow * kVtLd + lch * 8) * 2);
  auto issue = [&](int t) {
    const int k0 = t * FP_KT;
    const uint32_t so = (uint32_t)((t % S) * FP_KT * 64 * 2);
#pragma unroll
    for (int r = 0; r < FP_KT; r += 8 * NW) {
      const int key = min(k0 + r + lrow, kCtx - 1);
      fp_dma16(k_lds + so + r * 128, (uint32_t)((key * ld3 + lch * 8) * 2), kbase);
      fp_dma16(v_lds + so + r * 128, v_off + (uint32_t)(r * kVtLd * 2), vbase + k0);
    }
  };

  // fragment read offsets (elements) within a stage
  const int sw = (l32 >> 1) & 7;                       // swizzle of rows l32 and 32 + l32
  int koff[2][4];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const int row = kb * 32 + fp_perm(l32);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) koff[kb][kk] = row * 64 + (((kk * 2 + half) ^ ((row >> 1) & 7)) * 8);
  }

  f32x16 zero16;
#pragma unroll
  for (int r = 0; r < 16; ++r) zero16[r] = 0.f;
  // scores of tile t: four K fragments in flight per 32-key block
  auto scores = [&](int t, f32x16 (&s)[2]) {
    const bf16_t* Kc = Ks[t % S];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      bf16x8 kf[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) kf[kk] = *(const bf16x8*)(Kc + koff[kb][kk]);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk],
                                                        kk == 0 ? zero16 : s[kb], 0, 0, 0);
    }
  };

  f32x16 o0, o1;                                   // O^T dims 0..31, 32..63
#pragma unroll
  for (int r = 0; r < 16; ++r) o0[r] = o1[r] = 0.f;
  float m = 0.f, l = 0.f;
  bool zref = true;                                // every lane of the wave has m == 0
  const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3F803F80u);

  // softmax of tile t's scores (in s) and its P V product
  // (the rare branches carry an empty volatile asm so that the compiler
  // keeps them as branches instead of executing them on every tile)
  auto consume = [&](int t, f32x16 (&s)[2]) {
    const int k0 = t * FP_KT;
    // V fragments: chunk kb*4 + hf*2 + half of V^T rows l32 and 32 + l32
    const bf16_t* Vc = Vs[t % S];
    auto vfrag = [&](int kb, int hf, int row) {
      return *(const bf16x8*)(Vc + row * 64 + (((kb * 4 + hf * 2 + half) ^ sw) * 8));
    };
    if (!zref) {                                   // wave-uniform: some lane's m moved
      asm volatile("");
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] -= m;
    }
    if (k0 + FP_KT > kCtx) {                       // last tile: keys past 1500 do not exist
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = k0 + kb * 32 + (r >> 3) * 16 + half * 8 + (r & 7);
          if (key >= kCtx) s[kb][r] = -INFINITY;
        }
    }
    // probabilities of the tile against the current reference, packed to
    // bf16 (the P V product's B operand), and their sum
    uint32_t u[2][2][4];
    float lt = 0.f;
    auto probs = [&]() {
      float ls[4] = {0.f, 0.f, 0.f, 0.f};          // four independent sum chains
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // keys kb*32 + hf*16 + half*8 + 2i, +1: registers hf*8 + 2i, +1
            u[kb][hf][i] = pack2_bf16(__builtin_amdgcn_exp2f(s[kb][hf * 8 + 2 * i]),
                                      __builtin_amdgcn_exp2f(s[kb][hf * 8 + 2 * i + 1]));
            ls[i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u[kb][hf][i]),
                                                    ones, ls[i], false);
          }
      lt = (ls[0] + ls[1]) + (ls[2] + ls[3]);
    };
    probs();
    // Lazy reference: probabilities are exp2(s - m) with m = 0 as long as
    // every score of the wave stays within 2^6 of it, so the common case
    // needs no subtraction at all.  exp2(s - m) may then reach 2^64, which
    // fp32 sums and bf16 operands carry with unchanged relative precision
    // (both reach 2^127); the final 1/l cancels the offset.  The common case
    // does not look for the tile's maximum either: a score more than 2^6
    // above m (or +inf) makes its lane's probability sum exceed 2^64, and on
    // the first tile a lane whose scores all lie far below 0 sums to less
    // than 2^-64.  Only such tiles take the exact maximum: a first tile whose
    // maximum lies outside [-64, 64] sets m to it; a later maximum more than
    // 2^6 above m moves m up and rescales O and l; the tile's probabilities
    // are then recomputed.
    if (__any(lt > 0x1p64f) || (t == 0 && __any(lt < 0x1p-64f))) {
      asm volatile("");
      float tmax = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[kb][r]);
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      if (t == 0) {
        if (__any(fabsf(tmax) > 64.0f)) {          // 64 real keys: finite
          m = tmax;
          zref = false;
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kb][r] -= tmax;
        }
      } else if (__any(tmax > 64.0f)) {
        const float shift = fmaxf(tmax, 0.f);
        const float alpha = __builtin_amdgcn_exp2f(-shift);
        m += shift;
        zref = false;
        l *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          o0[r] *= alpha;
          o1[r] *= alpha;
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) s[kb][r] -= shift;
      }
      probs();
    }
    l += lt;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const bf16x8 pb = as_bf16x8(uint4{u[kb][hf][0], u[kb][hf][1], u[kb][hf][2], u[kb][hf][3]});
        o0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfrag(kb, hf, l32), pb, o0, 0, 0, 0);
        o1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfrag(kb, hf, 32 + l32), pb, o1, 0, 0, 0);
      }
  };

  // tile t+1 loads while tile t is consumed
  f32x16 sc[2];
  issue(0);
  for (int t = 0; t < NT; ++t) {
    fp_wait_vmcnt<0>();                            // tile t landed
    __syncthreads();                               // ... for every wave; tile t-1's stage free
    if (t + 1 < NT) issue(t + 1);
    scores(t, sc);
    consume(t, sc);
  }
  l += __shfl_xor(l, 32, 64);
  if (q >= kCtx) return;
  const float inv = 1.0f / l;
  bf16_t* op = out + ((int64_t)b * kCtx + q) * d + h * 64;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int d0 = g * 8 + half * 4;
    uint2 w0 = {pack2_bf16(o0[g * 4 + 0] * inv, o0[g * 4 + 1] * inv),
                pack2_bf16(o0[g * 4 + 2] * inv, o0[g * 4 + 3] * inv)};
    uint2 w1 = {pack2_bf16(o1[g * 4 + 0] * inv, o1[g * 4 + 1] * inv),
                pack2_bf16(o1[g * 4 + 2] * inv, o1[g * 4 + 3] * inv)};
    *(uint2*)(op + d0) = w0;
    *(uint2*)(op + 32 + d0) = w1;
  }
}

template <int NW>
static void launch_flash(const bf16_t* qkv, const bf16_t* vt, bf16_t* out, int B, int n_head,
                         hipStream_t s) {
  dim3 grid((kCtx + NW * 32 - 1) / (NW * 32), n_head, B);
  k_flash_bf16<NW><<<grid, NW * 64, 0, s>>>(qkv, vt, out, n_head);
}

// Waves of a block: four while the eight-wave blocks of all clips in flight (the
// groups of a batch run beside each other) would leave half of the 256 CUs idle,
// as 4-wave blocks then still have a CU each: encode of one large-v3 clip, 120
// blocks of eight waves, 4668 us, 240 of four 4459 (one small clip 1252, 1170; two
// base clips beside each other 735, 722).  With more they share CUs and
// fetch K and V twice as often: seven base clips (336 blocks) 1500 us with
// eight waves, 1550 with four; 32 small ones 17124, 17321.  A wave's work is the
// same in both, and so are the results.
void flash_attn_bf16(const bf16_t* qkv, const bf16_t* vt, bf16_t* out, int B, int n_head,
                     int clips_in_flight, hipStream_t s) {
  if (B <= 0) return;
  static_assert(kVtLd >= FP_KT * ((kCtx + FP_KT - 1) / FP_KT), "V^T rows cover every tile");
  if ((int64_t)((kCtx + 255) / 256) * n_head * std::max(B, clips_in_flight) <= 128)
    launch_flash<4>(qkv, vt, out, B, n_head, s);
  else
    launch_flash<8>(qkv, vt, out, B, n_head, s);
}

// Lays given q / k / v ([B*1500][d] float32) out as the encoder attention
// kernels read them: which = 0, 1 -> columns 0..d-1, d..2d-1 of qkv (q times
// qmul); which = 2 -> columns 2d..3d-1 (fp32), or V^T [b][h][dim][kVtLd]
// (bf16).
template <typename T>
__global__ void k_pack_attn_operand(const float* __restrict__ src, int which, int rows, int d,
                                    int n_head, float qmul, T* __restrict__ qkv,
                                    T* __restrict__ vt) {
  const int64_t n = (int64_t)rows * d;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / d;
    const int c = (int)(i - r * d);
    const float x = which == 0 ? src[i] * qmul : src[i];
    if (which < 2 || vt == nullptr) {
      St<T>::st(qkv, r * 3 * d + which * d + c, x);
    } else {
      const int64_t g = r / kCtx, t = r - g * kCtx;
      St<T>::st(vt, ((g * n_head + (c >> 6)) * kHeadDim + (c & 63)) * kVtLd + t, x);
    }
  }
}
template <typename T>
void pack_attn_operand(const float* src, int which, int rows, int d, int n_head, float qmul,
                       T* qkv, T* vt, hipStream_t s) {
  const int64_t n = (int64_t)rows * d;
  if (n <= 0) return;
  const int grid = (int)std::min<int64_t>((n + 255) / 256, 65536);
  k_pack_attn_operand<T><<<grid, 256, 0, s>>>(src, which, rows, d, n_head, qmul, qkv, vt);
}
template void pack_attn_operand<float>(const float*, int, int, int, int, float, float*, float*,
                                       hipStream_t);
template void pack_attn_operand<bf16_t>(const float*, int, int, int, int, float, bf16_t*,
                                        bf16_t*, hipStream_t);

// ---------------------------------------------------------------------------
// Encoder attention, fp32, on v_mfma_f32_16x16x4_f32
//
// Bound by the fp32 matrix rate (4 * 1500^2 * 64 flops a head: 23 us for the
// six heads of one clip at 148 TFLOP/s).  A block owns 16 NB queries of one
// (clip, head); its 8 waves take the 16-key tiles in turn (tile t goes to
// wave t % 8) and keep an online softmax of their own, merged through LDS at
// the end, so one clip's few query blocks still put two waves on every SIMD
// (one wave's exp2 and rescale run beside the other's MFMAs) and no barrier
// sits in the key loop.
//  * S^T = K Q^T: a lane's K operand is 16 bytes of one key's row and feeds
//    four MFMAs, so K goes from the QKV buffer straight to registers.
//  * In the MFMA output layout a lane holds one query's scores of keys
//    4 (lane / 16) + r, which is the B operand of O^T += V^T P^T for MFMA r;
//    the A operand is V[key][4 (lane % 16) + j] for dim component j: one
//    coalesced 16-byte load of a key's row feeds the four j.
//  * The query carries 1/sqrt(64) log2(e), so softmax works with exp2.
// Nothing a query's result is made of depends on NB, which the launcher
// picks so that the last round of blocks is not nearly empty.
// One clip of 6 heads: 50 us a layer, 1146 us as one thread per query.
// ---------------------------------------------------------------------------
constexpr int FF_NW = 8;
constexpr int FF_LD = 68;      // floats per merged query row in LDS (64 + pad)

template <int NB>
__global__ __launch_bounds__(FF_NW * 64) void k_flash_f32(const float* __restrict__ qkv,
                                                          float* __restrict__ out, int n_head) {
  constexpr int QT = 16 * NB, NT = (kCtx + 15) / 16;
  extern __shared__ __attribute__((aligned(16))) float fsm[];
  float* osh = fsm;                                // [FF_NW][QT][FF_LD]
  float2* mlsh = (float2*)(fsm + FF_NW * QT * FF_LD);   // [FF_NW][QT] (max, sum)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int h = blockIdx.y, b = blockIdx.z, q0 = blockIdx.x * QT;
  const int d = n_head * 64, ld3 = 3 * d;
  const float* base = qkv + (int64_t)b * kCtx * ld3 + h * 64;

  f32x4 qf[NB][4];
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const float* qp = base + (int64_t)min(q0 + n * 16 + l16, kCtx - 1) * ld3 + 4 * g;
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[n][s] = *(const f32x4*)(qp + 16 * s) * kQScaleLog2;
  }
  f32x4 o[NB][4];
  float m[NB], l[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    m[n] = -INFINITY;
    l[n] = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[n][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  f32x4 kf[4], vf[4];
  auto load = [&](int t) {
    const float* kp = base + (int64_t)min(t * 16 + l16, kCtx - 1) * ld3 + d + 4 * g;
#pragma unroll
    for (int s = 0; s < 4; ++s) kf[s] = *(const f32x4*)(kp + 16 * s);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      vf[r] = *(const f32x4*)(base + (int64_t)min(t * 16 + 4 * g + r, kCtx - 1) * ld3 + 2 * d + 4 * l16);
  };
  load(wave);
  for (int t = wave; t < NT; t += FF_NW) {
    f32x4 kc[4], vc[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      kc[s] = kf[s];
      vc[s] = vf[s];
    }
    if (t + FF_NW < NT) load(t + FF_NW);
    f32x4 p[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) p[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          p[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(kc[s][e], qf[n][s][e], p[n], 0, 0, 0);
    if (t * 16 + 16 > kCtx) {
#pragma unroll
      for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (t * 16 + 4 * g + r >= kCtx) p[n][r] = -INFINITY;
    }
    bool moved = false;
    float mn[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      float x = fmaxf(fmaxf(p[n][0], p[n][1]), fmaxf(p[n][2], p[n][3]));
      x = fmaxf(x, __shfl_xor(x, 16, 64));
      x = fmaxf(x, __shfl_xor(x, 32, 64));
      mn[n] = fmaxf(m[n], x);                      // finite: every tile holds real keys
      moved |= mn[n] != m[n];
    }
    if (__any(moved)) {
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const float f = __builtin_amdgcn_exp2f(m[n] - mn[n]);   // 0 on the first tile
        m[n] = mn[n];
        l[n] *= f;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[n][j] *= f;
      }
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) {
#pragma unroll
      for (int r = 0; r < 4; ++r) p[n][r] = __builtin_amdgcn_exp2f(p[n][r] - m[n]);
      l[n] += (p[n][0] + p[n][1]) + (p[n][2] + p[n][3]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < NB; ++n)
          o[n][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[r][j], p[n][r], o[n][j], 0, 0, 0);
  }
  // the wave's record of query l16: lane group g holds dims 16 g .. 16 g + 15
  // (element r of component j is dim 16 g + 4 r + j)
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    l[n] += __shfl_xor(l[n], 16, 64);
    l[n] += __shfl_xor(l[n], 32, 64);
    float* row = osh + (wave * QT + n * 16 + l16) * FF_LD + 16 * g;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *(f32x4*)(row + 4 * r) = f32x4{o[n][0][r], o[n][1][r], o[n][2][r], o[n][3][r]};
    if (g == 0) mlsh[wave * QT + n * 16 + l16] = make_float2(m[n], l[n]);
  }
  __syncthreads();
  for (int i = tid; i < QT * 16; i += FF_NW * 64) {
    const int q = i >> 4, c = (i & 15) * 4;
    if (q0 + q >= kCtx) break;                     // later items are later queries
    float2 ml[FF_NW];
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < FF_NW; ++w) {
      ml[w] = mlsh[w * QT + q];
      M = fmaxf(M, ml[w].x);
    }
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
#pragma unroll
    for (int w = 0; w < FF_NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(ml[w].x - M);
      den = fmaf(f, ml[w].y, den);
      num += f * *(const f32x4*)(osh + (w * QT + q) * FF_LD + c);
    }
    *(f32x4*)(out + ((int64_t)b * kCtx + q0 + q) * d + h * 64 + c) = num * (1.0f / den);
  }
}

template <int NB>
static void launch_flash_f32(const float* qkv, float* out, int B, int n_head, hipStream_t s) {
  constexpr int QT = 16 * NB;
  constexpr size_t lds = (size_t)FF_NW * QT * (FF_LD + 2) * sizeof(float);
  static_assert(lds <= 160 * 1024, "LDS");
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)k_flash_f32<NB>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)attr;
  k_flash_f32<NB><<<dim3((kCtx + QT - 1) / QT, n_head, B), FF_NW * 64, lds, s>>>(qkv, out, n_head);
}

// 32 or 48 queries a block: whichever needs less time in rounds of one block
// per CU, a round costing as much as its queries.  One clip of 6 heads has
// 282 blocks of 32 (a second round of 26) but 192 of 48.
void flash_attn_f32(const float* qkv, float* out, int B, int n_head, hipStream_t s) {
  if (B <= 0) return;
  auto cost = [&](int nb) {
    const int64_t blocks = (int64_t)((kCtx + 16 * nb - 1) / (16 * nb)) * n_head * B;
    return (blocks + 255) / 256 * nb;
  };
  if (cost(3) < cost(2))
    launch_flash_f32<3>(qkv, out, B, n_head, s);
  else
    launch_flash_f32<2>(qkv, out, B, n_head, s);
}

// ---------------------------------------------------------------------------
// Decode attention
// ---------------------------------------------------------------------------
// Eight consecutive head dims of one key / value row, in storage type.
template <typename T>
struct Row8;
template <>
struct Row8<float> {
  float4 a, c;
  __device__ __forceinline__ void keep(bool ok) {
    if (!ok) a = c = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // at byte offset `off` of a wave-uniform base
  __device__ __forceinline__ void load(const float* p, uint32_t off) {
    a = *(const float4*)((const char*)p + off);
    c = *(const float4*)((const char*)p + off + 16);
  }
  __device__ __forceinline__ void get(float* v) const {
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
  }
};
template <>
struct Row8<bf16_t> {
  uint4 u;
  __device__ __forceinline__ void keep(bool ok) {
    if (!ok) u = uint4{0u, 0u, 0u, 0u};
  }
  __device__ __forceinline__ void load(const bf16_t* p, uint32_t off) {
    u = *(const uint4*)((const char*)p + off);
  }
  __device__ __forceinline__ void get(float* v) const {
    v[0] = __uint_as_float(u.x << 16); v[1] = __uint_as_float(u.x & 0xffff0000u);
    v[2] = __uint_as_float(u.y << 16); v[3] = __uint_as_float(u.y & 0xffff0000u);
    v[4] = __uint_as_float(u.z << 16); v[5] = __uint_as_float(u.z & 0xffff0000u);
    v[6] = __uint_as_float(u.w << 16); v[7] = __uint_as_float(u.w & 0xffff0000u);
  }
};

// Decode cross attention: one block per (row, head, chunk of the 1500 keys).
// Each thread issues the loads of its share of the chunk's keys (8 lanes per
// key, 32 keys per pass, NP passes), K and V, before any arithmetic, so the
// value stream's latency hides behind the scores and the softmax; scores stay
// in registers (one cross-lane reduction per key), and three block barriers
// remain.  The block leaves a (max, sum, weighted values) record.
template <typename T>
__global__ __launch_bounds__(256) void k_dattn_cross(const float* __restrict__ q,
                                                     const T* __restrict__ cache,
                                                     int64_t slot_stride, int64_t layer_off,
                                                     const int32_t* __restrict__ slots, int n_head,
                                                     float* __restrict__ part) {
  constexpr int NCH = kCrossChunks<T>, NP = 48 / NCH;   // 32 * 48 = 1536 keys
  constexpr int CK = NP * 32;
  static_assert(CK * NCH >= kCtx && CK * (NCH - 1) < kCtx, "chunks cover the keys");
  __shared__ __attribute__((aligned(16))) float qs[64];
  __shared__ float red[2][4];
  __shared__ float ored[4][64];
  const int h = blockIdx.x, row = blockIdx.y, chunk = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d = n_head * 64;
  const int k0 = chunk * CK;
  const int kn = min(CK, kCtx - k0);
  const int sub = lane >> 3, dc = (lane & 7) * 8;
  const T* kb = cache + (int64_t)slots[row] * slot_stride + layer_off + (int64_t)h * kCtx * 64;
  const T* vb = kb + (int64_t)n_head * kCtx * 64;

  // all loads of the block's keys first, without a branch (past the chunk the
  // last key again, not used)
  Row8<T> kr[NP], vr[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const uint32_t off = (uint32_t)((k0 + min(p * 32 + wave * 8 + sub, kn - 1)) * 64 + dc) * sizeof(T);
    kr[p].load(kb, off);
    vr[p].load(vb, off);
  }
  if (tid < 64) qs[tid] = q[(int64_t)row * d + h * 64 + tid] * 0.125f;
  __syncthreads();
  float qv[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) qv[i] = qs[dc + i];

  // scores: 8 dims per lane, summed over the key's 8 lanes
  float sc[NP];
  float mx = -INFINITY;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    float kv[8];
    kr[p].get(kv);
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) a = fmaf(qv[i], kv[i], a);
    a = group8_sum_lanes(a);
    const int kk = p * 32 + wave * 8 + sub;
    sc[p] = kk < kn ? a : -INFINITY;
    mx = fmaxf(mx, sc[p]);
  }
  mx = stride8_max_lanes(mx);
  if (lane == 0) red[0][wave] = mx;
  __syncthreads();
  const float M = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));

  // probabilities and the weighted value sum
  float l = 0.f, acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const float pr = expf(sc[p] - M);                // 0 for keys past the chunk
    l += pr;
    float vv[8];
    vr[p].keep(p * 32 + wave * 8 + sub < kn);
    vr[p].get(vv);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = fmaf(pr, vv[i], acc[i]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = stride8_sum_lanes(acc[i]);
  l = stride8_sum_lanes(l);                          // (a key's eight lanes hold the same)
  if (lane < 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) ored[wave][dc + i] = acc[i];
  }
  if (lane == 0) red[1][wave] = l;
  __syncthreads();
  if (tid < 64) {
    float* rec = part + (((int64_t)row * n_head + h) * NCH + chunk) * DA_REC;
    rec[2 + tid] = ored[0][tid] + ored[1][tid] + ored[2][tid] + ored[3][tid];
    if (tid == 0) {
      rec[0] = M;
      rec[1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
  }
}

// One wave per (row, head).
template <typename T>
__global__ __launch_bounds__(256) void k_cross_merge(const float* __restrict__ part, int n,
                                                     T* __restrict__ out) {
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w < n) St<T>::st(out, (int64_t)w * kHeadDim + lane, cross_merge<T>(part, w, lane));
}

// Decode self attention: one block per (row, head) over the row's position + 1
// keys, writing the output directly.  The keys go in parts of 32 NP, so a
// thread holds only one part's K and V rows (bf16: three parts of 160 keys, five
// blocks per CU, which is what the short rows' latency needs);
// a further part, present only for rows long enough, loads its keys as soon as
// the part before has its scores and its values once that part's weighted sum
// is done, and joins through the usual online-softmax rescale (block-wide
// maxima, so all lanes share one reference).  The step's query, key and value
// are qkv [D][3d]; the new key and value, rounded to the storage type, go into
// the cache at the last position and into the scores from LDS.
template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
void k_dattn_self(const float* __restrict__ qkv, T* cache, int64_t slot_stride, int64_t layer_off,
                  const int32_t* __restrict__ slots, const int32_t* __restrict__ pos, int n_head,
                  T* __restrict__ out) {
  constexpr int NP = sizeof(T) == 2 ? 5 : 3, PART = 32 * NP;
  constexpr int NPART = (kTextCtx + PART - 1) / PART;
  __shared__ __attribute__((aligned(16))) float qs[64];
  __shared__ __attribute__((aligned(16))) T kvnew[2][64];
  __shared__ float red[NPART + 1][4];
  __shared__ float ored[4][64];
  const int h = blockIdx.x, row = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d = n_head * 64;
  const int n = pos[row] + 1;                       // keys, this step's included
  T* kb = cache + (int64_t)slots[row] * slot_stride + layer_off + (int64_t)h * kTextCtx * 64;
  T* vb = kb + (int64_t)n_head * kTextCtx * 64;
  const int sub = lane >> 3, dc = (lane & 7) * 8;
  auto key_of = [&](int part, int p) { return part * PART + p * 32 + wave * 8 + sub; };
  // cached keys (all but the last) of a part, without a branch: past them the
  // last cached key again, not used
  Row8<T> kr[NP], vr[NP];
  const int last = max(n - 2, 0);
  auto off_of = [&](int part, int p) {
    return (uint32_t)(min(key_of(part, p), last) * 64 + dc) * (uint32_t)sizeof(T);
  };
  auto load_k = [&](int part) {
#pragma unroll
    for (int p = 0; p < NP; ++p) kr[p].load(kb, off_of(part, p));
  };
  auto load_v = [&](int part) {
#pragma unroll
    for (int p = 0; p < NP; ++p) vr[p].load(vb, off_of(part, p));
  };
  load_k(0);
  load_v(0);
  if (wave < 3) {                                    // q, the new k, the new v
    const float v = qkv[((int64_t)row * 3 + wave) * d + h * 64 + lane];
    if (wave == 0) {
      qs[lane] = v * 0.125f;
    } else {
      St<T>::st(kvnew[wave - 1], lane, v);
      St<T>::st(wave == 1 ? kb : vb, (int64_t)(n - 1) * 64 + lane, v);
    }
  }
  __syncthreads();
  float qv[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) qv[i] = qs[dc + i];

  float M = -INFINITY, l = 0.f, acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
#pragma unroll
  for (int part = 0; part < NPART; ++part) {
    if (part * PART >= n) break;                     // block-uniform
    const bool more = (part + 1) * PART < n;
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (key_of(part, p) == n - 1) kr[p].load(&kvnew[0][dc], 0);
    float sc[NP];
    float mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      float kv[8];
      kr[p].get(kv);
      float a = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) a = fmaf(qv[i], kv[i], a);
      a = group8_sum_lanes(a);
      sc[p] = key_of(part, p) < n ? a : -INFINITY;
      mx = fmaxf(mx, sc[p]);
    }
    mx = stride8_max_lanes(mx);
    if (lane == 0) red[part][wave] = mx;
    __syncthreads();
    if (more) load_k(part + 1);                      // this part's keys are done with
    const float Mn =
        fmaxf(M, fmaxf(fmaxf(red[part][0], red[part][1]), fmaxf(red[part][2], red[part][3])));
    const float f = expf(M - Mn);                    // 0 on the first part (M = -inf)
    l *= f;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= f;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const float pr = expf(sc[p] - Mn);             // 0 for keys past the row
      l += pr;
      float vv[8];
      vr[p].keep(key_of(part, p) < n);
      if (key_of(part, p) == n - 1) vr[p].load(&kvnew[1][dc], 0);
      vr[p].get(vv);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = fmaf(pr, vv[i], acc[i]);
    }
    M = Mn;
    if (more) load_v(part + 1);                      // ... and so are its values
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = stride8_sum_lanes(acc[i]);
  l = stride8_sum_lanes(l);                          // (a key's eight lanes hold the same)
  if (lane < 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) ored[wave][dc + i] = acc[i];
  }
  if (lane == 0) red[NPART][wave] = l;
  __syncthreads();
  if (tid < 64) {
    const float o = ored[0][tid] + ored[1][tid] + ored[2][tid] + ored[3][tid];
    const float L = red[NPART][0] + red[NPART][1] + red[NPART][2] + red[NPART][3];
    St<T>::st(out, (int64_t)row * d + h * 64 + tid, o / L);
  }
}

int decode_attn_part_floats(int D, int n_head) { return D * n_head * kCrossChunks<float> * DA_REC; }

template <typename T>
void decode_self_attn(const float* qkv, T* cache, int64_t slot_stride, int64_t layer_off,
                      const int32_t* slots, const int32_t* pos, int D, int n_head, T* out,
                      hipStream_t s) {
  if (D > 0)
    k_dattn_self<T><<<dim3(n_head, D), 256, 0, s>>>(qkv, cache, slot_stride,
                                                    layer_off, slots, pos, n_head, out);
}
template <typename T>
void decode_cross_attn(const float* q, const T* cache, int64_t slot_stride, int64_t layer_off,
                       const int32_t* slots, int D, int n_head, float* part, hipStream_t s) {
  if (D > 0)
    k_dattn_cross<T><<<dim3(n_head, D, kCrossChunks<T>), 256, 0, s>>>(
        q, cache, slot_stride, layer_off, slots, n_head, part);
}
template <typename T>
void decode_cross_merge(const float* part, int D, int n_head, T* out, hipStream_t s) {
  if (D > 0) k_cross_merge<T><<<(D * n_head + 3) / 4, 256, 0, s>>>(part, D * n_head, out);
}
template void decode_self_attn<float>(const float*, float*, int64_t, int64_t, const int32_t*,
                                      const int32_t*, int, int, float*, hipStream_t);
template void decode_self_attn<bf16_t>(const float*, bf16_t*, int64_t, int64_t, const int32_t*,
                                       const int32_t*, int, int, bf16_t*, hipStream_t);
template void decode_cross_attn<float>(const float*, const float*, int64_t, int64_t, const int32_t*,
                                       int, int, float*, hipStream_t);
template void decode_cross_attn<bf16_t>(const float*, const bf16_t*, int64_t, int64_t,
                                        const int32_t*, int, int, float*, hipStream_t);
template void decode_cross_merge<float>(const float*, int, int, float*, hipStream_t);
template void decode_cross_merge<bf16_t>(const float*, int, int, bf16_t*, hipStream_t);

}  // namespace asr
