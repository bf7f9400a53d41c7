// Prompt-phase attention for bf16 tensors on the CDNA4 matrix cores (head_dim 128).
//
// Pass 1, attn_fwd_bf16 (Sec. 4.1 Eq. 4; Sec. 3 Eq. 3): row-stationary flash attention.  A
//   workgroup owns 256 query rows (8 wavefronts x 32), streams 64-key tiles of K and of the
//   pre-transposed V through LDS and keeps S^T = K Q^T in the MFMA accumulator layout, where
//   one lane owns one query column: row maxima and sums are then in-register reductions.
//   Emits O and the row log-sum-exp (base 2, of the scaled logits).
//   The P V product runs in fp16, not bf16: probabilities rounded to bf16 (8 significant bits)
//   alone cost up to 2^-8 relative on O, fp16 (11 bits) keeps it below 2^-11.  V is converted
//   once, in the transposing pre-pass, with a per-head power-of-two scale that maps max|v| to
//   2^13 (exact for bf16 inputs inside fp16's exponent range), and P carries a factor 2^12 so
//   that small probabilities stay in fp16's normal range; both factors cancel in O.
// Pass 2, colsum_bf16 (column sums of the attention matrix, Sec. 4.1; Eq. 6 prompt case):
//   key-stationary.  A workgroup owns 256 keys, streams query tiles, recomputes S^T with the
//   keys as the stationary MFMA operand, and accumulates P = exp2(S - lse) per key in
//   registers; the column sums come out without atomics, the G query heads of a KV group are
//   added in ascending order, and per-query-head partial sums of the column sums and their
//   squares feed the variance of Eq. 4.
// The column sums need every row's final normaliser, so they cannot come out of the single
// online-softmax pass; the second QK^T product is implementation overhead.
//
// v_mfma_f32_32x32x16_bf16 operand layout (lane l, m = l % 32, h = l / 32):
//   A[m][8h .. 8h+7], B[8h .. 8h+7][m], D[(r/4)*8 + 4h + r%4][m] for r = 0..15.
#include "d2o_internal.h"
#include <algorithm>
#include <type_traits>

#include "device_utils.h"

namespace d2o {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kD = 128;
// The attention kernel's LDS tiles are filled from memory directly (16 bytes per lane, 1 KB per instruction, consecutive in
// LDS): an instruction's four rows of a [token][d] tile (eight of a [d][key] tile) are a group without
// padding, and the lanes choose what they read: chunk k (16 bytes) of a row sits at k ^ (row & 3)
// (k ^ ((row >> 1) & 3)).  Groups are 64 bytes apart, so that the 16 lanes of a 128-bit access phase,
// which read one chunk of 16 rows, meet all banks once; the low bits of k only are permuted,
// which leaves the rest of an operand's address to the instruction's constant offset.
constexpr int kGroupLd = 512 + 32;  // elements from one group to the next
constexpr int kLdQ = kD + 8;        // LDS row pitch (elements) of the column-sum kernel's query tiles
__device__ __forceinline__ int swz(int chunk, int x) { return ((chunk & ~3) << 3) + (((chunk & 3) ^ x) << 3); }
__device__ __forceinline__ int at_k(int row, int chunk) { return (row >> 2) * kGroupLd + (row & 3) * kD + swz(chunk, row & 3); }
__device__ __forceinline__ int at_v(int row, int chunk) { return (row >> 3) * kGroupLd + (row & 7) * 64 + swz(chunk, (row >> 1) & 3); }
constexpr float kPShift = 12.f;  // probabilities are formed as 2^12 * p before the fp16 rounding
constexpr float kLazy = 3.f;     // log2 of the growth the exponent reference tolerates before it moves

// max |v| of a share of a (sequence, KV head)'s values, as the bit pattern of the non-negative float:
// vmax[head][share].  (Combined by atomics on one word per head, the words of all heads in a line or
// two of memory, 2048 workgroups queued for 15 us on them: 21.6 us at 32 heads x 4096 tokens, and
// the words had to be cleared by a launch of their own.)
__global__ __launch_bounds__(256) void vabsmax_kernel(const uint16_t* __restrict__ V, View vv, uint32_t* __restrict__ vmax,
                                                      int n) {
  __shared__ uint32_t red[4];
  const int h = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const uint16_t* src = V + b * vv.sb + h * vv.sh;
  uint32_t m = 0;
  const int step = gridDim.x * 256, col = (threadIdx.x & 15) * 8;
  for (int c0 = blockIdx.x * 256 + threadIdx.x; c0 < n * 16; c0 += 4 * step) {
    u32x4 v[4];  // four loads in flight (past the end: the last row again)
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = *reinterpret_cast<const u32x4*>(src + int64_t(min((c0 + u * step) >> 4, n - 1)) * vv.sn + col);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        m = max(m, (v[u][i] << 16) & 0x7FFFFFFFu);
        m = max(m, v[u][i] & 0x7FFF0000u);
      }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) vmax[(b * Hkv + h) * kVmaxShares + blockIdx.x] = max(max(red[0], red[1]), max(red[2], red[3]));
}

// Power-of-two factor that maps max|v| into [2^13, 2^14) (1 when the head is all zero).
__device__ __forceinline__ float v_scale_from_max(uint32_t maxbits) {
  const int e = int((maxbits >> 23) & 0xFF);  // biased exponent of max |v|
  if (e == 0 || e == 255) return 1.0f;
  const int k = min(max(e - 127 - 13, -100), 100);
  return __uint_as_float(uint32_t(127 - k) << 23);  // 2^-k
}

// V [b][h][n][d] (bf16) -> VT [b][h][npad/64][d][64] (fp16, scaled), zero for keys >= n: the
// transposed values of every 64-key tile are contiguous (a [d][npad] layout would put a tile's
// rows a power-of-two stride apart, all on one memory channel).
__global__ __launch_bounds__(256) void transpose_v(const uint16_t* __restrict__ V, View vv, uint16_t* __restrict__ VT,
                                                   const uint32_t* __restrict__ vmax, float* __restrict__ unscale,
                                                   int n, int npad, int shares) {
  __shared__ uint16_t t[64][kD + 2];
  const int k0 = blockIdx.x * 64, h = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y, lane = threadIdx.x & 63;
  static_assert(kVmaxShares == 64, "a share per lane");
  uint32_t vm = lane < shares ? vmax[(b * Hkv + h) * kVmaxShares + lane] : 0u;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) vm = max(vm, (uint32_t)__shfl_xor((int)vm, o, 64));
  const float mul = v_scale_from_max(vm);
  if (blockIdx.x == 0 && threadIdx.x == 0) unscale[b * Hkv + h] = 1.0f / mul;
  const uint16_t* src = V + b * vv.sb + h * vv.sh;
  for (int c = threadIdx.x; c < 64 * 16; c += 256) {
    const int row = c >> 4, col = (c & 15) * 8;
    u32x4 v = {0, 0, 0, 0};
    if (k0 + row < n) v = *reinterpret_cast<const u32x4*>(src + int64_t(k0 + row) * vv.sn + col);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const _Float16 lo = (_Float16)(__uint_as_float(v[i] << 16) * mul);
      const _Float16 hi = (_Float16)(__uint_as_float(v[i] & 0xFFFF0000u) * mul);
      t[row][col + 2 * i] = __builtin_bit_cast(uint16_t, lo);
      t[row][col + 2 * i + 1] = __builtin_bit_cast(uint16_t, hi);
    }
  }
  __syncthreads();
  uint16_t* dst = VT + (int64_t(b) * Hkv + h) * kD * npad;
  for (int c = threadIdx.x; c < kD * 8; c += 256) {
    const int dd = c >> 3, kc = (c & 7) * 8;
    uint16_t o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = t[kc + i][dd];
    u32x4 v;
    v[0] = o[0] | (uint32_t(o[1]) << 16); v[1] = o[2] | (uint32_t(o[3]) << 16);
    v[2] = o[4] | (uint32_t(o[5]) << 16); v[3] = o[6] | (uint32_t(o[7]) << 16);
    *reinterpret_cast<u32x4*>(dst + (int64_t(blockIdx.x) * kD + dd) * 64 + kc) = v;
  }
}

// MFMA row m -> key offset inside a 32-key sub-tile, chosen so that accumulator registers
// 8*kb .. 8*kb+7 of lane-half h hold the 8 consecutive keys 16*kb + 8*h .. +7: exactly the
// B-operand slice the P V product needs, with no cross-lane movement.
__device__ __forceinline__ int perm_key(int m) { return (m & ~0xC) | ((m & 4) << 1) | ((m & 8) >> 1); }

// Workgroups are handed to the chip's eight XCDs (each with its own L2) round-robin in launch
// order.  With the head as the slow grid index a head's workgroups land on all eight, and every
// L2 fetches every head's K / V tiles from memory.  This remaps (block, head) so that all
// workgroups of a head run on one XCD, heads that share a KV head on the same one, and an XCD
// works through its heads one after the other: the workgroups of a head, which walk the same
// tiles at about the same time, then share them in one L2.  hz = head + heads * sequence.
__device__ __forceinline__ void xcd_remap(int nx, int nhz, int& bx, int& hz) {
  constexpr int kXcd = 8;
  if (nhz % kXcd) return;  // identity when the heads do not divide over the XCDs
  const int lin = bx + nx * hz, xcd = lin % kXcd, s = lin / kXcd;
  hz = xcd * (nhz / kXcd) + s / nx;
  bx = s % nx;
}

// The same for a launch of single blocks of very different lengths, the longest (bx = 0) first in every XCD over
// all of its heads: what joins a busy CU at the end is short.
__device__ __forceinline__ void xcd_remap_longest_first(int nx, int nhz, int& bx, int& hz) {
  constexpr int kXcd = 8;
  const int lin = bx + nx * hz, per = nhz / kXcd;
  if (nhz % kXcd) {
    hz = lin % nhz;
    bx = lin / nhz;
  } else {
    const int s = lin / kXcd;
    hz = lin % kXcd * per + s % per;
    bx = s / per;
  }
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return Elem<uint16_t>::from_f32(lo) | uint32_t(Elem<uint16_t>::from_f32(hi)) << 16;
}

constexpr int kKsElems = 16 * kGroupLd;  // one K tile in LDS
constexpr int kVsElems = 16 * kGroupLd;  // one V^T tile in LDS
constexpr int kAttnSmemBytes = 2 * (kKsElems + kVsElems) * 2;
constexpr int kAttnRW = 1;                     // 32-row blocks per wavefront

// NW wavefronts per workgroup, each owning RW 32-row MFMA column blocks (blocks of one
// wavefront share every K / V^T operand read from LDS).  Built as 8 x 1: 256 query rows per
// workgroup, two wavefronts per SIMD, which measured faster than 4 x 2; and as 4 x 1 for launches that
// do not fill the chip with those (see the launch).  K and V^T tiles of 64
// keys are double-buffered in LDS.  A tile costs a wavefront about as many vector-ALU cycles
// (32 exponentials per lane at a quarter of the ALU rate) as matrix-core cycles (32 MFMAs), so
// the two wavefronts of a SIMD alternate between the two units (see the schedule below).
template <int RW, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_fwd_bf16(const uint16_t* __restrict__ Q, View qv,
                                                     const uint16_t* __restrict__ K, View kv,
                                                     const uint16_t* __restrict__ VT, const float* __restrict__ unscale,
                                                     void* __restrict__ O, View ov, float* __restrict__ lse2, int n,
                                                     int npad, int G, int out_f32, int nblk, int paired) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  uint16_t* Ks = smem;                 // [2][kKsElems]
  uint16_t* Vs = smem + 2 * kKsElems;  // [2][kVsElems]
  const int Hq = gridDim.y, Hkv = Hq / G;
  int bx = blockIdx.x, hz = blockIdx.y + Hq * blockIdx.z;
  if (paired)
    xcd_remap(gridDim.x, Hq * gridDim.z, bx, hz);
  else
    xcd_remap_longest_first(gridDim.x, Hq * gridDim.z, bx, hz);
  const int hq = hz % Hq, b = hz / Hq, hk = hq / G;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 31, h = lane >> 5;
  constexpr int kWR = 32 * RW;   // rows per wavefront
  constexpr int NT = 64 * NW;    // threads
  constexpr int BM = NW * kWR;   // query rows per workgroup
  const float scale2 = kLog2e / sqrtf(float(kD));
  // The work of a row block grows with its position (causal).  A workgroup takes row block
  // nblk - 1 - x (the longer one first) and then row block x: every workgroup has the same
  // amount of work and the launch fills the chip in whole rounds (with one row block per
  // workgroup the longest ones ran on a nearly empty chip at the end: 80 % packing).
  const uint16_t* kbase = K + b * kv.sb + hk * kv.sh;
  const uint16_t* vtbase = VT + (int64_t(b) * Hkv + hk) * kD * npad;
  // tile loads: a wavefront fills 64 / NW rows of K (four per instruction) and 128 / NW of V^T (eight)
  auto load_k = [&](int t) {
#pragma unroll
    for (int i = 0; i < 16 / NW; ++i) {
      // key r of a 32-key sub-tile is stored at LDS row perm_key(r) (an involution), so that
      // MFMA row m, which must see key perm_key(m), reads LDS row m
      const int r0 = (w * (16 / NW) + i) * 4, lrow = r0 + (lane >> 4);
      const int row = (lrow & 32) | perm_key(lrow & 31);
      load_lds16(kbase + int64_t(min(t * 64 + row, n - 1)) * kv.sn + swz(lane & 15, lane >> 4),
                 Ks + (t & 1) * kKsElems + (r0 >> 2) * kGroupLd);
    }
  };
  auto load_v = [&](int t) {
#pragma unroll
    for (int i = 0; i < 16 / NW; ++i) {
      const int r0 = (w * (16 / NW) + i) * 8, row = r0 + (lane >> 3);
      load_lds16(vtbase + (int64_t(t) * kD + row) * 64 + swz(lane & 7, (lane >> 4) & 3),
                 Vs + (t & 1) * kVsElems + (r0 >> 3) * kGroupLd);
    }
  };
  bf16x8 bq[RW][8];
  auto tiles_of = [&](int blk) { return min(blk * BM + BM - 1, n - 1) / 64 + 1; };
  // The first tiles of a block and its query rows, all on their way together, the second block's while the
  // first one's output rows are formed and written.  (A block of n tiles takes n times 2 us and, however short, several us
  // at its ends: with the queries waited for before the tiles were requested, and the output rows written 8
  // instead of 16 bytes per lane, 128 heads of 1024 tokens 59.3 us, now 54.5; 32 heads of 3072 113 -> 109, of 4096 162 -> 156.)
  auto request = [&](int blk) {
    load_k(0);
#pragma unroll
    for (int j = 0; j < RW; ++j) {
      const uint16_t* qp = Q + b * qv.sb + hq * qv.sh + int64_t(min(blk * BM + w * kWR + j * 32 + m, n - 1)) * qv.sn;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) bq[j][ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 16 + h * 8);
    }
    load_v(0);
    if (tiles_of(blk) > 1) load_k(1);
  };
  const int passes = paired && bx < nblk - 1 - bx ? 2 : 1;
  request(nblk - 1 - bx);
  for (int pass = 0; pass < passes; ++pass) {
  const int blk = pass == 0 ? nblk - 1 - bx : bx;
  const int wr0 = blk * BM + w * kWR;  // first row of this wavefront

  f32x16 o[RW][4];
#pragma unroll
  for (int j = 0; j < RW; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[j][i][r] = 0.f;
  float mrun[RW], lsum[RW];
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    mrun[j] = -INFINITY;
    lsum[j] = 0.f;
  }

  const int ntile = tiles_of(blk);

  // ---- the three stages of a tile, for this wavefront's rows
  f32x16 s[RW][2];
  f16x8 pb[RW][2][2];
  auto active = [&](int t) { return t * 64 <= wr0 + kWR - 1; };  // else the tile is above the diagonal
  auto qk = [&](int t) {  // S^T = K Q^T of tile t (K from its LDS buffer)
    const uint16_t* ksb = Ks + (t & 1) * kKsElems;
#pragma unroll
    for (int j = 0; j < RW; ++j)
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[j][st][r] = 0.f;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&ksb[at_k(st * 32 + m, ks * 2 + h)]);
#pragma unroll
        for (int j = 0; j < RW; ++j)
          s[j][st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bq[j][ks], s[j][st], 0, 0, 0);
      }
  };
  auto softmax = [&](int t) {  // s -> probabilities pb (fp16, scaled), running maximum and sum, rescale of o
    const int k0 = t * 64;
    // register r of sub-tile st holds key k0 + 32*st + 16*(r/8) + 8*h + r%8
    const bool diag = k0 + 63 > wr0;
#pragma unroll
    for (int j = 0; j < RW; ++j) {
      const int q_row = wr0 + j * 32 + m;
      if (diag) {
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = k0 + st * 32 + (r >> 3) * 16 + h * 8 + (r & 7);
            if (key > q_row) s[j][st][r] = -INFINITY;
          }
      }
      float mx = s[j][0][0];
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[j][st][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      // Exponent reference with 2^12 headroom.  It follows the row maximum lazily: it moves only
      // when the maximum has outgrown it by more than 2^kLazy, so the probabilities stay below
      // 2^(12 + kLazy), inside fp16, and the rescale of the accumulators becomes rare.
      const float mcand = fmaf(mx, scale2, -kPShift);
      const bool grew = mcand > mrun[j] + kLazy;
      const float mnew = grew ? mcand : mrun[j];
      const float alpha = __builtin_amdgcn_exp2f(mrun[j] - mnew);
      mrun[j] = mnew;
      float psum = 0.f;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[j][st][r], scale2, -mnew));
          psum += p;
          pb[j][st][r >> 3][r & 7] = (_Float16)p;
        }
      lsum[j] = fmaf(lsum[j], alpha, psum);
      if (__any(grew)) {  // wavefront-uniform: skip the rescale when no row's maximum moved
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[j][i][r] *= alpha;
      }
    }
  };
  // o += V^T P^T of tile t, then (WITH_QK) S^T = K Q^T of tile t + 1: 16 + 16 MFMAs whose LDS
  // operands are fetched two batches of four ahead, so that the matrix core never waits for an
  // LDS round trip (the compiler, left alone, keeps only two reads in flight).
  auto mma_operand = [&](int t, int idx) -> u32x4 {
    if (idx < 16) {  // P V: idx = (st, kb, dc)
      const int st = idx >> 3, kb = (idx >> 2) & 1, dc = idx & 3;
      return *reinterpret_cast<const u32x4*>(&Vs[(t & 1) * kVsElems + at_v(dc * 32 + m, st * 4 + kb * 2 + h)]);
    }
    const int st = (idx - 16) & 1, ks = (idx - 16) >> 1;  // Q K^T of the next tile, the two sub-tiles alternating
    return *reinterpret_cast<const u32x4*>(&Ks[((t + 1) & 1) * kKsElems + at_k(st * 32 + m, ks * 2 + h)]);
  };
  auto mma_issue = [&](int idx, const u32x4& a) {
    if (idx < 16) {
      const int st = idx >> 3, kb = (idx >> 2) & 1, dc = idx & 3;
#pragma unroll
      for (int j = 0; j < RW; ++j)
        o[j][dc] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), pb[j][st][kb], o[j][dc], 0, 0, 0);
    } else {
      const int st = (idx - 16) & 1, ks = (idx - 16) >> 1;
#pragma unroll
      for (int j = 0; j < RW; ++j) {
        if (ks == 0) {
          const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          s[j][st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), bq[j][ks], zero, 0, 0, 0);
        } else {
          s[j][st] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), bq[j][ks], s[j][st], 0, 0, 0);
        }
      }
    }
  };
  auto mma_phase = [&](int t, auto with_qk) {
    constexpr int NB = decltype(with_qk)::value ? 8 : 4;  // batches of four MFMAs
    u32x4 A[2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) A[0][i] = mma_operand(t, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) A[1][i] = mma_operand(t, 4 + i);
#pragma unroll
    for (int bt = 0; bt < NB; ++bt) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 4; ++i) mma_issue(4 * bt + i, A[bt & 1][i]);
      __builtin_amdgcn_sched_barrier(0);
      if (bt + 2 < NB) {
#pragma unroll
        for (int i = 0; i < 4; ++i) A[bt & 1][i] = mma_operand(t, 4 * (bt + 2) + i);
      }
    }
  };
  // The wavefront in its matrix phase issues first: its instructions are few and keep the matrix core busy, the
  // other wavefront's softmax fills the slots between them (32768 tokens, 32 heads: 8.39 -> 8.08 ms; with the
  // softmax first 8.19).
  auto pv_qk = [&](int t, bool with_qk) {
    __builtin_amdgcn_s_setprio(1);
    if (with_qk)
      mma_phase(t, std::true_type{});
    else
      mma_phase(t, std::false_type{});
    __builtin_amdgcn_s_setprio(0);
  };

  // ---- ping-pong schedule.  The two wavefronts that share a SIMD (w and w + NW/2) run half a
  // tile apart: while one forms its probabilities on the vector ALU, the other runs its two
  // matrix products (P V of the tile, then Q K^T of the next) on the matrix core, and they swap
  // in the middle of the iteration.  K is staged two tiles ahead, V^T one tile ahead.
  const bool late = w >= NW / 2;
  // Pin the arrival of the Q operands here: otherwise the wait for them is placed inside the
  // loop, behind the tile loads issued there, and stalls the matrix products on those.
#pragma unroll
  for (int j = 0; j < RW; ++j)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) asm volatile("" ::"v"(bq[j][ks]));
  wait_vm<0>();
  __syncthreads();
  if (active(0)) {
    qk(0);
    if (!late) softmax(0);
  }
  __syncthreads();
  for (int t = 0; t < ntile; ++t) {
    const bool more = t + 1 < ntile, more2 = t + 2 < ntile;
    // V(t-1) and K(t) were last read before this iteration: their buffers take V(t+1), K(t+2)
    if (more2) load_k(t + 2);
    if (more) load_v(t + 1);
    if (active(t)) {
      if (late) {
        softmax(t);
      } else {
        pv_qk(t, more && active(t + 1));
      }
    }
    // no barrier between the two halves of an iteration: tiles are staged into buffers that
    // nobody reads during this iteration, and the half-tile offset between the two wavefronts
    // of a SIMD is re-established by the barrier at the end of every iteration
    if (late) {
      if (active(t)) pv_qk(t, more && active(t + 1));
    } else if (more && active(t + 1)) {
      softmax(t + 1);
    }
    wait_vm<0>();  // this wavefront's part of the next tiles is in LDS
    __syncthreads();
  }
  if (pass + 1 < passes) request(bx);  // (nobody reads the tiles any more)
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    const int q_row = wr0 + j * 32 + m;
    const float ltot = lsum[j] + __shfl_xor(lsum[j], 32, 64);
    if (q_row < n) {
      if (h == 0) lse2[(int64_t(b) * Hq + hq) * npad + q_row] = mrun[j] + log2f(ltot);
      if (O) {
        const float inv = unscale[b * Hkv + hk] / ltot;
        const int64_t ooff = b * ov.sb + hq * ov.sh + int64_t(q_row) * ov.sn;
        // registers 4 rg .. 4 rg + 3 hold d = 32 dc + 8 rg + 4 h + 0..3
#pragma unroll
        for (int dc = 0; dc < 4; ++dc) {
          if (out_f32) {
#pragma unroll
            for (int rg = 0; rg < 4; ++rg) {
              f32x4 v;
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = o[j][dc][4 * rg + i] * inv;
              *reinterpret_cast<f32x4*>(static_cast<float*>(O) + ooff + dc * 32 + rg * 8 + h * 4) = v;
            }
          } else {
            // the lanes of a row (h = 0, 1) swap halves of a register pair, so that each stores eight
            // consecutive d: 16 h2 + 8 h of the 32 columns
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
              uint32_t x[2], y[2];
#pragma unroll
              for (int i = 0; i < 2; ++i) {
                x[i] = pack_bf16(o[j][dc][8 * h2 + 2 * i] * inv, o[j][dc][8 * h2 + 2 * i + 1] * inv);
                y[i] = pack_bf16(o[j][dc][8 * h2 + 4 + 2 * i] * inv, o[j][dc][8 * h2 + 5 + 2 * i] * inv);
              }
              const auto s0 = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false);
              const auto s1 = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
              const u32x4 v = {s0[0], s1[0], s0[1], s1[1]};
              *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(O) + ooff + dc * 32 + h2 * 16 + h * 8) = v;
            }
          }
        }
      }
    }
  }
  }
}

// A workgroup owns BN = 32 KW keys (KW wavefronts x 32 keys, the stationary A operand) of one query head and streams query tiles of TQ rows through LDS, double-buffered; QW groups of such wavefronts share
// a tile's 32-row sub-tiles.  Tiles are visited from the END of the prompt downwards: every
// workgroup of a head then reads the same query tiles at about the same time (all start at
// the last tile), so the tiles are served from L2 instead of HBM.  The tiles pass through registers
// on their way to LDS: loaded straight into it, which gains the attention kernel 3 %, this one
// takes 4 % (32768 tokens) to 13 % longer.  (64 keys per wavefront, every LDS operand feeding two products, with two
// wavefronts per SIMD: 4.85 instead of 4.61 ms at 32768 tokens.)  Query heads that share a KV head are
// workgroups of their own: one after the other in one workgroup, 8 KV heads of 2048 tokens
// with four query heads each were 32 workgroups and 209 us instead of 43.
template <int KW, int QW, int TQ>
__global__ __launch_bounds__(64 * KW * QW) __attribute__((amdgpu_waves_per_eu(4, 4))) void colsum_bf16(const uint16_t* __restrict__ Q, View qv,
                                                           const uint16_t* __restrict__ K, View kv,
                                                           const float* __restrict__ lse2, float* __restrict__ colsum,
                                                           double* __restrict__ varpart, int n, int npad, int G,
                                                           int nblk, int paired) {
  constexpr int NW = KW * QW, NT = 64 * NW, BN = 32 * KW;
  constexpr int NQI = TQ / 32 / QW;            // sub-tiles per wavefront and tile
  constexpr int NP = TQ > 64 ? NQI : 1;        // parts in which the next tile is brought, one per sub-tile: fewer registers (12
                                               // of the 128 are spilled even so, 2 with tiles of 64 queries)
  constexpr int NCH = TQ * 16 / NT / NP;       // 16-byte loads per thread and part
  static_assert(BN <= NT && BN % 128 == 0 && TQ % (32 * QW) == 0 && BN % TQ == 0, "a thread per key, whole sub-tiles per wavefront");
  __shared__ __attribute__((aligned(16))) uint16_t Qs[2][TQ * kLdQ];
  __shared__ float ls[2][TQ];
  __shared__ float cs[QW][BN];
  __shared__ double red[NW][2];
  const int Hq = gridDim.y;
  int bx = blockIdx.x, hz = blockIdx.y + Hq * blockIdx.z;
  if (paired)
    xcd_remap(gridDim.x, Hq * gridDim.z, bx, hz);
  else
    xcd_remap_longest_first(gridDim.x, Hq * gridDim.z, bx, hz);
  const int hq = hz % Hq, b = hz / Hq, hk = hq / G;
  const int tid = threadIdx.x, w = tid >> 6, kw = w % KW, qw = w / KW, lane = tid & 63, m = lane & 31, h = lane >> 5;
  const float scale2 = kLog2e / sqrtf(float(kD));
  const uint16_t* qb = Q + b * qv.sb + hq * qv.sh;
  const float* lrow = lse2 + (int64_t(b) * Hq + hq) * npad;
  // The work of a key block grows with the number of queries behind it (causal), from one
  // query tile for the last block to all of them for the first.  A workgroup takes block x and
  // then block nblk - 1 - x: every workgroup then has the same amount of work and the launch
  // fills the chip in whole rounds (with one block per workgroup the CUs held 1.3 of 2 possible
  // workgroups on average, and the longest workgroup alone was a fifth of the kernel time).
  for (int pass = 0; pass < 1 + paired; ++pass) {
    const int tile = pass == 0 ? bx : nblk - 1 - bx;
    if (pass == 1 && tile <= bx) break;
    const int kb0 = tile * BN, kw0 = kb0 + kw * 32;  // first key of the workgroup / wavefront
    const uint16_t* kp = K + b * kv.sb + hk * kv.sh + int64_t(min(kw0 + m, n - 1)) * kv.sn;
    bf16x8 ak[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) ak[ks] = *reinterpret_cast<const bf16x8*>(kp + ks * 16 + h * 8);
    const int nqt = (n - kb0 + TQ - 1) / TQ;  // query tiles [kb0 + TQ j, kb0 + TQ j + TQ), visited j descending
    float acc[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    u32x4 qr[NCH];
    float lr = 0.f;
    auto load16 = [&](int j, int i) {  // this thread's load i of tile j
      const int c = tid + NT * i, row = c >> 4, col = (c & 15) * 8;
      return *reinterpret_cast<const u32x4*>(qb + int64_t(min(kb0 + TQ * j + row, n - 1)) * qv.sn + col);
    };
    auto store16 = [&](int buf, int i, const u32x4& v) {
      const int c = tid + NT * i, row = c >> 4, col = (c & 15) * 8;
      *reinterpret_cast<u32x4*>(&Qs[buf][row * kLdQ + col]) = v;
    };
    auto issue = [&](int j, int part) {
      const int q0 = kb0 + TQ * j;
#pragma unroll
      for (int i = 0; i < NCH; ++i) qr[i] = load16(j, part * NCH + i);
      if (part == 0 && tid < TQ) lr = (q0 + tid < n) ? lrow[q0 + tid] : INFINITY;  // +inf => p = 0
    };
    auto stage = [&](int buf, int part) {
#pragma unroll
      for (int i = 0; i < NCH; ++i) store16(buf, part * NCH + i, qr[i]);
      if (part == 0 && tid < TQ) ls[buf][tid] = lr;
    };
    __syncthreads();  // the previous block's readers are done with both buffers
    {  // the first tile whole
      issue(nqt - 1, 0);
      u32x4 more[NP * NCH];
#pragma unroll
      for (int i = NCH; i < NP * NCH; ++i) more[i] = load16(nqt - 1, i);
      stage(0, 0);
#pragma unroll
      for (int i = NCH; i < NP * NCH; ++i) store16(0, i, more[i]);
    }
    __syncthreads();
    for (int it = 0; it < nqt; ++it) {
      const int jt = nqt - 1 - it, buf = it & 1, q0 = kb0 + TQ * jt;
      if (NP == 1 && jt > 0) issue(jt - 1, 0);
#pragma unroll
      for (int qi = 0; qi < NQI; ++qi) {
        if (NP > 1 && jt > 0) issue(jt - 1, qi);
        // (where groups share a tile, a group's sub-tiles from the last to the first: the order of its additions does not
        // depend on the tile's size)
        const int qt = (QW > 1 ? NQI - 1 - qi : qi) * QW + qw, qbase = q0 + qt * 32;
        if (qbase + 31 >= kw0) {  // (else every query precedes every key of this wavefront)
          const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          f32x16 sacc = zero;
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) {
            const bf16x8 bqv = *reinterpret_cast<const bf16x8*>(&Qs[buf][(qt * 32 + m) * kLdQ + ks * 16 + h * 8]);
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak[ks], bqv, sacc, 0, 0, 0);
          }
          // register r: key kw0 + (r/4)*8 + 4h + r%4, query qbase + m
          const float lq = ls[buf][qt * 32 + m];
          const int query = qbase + m;
          if (qbase < kw0 + 31) {  // diagonal tile: mask query < key
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int key = kw0 + (r >> 2) * 8 + h * 4 + (r & 3);
              const float p = __builtin_amdgcn_exp2f(fmaf(sacc[r], scale2, -lq));
              acc[r] += (query >= key) ? p : 0.f;
            }
          } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += __builtin_amdgcn_exp2f(fmaf(sacc[r], scale2, -lq));
          }
        }
        if (NP > 1 && jt > 0) stage(buf ^ 1, qi);
      }
      if (NP == 1 && jt > 0) stage(buf ^ 1, 0);
      __syncthreads();
    }
    // add the 32 query columns held by the lanes of each half (by halves: the selection of a long prompt decides
    // near-ties on a score's last bits, so the order stays as it is), then the groups that shared the tiles
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float v = half_wave_sum(acc[r]);
      if (m == 0) cs[qw][kw * 32 + (r >> 2) * 8 + h * 4 + (r & 3)] = v;
    }
    __syncthreads();
    double c1 = 0.0, c2 = 0.0;
    if (tid < BN && kb0 + tid < n) {
      float c = cs[0][tid];
#pragma unroll
      for (int i = 1; i < QW; ++i) c += cs[i][tid];
      colsum[(int64_t(b) * Hq + hq) * npad + kb0 + tid] = c;
      c1 = double(c);
      c2 = double(c) * double(c);
    }
    // partial sums per 128-key block (the unit the density reduction adds up): two wavefronts' keys each
    c1 = fast_wave_sum(c1);
    c2 = fast_wave_sum(c2);
    if (lane == 0) {
      red[w][0] = c1;
      red[w][1] = c2;
    }
    __syncthreads();
    if (tid < BN / 128 && kb0 + 128 * tid < npad) {
      double* vp = varpart + ((int64_t(b) * Hq + hq) * (npad / 128) + tile * (BN / 128) + tid) * 2;
      vp[0] = red[2 * tid][0] + red[2 * tid + 1][0];
      vp[1] = red[2 * tid][1] + red[2 * tid + 1][1];
    }
  }
}

template <int KW, int QW, int TQ>
void run_colsum(d2o_ctx* c, View Q, View K, float* colsum, int n, bool paired, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const int nblk = (n + 32 * KW - 1) / (32 * KW);
  colsum_bf16<KW, QW, TQ><<<dim3(paired ? (nblk + 1) / 2 : nblk, cf.n_q_heads, cf.batch), 64 * KW * QW, 0, s>>>(
      (const uint16_t*)Q.ptr, Q, (const uint16_t*)K.ptr, K, c->lse, colsum, c->varpart, n, c->npad, cf.n_q_heads / cf.n_kv_heads,
      nblk, paired ? 1 : 0);
}

template <int NW>
hipError_t run_attn(d2o_ctx* c, View Q, View K, View O, int n, bool paired, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  constexpr int BM = 32 * kAttnRW * NW;
  const int nblk = (n + BM - 1) / BM;
  // the attribute is per device; setting it is a cheap host-side call, so it is not cached
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_fwd_bf16<kAttnRW, NW>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kAttnSmemBytes);
  if (e != hipSuccess) return e;
  attn_fwd_bf16<kAttnRW, NW><<<dim3(paired ? (nblk + 1) / 2 : nblk, cf.n_q_heads, cf.batch), 64 * NW, kAttnSmemBytes, s>>>(
      (const uint16_t*)Q.ptr, Q, (const uint16_t*)K.ptr, K, (const uint16_t*)c->vt, c->vt_unscale, O.ptr, O, c->lse, n,
      c->npad, cf.n_q_heads / cf.n_kv_heads, cf.out_f32, nblk, paired ? 1 : 0);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_bf16(d2o_ctx* c, int layer, View Q, View K, View V, View O, int n, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const int G = cf.n_q_heads / cf.n_kv_heads;
  float* score = c->score_pre + size_t(layer) * cf.batch * cf.n_kv_heads * c->npad;
  const int shares = std::min(kVmaxShares, (n * 16 + 255) / 256);
  vabsmax_kernel<<<dim3(shares, cf.n_kv_heads, cf.batch), 256, 0, s>>>((const uint16_t*)V.ptr, V, c->vmax_bits, n);
  transpose_v<<<dim3(c->npad / 64, cf.n_kv_heads, cf.batch), 256, 0, s>>>((const uint16_t*)V.ptr, V, (uint16_t*)c->vt,
                                                                         c->vmax_bits, c->vt_unscale, n, c->npad, shares);
  {
    KernelTimer kt(c, D2O_K_ATTN_FWD, s);
    // Row blocks of 256, two per workgroup (a long and a short one); where there are so few rows that the chip holds
    // all blocks of 128, a workgroup each and two per CU, those: the longest block then takes half as long.
    // (32 heads: 1000 tokens 51 -> 35 us, 2048 tokens 79 -> 68; 8 heads, 500 tokens 36 -> 21; 16 heads, 2900 tokens
    // 100 -> 83; 2 heads, 24000 tokens 638 -> 623, 30000 tokens 771 -> 786.)
    const bool few = int64_t((n + 127) / 128) * cf.n_q_heads * cf.batch <= 512;
    const hipError_t e = few ? run_attn<4>(c, Q, K, O, n, false, s) : run_attn<8>(c, Q, K, O, n, true, s);
    if (e != hipSuccess) return e;
  }
  KernelTimer kt(c, D2O_K_COLSUM, s);
  // with several query heads per KV head the column sums of each go to c->colpart; launch_density adds them up
  float* colsum = G == 1 ? score : c->colpart;
  // 256 keys per workgroup, eight wavefronts, where such workgroups fill the chip (two fit a CU); below, half as
  // many keys, the eight wavefronts sharing them and the tile's queries, and a block per workgroup instead
  // of two where there is a CU for each.  (32 heads: 1000 tokens 41, 25 and 21 us; 2048 tokens 61, 38 and 37; 4096 tokens
  // 118, 118; 8192 tokens 325, 374; 8 heads of 16384 tokens 386, 377; 4 heads of 14000 tokens 173 in pairs, 183 singly.)
  if (int64_t((n + 511) / 512) * cf.n_q_heads * cf.batch < 512) {
    const bool paired = int64_t((n + 127) / 128) * cf.n_q_heads * cf.batch > 256;
    // Tiles of 128 queries, a barrier for twice the products, where a workgroup has its CU alone or many tiles (4 heads
    // of 14000 tokens 174 -> 158 us, 16 of 4096 62 -> 57, 40 of 1500 29 -> 27.5, 32 of 4096 106 -> 98, 64 of 2048 59 -> 57.5);
    // two workgroups per CU with few tiles hide each other's barriers (256 heads of 500 tokens 25 -> 29, 128 of 1024 33.5 -> 34.4).
    const int64_t workgroups = (paired ? (n + 255) / 256 : (n + 127) / 128) * int64_t(cf.n_q_heads) * cf.batch;
    if (workgroups <= 256 || n >= 2048)
      run_colsum<4, 2, 128>(c, Q, K, colsum, n, paired, s);
    else
      run_colsum<4, 2, 64>(c, Q, K, colsum, n, paired, s);
  } else {  // (in tiles of 128: 32 heads of 32768 tokens 4.21 -> 4.15 ms, 128 of 2048 85 -> 88 us, 256 of 700 38 -> 44)
    run_colsum<8, 1, 64>(c, Q, K, colsum, n, true, s);
  }
  return hipGetLastError();
}

}  // namespace d2o
