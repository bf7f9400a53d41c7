// Token-level operation after prompt encoding (Sec. 4.2): selection (Eq. 7-8), compaction into
// the cache, nearest-neighbour matching (Eq. 9), the initial threshold (Eq. 10, t = 0) and the
// similarity-weighted merge (Eq. 11-12).
//
// Every decision (top-N membership, arg-max of the cosine, threshold test) is taken on exact
// integer keys or in fp64 with the operation order of the defining formulas, so that index
// outputs do not depend on reduction shapes; the bf16 matrix-core product in match_filter_bf16
// only pre-selects candidates and flags rows whose two best candidates are too close for fp32.
#include "d2o_internal.h"
#include "decode_common.h"
#include "device_utils.h"

namespace d2o {
namespace {

// ------------------------------------------------------------------------------------------
// Selection.  One workgroup per (sequence, KV head).  Radix-select of the N_hh-th largest
// score among positions [T, n-M) on order-preserving 32-bit keys, then an ordered compaction
// that keeps, among keys equal to the threshold, the lowest positions first.

__device__ __forceinline__ uint32_t order_key(float x) {
  if (x == 0.f) x = 0.f;  // -0 and +0 compare equal
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ uint64_t order_key(double x) {
  if (x == 0.0) x = 0.0;
  const uint64_t b = uint64_t(__double_as_longlong(x));
  return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}

// Exclusive prefix sums of one integer per thread over the block, in thread order, and the
// block total (read by all threads).
__device__ __forceinline__ void block_scan_int(int v, int& ex, int& tot, int* wa) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  __syncthreads();
  if (lane == 63) wa[w] = inc;
  __syncthreads();
  int off = 0, total = 0;
  for (int i = 0; i < nw; ++i) {
    if (i < w) off += wa[i];
    total += wa[i];
  }
  ex = off + inc - v;
  tot = total;
}

// S: score type (fp32 column sums after prompt encoding; fp64 cumulative scores of a cache that a
// block of tokens was appended to).  nvec, when given, holds the number of entries per head.
// PACKED: the layer's geometry comes with the launch; it goes to `meta` (and, fp8 cache, with row 0 as every head's
// start to `stage`) here, where a launch of its own cost 3 us.
template <typename S, bool PACKED>
__global__ __launch_bounds__(1024) void select_kernel(const S* __restrict__ score, MetaPack pack, int32_t* __restrict__ meta,
                                                      int32_t* __restrict__ stage, int32_t* __restrict__ amb_cnt,
                                                      int32_t* __restrict__ ret, int32_t* __restrict__ evi,
                                                      int32_t* __restrict__ cnt, int n_all, const int32_t* __restrict__ nvec,
                                                      int npad, int n_sink) {
  typedef decltype(order_key(S())) Key;
  constexpr int kTopShift = int(sizeof(Key)) * 8 - 8;
  __shared__ int hist[256];
  __shared__ int wa[16];
  __shared__ Key sh_prefix;
  __shared__ int sh_need;
  const int hk = blockIdx.x, b = blockIdx.y, Hkv = gridDim.x;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int n = nvec ? nvec[bh] : n_all;
  const S* sc = score + bh * npad;
  int32_t* r = ret + bh * npad;
  int32_t* e = evi + bh * npad;
  const int tid = threadIdx.x;
  if (PACKED && tid < 4) {
    meta[bh * 4 + tid] = pack.v[bh * 4 + tid];
    if (stage) stage[bh * 4 + tid] = tid == 0 ? 0 : pack.v[bh * 4 + tid];
  }
  if (tid == 0) amb_cnt[bh] = 0;  // (counted up by match_filter_bf16)
  const int budget = PACKED ? pack.v[bh * 4 + 1] : meta[bh * 4 + 1], recent = PACKED ? pack.v[bh * 4 + 2] : meta[bh * 4 + 2];
  if (budget >= n) {
    for (int j = tid; j < n; j += blockDim.x) r[j] = j;
    if (tid == 0) {
      cnt[bh * 2] = n;
      cnt[bh * 2 + 1] = 0;
    }
    return;
  }
  const int lo = n_sink, hi = n - recent;   // middle range [lo, hi)
  const int nhh = budget - n_sink - recent;  // heavy hitters to keep, 0 <= nhh < hi - lo
  // ---- radix select: find the key value of the nhh-th largest and how many equal keys to take
  Key prefix = 0, mask = 0;
  int need = nhh;
  if (nhh > 0) {
    for (int shift = kTopShift; shift >= 0; shift -= 8) {
      for (int i = tid; i < 256; i += blockDim.x) hist[i] = 0;
      __syncthreads();
      for (int j = lo + tid; j < hi; j += blockDim.x) {
        const Key k = order_key(sc[j]);
        if ((k & mask) == prefix) atomicAdd(&hist[int(k >> shift) & 255], 1);
      }
      __syncthreads();
      if (tid < 64) {
        // the highest bin at which the count of keys in this and all higher bins reaches `need`
        // (it exists: the candidates number at least `need`): lane i holds the bins 255 - 4 i
        // down to 252 - 4 i, and a scan over the lanes counts the keys above them
        const int b0 = 255 - 4 * tid;
        const int h0 = hist[b0], h1 = hist[b0 - 1], h2 = hist[b0 - 2], h3 = hist[b0 - 3];
        const int tot = h0 + h1 + h2 + h3;
        int inc = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int v = __shfl_up(inc, o, 64);
          if (tid >= o) inc += v;
        }
        const int above = inc - tot;
        if (above < need && need <= inc) {
          int rem = need - above, bin = b0;
          if (h0 < rem) {
            rem -= h0;
            bin = b0 - 1;
            if (h1 < rem) {
              rem -= h1;
              bin = b0 - 2;
              if (h2 < rem) {
                rem -= h2;
                bin = b0 - 3;
              }
            }
          }
          sh_prefix = prefix | (Key(bin) << shift);
          sh_need = rem;
        }
      }
      __syncthreads();
      prefix = sh_prefix;
      need = sh_need;
      mask |= Key(0xFF) << shift;
      __syncthreads();
    }
  }
  // prefix = threshold key; `need` of the keys equal to it are kept, lowest positions first.
  // Ordered compaction, four consecutive positions per thread and round: two block-wide scans
  // (ties, then kept entries) per 4096 positions.
  constexpr int PT = 4;
  int base_keep = 0, base_eq = 0;
  for (int j0 = 0; j0 < n; j0 += PT * blockDim.x) {
    const int jt = j0 + PT * tid;
    bool keep[PT], eq[PT];
    int neq = 0;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      const int j = jt + u;
      keep[u] = false;
      eq[u] = false;
      if (j < n) {
        if (j < lo || j >= hi) {
          keep[u] = true;
        } else if (nhh > 0) {
          const Key k = order_key(sc[j]);
          keep[u] = k > prefix;
          eq[u] = k == prefix;
        }
      }
      neq += eq[u] ? 1 : 0;
    }
    int ex_eq, tot_eq;
    block_scan_int(neq, ex_eq, tot_eq, wa);
    int nkeep = 0, seen_eq = base_eq + ex_eq;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      if (eq[u]) {
        if (seen_eq < need) keep[u] = true;
        ++seen_eq;
      }
      nkeep += keep[u] ? 1 : 0;
    }
    int ex_keep, tot_keep;
    block_scan_int(nkeep, ex_keep, tot_keep, wa);
    int kept = base_keep + ex_keep;  // kept entries before position jt + u
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      const int j = jt + u;
      if (j < n) {
        if (keep[u])
          r[kept] = j;
        else
          e[j - kept] = j;
      }
      kept += keep[u] ? 1 : 0;
    }
    base_keep += tot_keep;
    base_eq += tot_eq;
  }
  if (tid == 0) {
    cnt[bh * 2] = base_keep;
    cnt[bh * 2 + 1] = n - base_keep;
  }
}

// 1/|k| in fp32 from the squares' sum (used by the bf16 candidate filter only), and a 16-byte share of that sum.
__device__ __forceinline__ float inverse_norm(float s) { return s > 0.f ? 1.0f / sqrtf(s) : 0.f; }
__device__ __forceinline__ float add_squares(const u32x4& v, float s) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = __uint_as_float(v[i] << 16), hi = __uint_as_float(v[i] & 0xFFFF0000u);
    s = fmaf(lo, lo, s);
    s = fmaf(hi, hi, s);
  }
  return s;
}

// ------------------------------------------------------------------------------------------
// Compaction: retained rows of K, V into the layer's cache region; scores widen to fp64.
// APPEND: the source is the position-ordered copy of a cache: fp64 scores (sc64) and token
// positions (apos) indexed like its rows.  bf16: a retained key's inverse norm, by its rank, on the way (the filter takes
// the evicted keys' from the rows that it holds; a pass over all keys here was most of this kernel's time).
template <typename T, bool APPEND>
__global__ __launch_bounds__(256) void gather_kernel(const T* __restrict__ K, View kv, const T* __restrict__ V, View vv,
                                                     const float* __restrict__ score, const double* __restrict__ sc64,
                                                     const int32_t* __restrict__ apos, const int32_t* __restrict__ ret,
                                                     const int32_t* __restrict__ cnt, const int32_t* __restrict__ meta,
                                                     T* __restrict__ cK, T* __restrict__ cV, double* __restrict__ cscore,
                                                     int32_t* __restrict__ cpos, int32_t* __restrict__ ccount,
                                                     int npad, int d, int64_t slots, const int32_t* __restrict__ row_meta,
                                                     int64_t row_slots, float* __restrict__ invn) {
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int nret = cnt[bh * 2];
  constexpr int kVec = 16 / sizeof(T);
  const int tpr = d / kVec;                 // threads per row
  const int rows_per_blk = 256 / tpr;
  const int slot = blockIdx.x * rows_per_blk + threadIdx.x / tpr;
  if (blockIdx.x == 0 && threadIdx.x == 0) ccount[bh] = nret;
  if (slot >= nret) return;
  const int c = (threadIdx.x % tpr) * kVec;
  const int pos = ret[bh * npad + slot];
  const int64_t dst = (bh * slots + meta[bh * 4 + 0] + slot);
  // (the rows may live elsewhere than scores and positions: the bf16 staging rows of an fp8 cache)
  const int64_t dst_row = (bh * row_slots + row_meta[bh * 4 + 0] + slot);
  const u32x4 k16 = *reinterpret_cast<const u32x4*>(K + b * kv.sb + hk * kv.sh + int64_t(pos) * kv.sn + c);
  const u32x4 v16 = *reinterpret_cast<const u32x4*>(V + b * vv.sb + hk * vv.sh + int64_t(pos) * vv.sn + c);
  *reinterpret_cast<u32x4*>(cK + dst_row * d + c) = k16;
  *reinterpret_cast<u32x4*>(cV + dst_row * d + c) = v16;
  if constexpr (sizeof(T) == 2) {  // (head_dim 128: sixteen lanes per row, all of them here or none)
    float sq = add_squares(k16, 0.f);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (c == 0) invn[bh * npad + slot] = inverse_norm(sq);
  }
  if (c == 0) {
    cscore[dst] = APPEND ? sc64[bh * npad + pos] : double(score[bh * npad + pos]);
    cpos[dst] = APPEND ? apos[bh * npad + pos] : pos;
  }
}

// ------------------------------------------------------------------------------------------
// Matching.

// Candidate filter on the matrix cores.  A workgroup owns 128 evicted rows (4 wavefronts x 32,
// the stationary B operand) and streams the retained keys, read contiguously from the cache
// region they were compacted into, in double-buffered tiles of 64 through LDS (the A operand),
// so each lane owns one evicted row and sees 16 retained keys per MFMA tile.
//   COLLECT = false: per row, track the best and second-best fp32 cosine and the best's
//     retained rank.  A row whose two best values differ by less than kAmbiguous is flagged and
//     its acceptance threshold (best - kAmbiguous, in the un-normalised domain) is stored.
//   COLLECT = true: second sweep over the flagged rows only (a list in no particular order; the rows are
//     independent of each other): every retained
//     key whose fp32 cosine reaches the row's threshold is appended to the row's candidate
//     list (up to kMaxCand; more than that falls back to the exhaustive search).  The sweep
//     repeats the first one's arithmetic exactly, so the best value is found again.  Few rows are
//     flagged (a workgroup or two per head), so the retained keys are split over `ksplit`
//     workgroups per row block: the lists are appended with atomics and read order-free.
// The filter is bound by the vector ALU (68 instructions per 32 x 32 sub-tile and wavefront beside 8 products), as
// long as no wavefront waits for LDS: with the operands and inverse norms requested half a sub-tile ahead and the
// padding confined to the last tile, at four wavefronts per SIMD, 940 -> 867 us (32768 tokens, 32 heads, a tenth
// kept), 37 -> 34 (4096, a fifth), 54 -> 41 (256 of 2304 rows leave).
// kAmbiguous bounds twice the error of one filtered cosine: at most one rounding per accumulated
// product (128 * 2^-24 of |k_i||k_j|) plus the two fp32 inverse norms, 1.6e-5 in total, plus the
// four mantissa bits that carry the register number (2 * 16 * 2^-24 = 1.9e-6).
constexpr float kAmbiguous = 2.4e-5f;
constexpr int kMaxCand = 8;
constexpr int kLdM = 128 + 8;

// Best and second-best value of a lane's evicted row, two operations per value: the low four
// mantissa bits of a value are replaced by its register number (a change of at most 16
// units in the last place, which kAmbiguous covers), so that the maximum carries the
// position inside the sub-tile with it; which sub-tile it came from is noted once per
// sub-tile.  Values that are equal up to those bits end up flagged as ambiguous and are
// decided by the exact refinement.
struct BestTwo {
  float m1 = -INFINITY, m2 = -INFINITY;
  int isub = 0;  // first retained rank of the sub-tile the best came from
  __device__ __forceinline__ void take(const float (&tv)[16], int first) {
    const float before = m1;
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
      float key[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) key[i] = __uint_as_float((__float_as_uint(tv[r + i]) & ~15u) | uint32_t(r + i));
      // (the maximum as the instruction itself: fmaxf would first re-canonicalise a value that was put
      // together from bits; and in pairs: apart, the compiler runs all maxima first and keeps them)
      asm("v_med3_f32 %1, %0, %1, %2\n\tv_max_f32 %0, %0, %2\n\t"
          "v_med3_f32 %1, %0, %1, %3\n\tv_max_f32 %0, %0, %3\n\t"
          "v_med3_f32 %1, %0, %1, %4\n\tv_max_f32 %0, %0, %4\n\t"
          "v_med3_f32 %1, %0, %1, %5\n\tv_max_f32 %0, %0, %5"
          : "+&v"(m1), "+&v"(m2)
          : "v"(key[0]), "v"(key[1]), "v"(key[2]), "v"(key[3]));
    }
    isub = (m1 != before) ? first : isub;
  }
  // the best's retained rank: its sub-tile, and the register number carried in its low bits (h: the lane's half)
  __device__ __forceinline__ int rank(int h) const {
    const int r = int(__float_as_uint(m1) & 15u);
    return isub + (r >> 2) * 8 + h * 4 + (r & 3);
  }
};

// Adds another candidate for best, of retained rank oi, and its second to (best, second, bi).
__device__ __forceinline__ void join_best(float& best, float& second, int& bi, float om1, float om2, int oi) {
  second = fmaxf(fminf(best, om1), fmaxf(second, om2));
  bi = (om1 > best) ? oi : bi;
  best = fmaxf(best, om1);
}

// The inverse norm of an evicted key from the operands of its two lanes.
__device__ __forceinline__ float evicted_norm(const bf16x8 (&be)[8]) {
  float s = 0.f;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) s = add_squares(__builtin_bit_cast(u32x4, be[ks]), s);
  return inverse_norm(s + __shfl_xor(s, 32, 64));
}

// A row's candidate, its threshold for the second sweep, and the list of ambiguous rows.  ie: the row's inverse norm.
__device__ __forceinline__ void note_row(float best, float second, int bi, float ie, int erank, int64_t base, int64_t bh,
                                         int32_t* cand, float* thr, int32_t* amb_list, int32_t* amb_cnt, int32_t* ncand) {
  const float margin = ie > 0.f ? kAmbiguous / ie : INFINITY;  // threshold in the un-normalised domain
  const bool amb = !(best - second >= margin);                // also true for NaN / equal / zero norm
  cand[base + erank] = bi | (amb ? int(0x80000000u) : 0);
  thr[base + erank] = best - margin;
  if (amb) {
    amb_list[base + atomicAdd(&amb_cnt[bh], 1)] = erank;
    ncand[base + erank] = 0;
  }
}

template <bool COLLECT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(COLLECT ? 3 : 4, 4))) void match_filter_bf16(const uint16_t* __restrict__ K, View kv,
                                                         const uint16_t* __restrict__ cK,
                                                         const int32_t* __restrict__ meta, int64_t slots,
                                                         const float* __restrict__ invn,
                                                         const int32_t* __restrict__ evi,
                                                         const int32_t* __restrict__ cnt, int32_t* __restrict__ cand,
                                                         float* __restrict__ thr, int32_t* __restrict__ amb_list,
                                                         int32_t* __restrict__ amb_cnt,
                                                         int32_t* __restrict__ ncand, int32_t* __restrict__ clist,
                                                         int npad, int ksplit) {
  constexpr int kTile = 64;     // retained keys per LDS tile
  constexpr int NCH = kTile * 16 / 256;  // 16-byte chunks of a tile per thread
  __shared__ __attribute__((aligned(16))) uint16_t Rs[2][kTile * kLdM];
  __shared__ __attribute__((aligned(16))) float rin[2][kTile];    // 1/|k| of the staged retained keys
  __shared__ __attribute__((aligned(16))) float rbias[2][kTile];  // 0, or -3e38 for padding rows (finite: the low
                                                                  // mantissa bits of a value get overwritten below)
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int nret = cnt[bh * 2], nevi = cnt[bh * 2 + 1];
  const int nrows = COLLECT ? amb_cnt[bh] : nevi;
  const int e0 = (int(blockIdx.x) / ksplit) * 128, part = int(blockIdx.x) % ksplit;
  if (e0 >= nrows) return;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 31, h = lane >> 5;
  const uint16_t* kb = K + b * kv.sb + hk * kv.sh;
  // the retained keys, in retained order, already sit contiguously in the layer's cache
  // region (compaction runs first; merging, which changes them, runs after the matching)
  const uint16_t* rk = cK + (bh * slots + meta[bh * 4 + 0]) * 128;
  const int32_t* el = evi + bh * npad;
  const float* inl = invn + bh * npad;  // by retained rank
  const int row = e0 + w * 32 + m;
  const bool live = row < nrows;
  const int erank = COLLECT ? amb_list[bh * npad + min(row, nrows - 1)] : min(row, nrows - 1);
  const int epos = el[erank];
  bf16x8 be[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    be[ks] = *reinterpret_cast<const bf16x8*>(kb + int64_t(epos) * kv.sn + ks * 16 + h * 8);
  BestTwo two;
  const float mythr = COLLECT ? thr[bh * npad + erank] : 0.f;
  // Tiles travel global -> registers -> LDS: the next tile is requested when work on a tile
  // starts and written to the other LDS buffer when it ends.
  u32x4 rg[NCH];
  float rv = 0.f;
  const int ntile = (nret + kTile - 1) / kTile;
  const int tper = (ntile + ksplit - 1) / ksplit;
  const int tbeg = part * tper, tend = min(ntile, tbeg + tper);  // this workgroup's tiles
  if (tbeg >= tend) return;
  const int tfull = min(tend, nret / kTile);  // the first tile that is not full
  auto issue = [&](int t) {
    const int r0 = t * kTile;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + 256 * i, rrow = c >> 4, col = (c & 15) * 8;
      rg[i] = *reinterpret_cast<const u32x4*>(rk + int64_t(min(r0 + rrow, nret - 1)) * 128 + col);
    }
    if (tid < kTile) rv = (r0 + tid < nret) ? inl[r0 + tid] : -1.f;  // -1 marks a padding row
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = tid + 256 * i, rrow = c >> 4, col = (c & 15) * 8;
      *reinterpret_cast<u32x4*>(&Rs[buf][rrow * kLdM + col]) = rg[i];
    }
    if (tid < kTile) {
      rin[buf][tid] = rv < 0.f ? 0.f : rv;
      rbias[buf][tid] = rv < 0.f ? -3.0e38f : 0.f;
    }
  };
  auto one_tile = [&](int t, auto last) {  // `last`: the tile that may hold rows past the end
    constexpr bool padded = decltype(last)::value;
    const int buf = t & 1, r0 = t * kTile;
    if (t + 1 < tend) issue(t + 1);
    auto operand = [&](int st, int ks) {
      return *reinterpret_cast<const bf16x8*>(&Rs[buf][(st * 32 + m) * kLdM + ks * 16 + h * 8]);
    };
    bf16x8 a[4];
    f32x4 ri[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a[ks] = operand(0, ks);
    // The operands of the second four products arrive during the first four, those of the next sub-tile's first
    // four and the inverse norms during the second four.
    auto mma = [&](int st) -> f32x16 {
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      f32x16 s = zero;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks & 3], be[ks], s, 0, 0, 0);
        if (ks < 4)
          a[ks] = operand(st, ks + 4);
        else if (st == 0)
          a[ks & 3] = operand(1, ks & 3);
        if (ks >= 4) ri[ks & 3] = *reinterpret_cast<const f32x4*>(&rin[buf][st * 32 + (ks & 3) * 8 + h * 4]);
        __builtin_amdgcn_sched_barrier(0);
      }
      return s;
    };
    auto post = [&](const f32x16& s, int st) {
      // register r: retained row st*32 + (r/4)*8 + 4h + r%4 of this tile, evicted row = lane's;
      // the four rows of a register group are neighbours, so their 1/|k| came in one LDS read
      float tv[16];
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int rb = st * 32 + g4 * 8 + h * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) tv[g4 * 4 + i] = s[g4 * 4 + i] * ri[g4][i];
        if (padded) {
          const f32x4 bi = *reinterpret_cast<const f32x4*>(&rbias[buf][rb]);
#pragma unroll
          for (int i = 0; i < 4; ++i) tv[g4 * 4 + i] += bi[i];
        }
      }
      if (COLLECT) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int rr = st * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
          if (live && tv[r] >= mythr) {
            const int k = atomicAdd(&ncand[bh * npad + erank], 1);
            if (k < kMaxCand) clist[(bh * npad + erank) * kMaxCand + k] = r0 + rr;
          }
        }
      } else {
        two.take(tv, r0 + st * 32);
      }
    };
    // (two sub-tiles as two independent accumulation chains need 160 registers and cost a
    // wavefront per SIMD: slower)
    post(mma(0), 0);
    if (!padded || nret - r0 > 32) post(mma(1), 1);
    if (t + 1 < tend) stage(buf ^ 1);
    __syncthreads();
  };
  issue(tbeg);
  stage(tbeg & 1);
  __syncthreads();
#pragma unroll 1
  for (int t = tbeg; t < tfull; ++t) one_tile(t, std::false_type{});
  if (tfull < tend) one_tile(tfull, std::true_type{});
  if (COLLECT) return;
  // combine the two lane halves that share an evicted row
  float best = two.m1, second = two.m2;
  int bi = two.rank(h);
  join_best(best, second, bi, __shfl_xor(best, 32, 64), __shfl_xor(second, 32, 64), __shfl_xor(bi, 32, 64));
  const float ie = evicted_norm(be);
  if (h == 0 && live) note_row(best, second, bi, ie, erank, bh * npad, bh, cand, thr, amb_list, amb_cnt, ncand);
}

// The first sweep for launches of few rows: 32 evicted rows per workgroup, whose wavefronts take the 32-key sub-tiles
// in turn, operands and inverse norms straight from memory one sub-tile ahead (no wavefront shares
// them, so LDS would only add a barrier per tile), and join their best two at the end.  Same values, in
// the same order of products.  Bound by the operands' way from the L2, which every 32 rows take (eight
// wavefronts instead of four: level).  A launch of few rows leaves most of the chip idle in blocks of 128: both
// sweeps of 32 heads, 256 rows against 2048 keys, 53 -> 37 us, 200 against 800 keys 29 -> 22; from two workgroups per
// CU on the blocks of 128, which read the keys a quarter as often, are the faster ones (512 rows against 128 keys 18.4
// where this takes 20.4, 800 against 200 18.5 where it takes 31).
constexpr int kFewWaves = 4;
__global__ __launch_bounds__(64 * kFewWaves) void match_filter_few(const uint16_t* __restrict__ K, View kv,
                                                                   const uint16_t* __restrict__ cK,
                                                                   const int32_t* __restrict__ meta, int64_t slots,
                                                                   const float* __restrict__ invn,
                                                                   const int32_t* __restrict__ evi,
                                                                   const int32_t* __restrict__ cnt,
                                                                   int32_t* __restrict__ cand, float* __restrict__ thr,
                                                                   int32_t* __restrict__ amb_list,
                                                                   int32_t* __restrict__ amb_cnt,
                                                                   int32_t* __restrict__ ncand, int npad) {
  __shared__ __attribute__((aligned(16))) float rin[kFewWaves][32];  // of the wavefront's sub-tile
  __shared__ float best_s[kFewWaves][32], second_s[kFewWaves][32];
  __shared__ int rank_s[kFewWaves][32];
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int nret = cnt[bh * 2], nevi = cnt[bh * 2 + 1];
  const int e0 = int(blockIdx.x) * 32;
  if (e0 >= nevi || nret == 0) return;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 31, h = lane >> 5;
  const uint16_t* rk = cK + (bh * slots + meta[bh * 4 + 0]) * 128;
  const float* inl = invn + bh * npad;  // by retained rank
  const int erank = min(e0 + m, nevi - 1);
  const int epos = evi[bh * npad + erank];
  const uint16_t* erow = K + b * kv.sb + hk * kv.sh + int64_t(epos) * kv.sn;
  bf16x8 be[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) be[ks] = *reinterpret_cast<const bf16x8*>(erow + ks * 16 + h * 8);
  const int nsub = (nret + 31) / 32;
  auto rank_of = [&](int j) { return min(j * 32 + m, nret - 1); };
  auto load = [&](bf16x8 (&a)[8], int j) {
    const uint16_t* row = rk + int64_t(rank_of(j)) * 128 + h * 8;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) a[ks] = *reinterpret_cast<const bf16x8*>(row + ks * 16);
  };
  BestTwo two;
  // a, norm: sub-tile j; a_next, norm_next: the wavefront's next one
  auto one = [&](int j, const bf16x8 (&a)[8], float norm, bf16x8 (&a_next)[8], float& norm_next) {
    if (h == 0) rin[w][m] = norm;
    // (within the wavefront; LDS serves its requests in order, so the hand-over needs compiler ordering only)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    load(a_next, j + kFewWaves);
    norm_next = inl[rank_of(j + kFewWaves)];
    f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], be[ks], s, 0, 0, 0);
    float tv[16];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const f32x4 ri = *reinterpret_cast<const f32x4*>(&rin[w][g4 * 8 + h * 4]);
#pragma unroll
      for (int i = 0; i < 4; ++i) tv[g4 * 4 + i] = s[g4 * 4 + i] * ri[i];
    }
    if (j * 32 + 32 > nret) {  // copies of the last row past the end: the lowest value, or NaN as the row itself
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (j * 32 + (r >> 2) * 8 + h * 4 + (r & 3) >= nret) tv[r] = s[r] * 0.f - 3.0e38f;
    }
    two.take(tv, j * 32);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  bf16x8 a0[8], a1[8];
  float n0 = 0.f, n1 = 0.f;
  if (w < nsub) {
    load(a0, w);
    n0 = inl[rank_of(w)];
#pragma unroll 1
    for (int j = w; j < nsub; j += 2 * kFewWaves) {
      one(j, a0, n0, a1, n1);
      if (j + kFewWaves < nsub) one(j + kFewWaves, a1, n1, a0, n0);
    }
  }
  float best = two.m1, second = two.m2;
  int bi = two.rank(h);
  join_best(best, second, bi, __shfl_xor(best, 32, 64), __shfl_xor(second, 32, 64), __shfl_xor(bi, 32, 64));
  const float ie = evicted_norm(be);
  if (h == 0) {
    best_s[w][m] = best;
    second_s[w][m] = second;
    rank_s[w][m] = bi;
  }
  __syncthreads();
  if (tid < 32 && e0 + tid < nevi) {
#pragma unroll
    for (int u = 1; u < kFewWaves; ++u) join_best(best, second, bi, best_s[u][tid], second_s[u][tid], rank_s[u][tid]);
    note_row(best, second, bi, ie, erank, bh * npad, bh, cand, thr, amb_list, amb_cnt, ncand);
  }
}

// Exact similarity in fp64, operation order of Eq. 9 as written: dot / (|k_i| * |k_j|), 0 when
// a norm is 0.  A group of 16 lanes (one 16-byte slice of the key each) serves one evicted row:
// unambiguous rows evaluate their single candidate, ambiguous rows their short candidate list;
// rows without a usable list (and every row when no filter ran) are then searched exhaustively,
// one at a time, with the wavefront's lanes striding over the retained keys, first maximum in
// ascending retained order.  Products of bf16 values are exact in fp64 and their sums stay
// exact at these magnitudes, so the result does not depend on the summation tree.
template <typename T>
__device__ __forceinline__ void load8(const T* p, double* out);
template <>
__device__ __forceinline__ void load8<uint16_t>(const uint16_t* p, double* out) {
  const u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[2 * i] = double(__uint_as_float(v[i] << 16));
    out[2 * i + 1] = double(__uint_as_float(v[i] & 0xFFFF0000u));
  }
}
template <>
__device__ __forceinline__ void load8<float>(const float* p, double* out) {  // 16 bytes: 4 elements
  const float4 a = reinterpret_cast<const float4*>(p)[0];
  out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
}

// Lanes of one row group (TPR lanes: 16, or 32 for 512-byte rows) add their partial sums.
template <int TPR>
__device__ __forceinline__ double group_sum(double v) {
  v = row16_sum(v);
  if constexpr (TPR == 32) v += __shfl_xor(v, 16, 64);
  return v;
}

template <typename T, int D>
__host__ __device__ constexpr int refine_rows_per_wave() {
  return sizeof(T) == 2 ? 64 / (D * int(sizeof(T)) / 16) : 1;
}
template <typename T, int D>
__global__ __launch_bounds__(256) void match_refine(const T* __restrict__ K, View kv, const int32_t* __restrict__ ret,
                                                    const int32_t* __restrict__ evi, const int32_t* __restrict__ cnt,
                                                    const int32_t* __restrict__ cand, const int32_t* __restrict__ ncand,
                                                    const int32_t* __restrict__ clist, double* __restrict__ ustar,
                                                    int32_t* __restrict__ tgt, int npad, int use_filter) {
  constexpr int kVec = 16 / sizeof(T);  // elements per 16-byte load
  constexpr int TPR = D / kVec;         // lanes that share one evicted row
  // evicted rows per wavefront; fp32 rows are all searched exhaustively, by the whole wavefront one after
  // the other, so a wavefront takes one (with four, 512 tokens and 4 heads were 96 wavefronts: 20 us, now 12 us)
  constexpr int RW = refine_rows_per_wave<T, D>();
  __shared__ double ke[4][D];
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int nret = cnt[bh * 2], nevi = cnt[bh * 2 + 1];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, grp = lane / TPR, tc = lane % TPR;
  if (int(blockIdx.x) * 4 * RW >= nevi) return;  // block-uniform
  const int erank_raw = (blockIdx.x * 4 + w) * RW + grp % RW;
  const bool valid = erank_raw < nevi && grp < RW;
  const int erank = min(erank_raw, nevi - 1);
  const T* kb = K + b * kv.sb + hk * kv.sh;
  const int32_t* rl = ret + bh * npad;
  const int epos = evi[bh * npad + erank];
  // this lane's slice of the evicted key
  double x[kVec];
  load8<T>(kb + int64_t(epos) * kv.sn + tc * kVec, x);
  double ne = 0.0;
#pragma unroll
  for (int e = 0; e < kVec; ++e) ne = fma(x[e], x[e], ne);
  const double sne = sqrt(group_sum<TPR>(ne));
  // candidates: one (unambiguous), a short list (ambiguous), or every retained key (ncd < 0)
  int ncd = -1, single = -1;
  const int32_t* cl = clist + (bh * npad + erank) * kMaxCand;
  if (use_filter) {
    const int cnd = cand[bh * npad + erank];
    if (cnd >= 0) {
      single = cnd;
      ncd = 1;
    } else {
      ncd = ncand[bh * npad + erank];
      if (ncd > kMaxCand || ncd == 0) ncd = -1;  // overflow (or zero-norm row): exhaustive search
    }
  }
  double best = -2.0;
  int bj = 0x7FFFFFFF;
  // ---- listed candidates: the row group evaluates them one after the other
  int nloop = max(ncd, 0);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) nloop = max(nloop, __shfl_xor(nloop, o, 64));
  for (int q = 0; q < nloop; ++q) {
    const bool on = q < ncd;
    const int j = on ? (single >= 0 ? single : cl[q]) : 0;
    double y[kVec];
    load8<T>(kb + int64_t(rl[j]) * kv.sn + tc * kVec, y);
    double dot = 0.0, nr = 0.0;
#pragma unroll
    for (int e = 0; e < kVec; ++e) {
      dot = fma(x[e], y[e], dot);
      nr = fma(y[e], y[e], nr);
    }
    dot = group_sum<TPR>(dot);
    nr = group_sum<TPR>(nr);
    const double den = sne * sqrt(nr);
    const double u = den > 0.0 ? dot / den : 0.0;
    if (on && (u > best || (u == best && j < bj))) {
      best = u;
      bj = j;
    }
  }
  // ---- exhaustive search, one row at a time, the wavefront's lanes striding over the retained keys
  unsigned long long todo = __ballot(valid && ncd < 0 && tc == 0);
  while (todo) {
    const int src = __ffsll((long long)todo) - 1;  // first lane of the row group to serve
    todo &= todo - 1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane / TPR == src / TPR) {
#pragma unroll
      for (int e = 0; e < kVec; ++e) ke[w][tc * kVec + e] = x[e];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const double sne_r = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(sne), src),
                                          __builtin_amdgcn_readlane(__double2loint(sne), src));
    double fb = -2.0;
    int fj = 0x7FFFFFFF;
    for (int j = lane; j < nret; j += 64) {
      const T* rr = kb + int64_t(rl[j]) * kv.sn;
      double dot = 0.0, nr = 0.0;
      constexpr int kUnroll = sizeof(T) == 2 ? 1 : 4;
      // (bf16 rows come here as exceptions: unrolled, this loop's registers would halve the wavefronts
      // that the listed candidates above need in flight; fp32 rows always do)
#pragma unroll kUnroll
      for (int c = 0; c < D; c += kVec) {
        double y[kVec];
        load8<T>(rr + c, y);
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
          dot = fma(ke[w][c + i], y[i], dot);
          nr = fma(y[i], y[i], nr);
        }
      }
      const double den = sne_r * sqrt(nr);
      const double u = den > 0.0 ? dot / den : 0.0;
      if (u > fb) {  // j ascends within a lane: strict > keeps the first maximum
        fb = u;
        fj = j;
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ob = __shfl_xor(fb, o, 64);
      const int oj = __shfl_xor(fj, o, 64);
      if (ob > fb || (ob == fb && oj < fj)) {
        fb = ob;
        fj = oj;
      }
    }
    if (lane == src) {
      best = fb;
      bj = fj;
    }
  }
  if (tc == 0 && valid) {
    const bool none = bj == 0x7FFFFFFF;  // a non-finite key: no cosine compares above the start, and no threshold is reached
    ustar[bh * npad + erank] = none ? __longlong_as_double(0x7FF8000000000000ll) : best;
    tgt[bh * npad + erank] = none ? 0 : bj;
  }
}

// ------------------------------------------------------------------------------------------
// Threshold (Eq. 10, t = 0) and grouping of the passing tokens by target.  One workgroup per
// (sequence, KV head).  Group members are stored unordered; merge_kernel visits them in
// ascending evicted order.  One workgroup per head is a chain of memory round trips: the slots'
// counters live in LDS up to kGroupSlots retained tokens (as words in memory beyond), and a thread has
// four tokens in flight.  (One token at a time and counters in memory: 16.9 us at 32 heads x 4096
// tokens, 112 us at 32768; now 8.5 and 41 us.)
// The workgroups with z = 1 choose the eviction candidates of the next generation step meanwhile (they need
// the compacted scores only).
constexpr int kGroupSlots = 15360;  // 60 KB
struct FirstCandidates {  // the layer's arrays, [B][Hkv]
  const double* cscore;
  const int32_t *cpos, *ccount, *meta;
  int32_t* cand;
  int64_t slots;
  int new_pos, n_sink;
};
__global__ __launch_bounds__(1024) void threshold_group_kernel(const double* __restrict__ ustar,
                                                               const int32_t* __restrict__ tgt,
                                                               const int32_t* __restrict__ cnt, uint8_t* __restrict__ pass,
                                                               int32_t* __restrict__ gcnt, int32_t* __restrict__ goff,
                                                               int32_t* __restrict__ gcur, int32_t* __restrict__ gsrc,
                                                               double* __restrict__ tau_out, int npad, double tau_force,
                                                               int ema, double beta, FirstCandidates fc) {
  __shared__ double red[16];
  __shared__ int wa[16];
  __shared__ int slot_lds[kGroupSlots];  // counts of the slots' sources, then the places of their next ones
  const int hk = blockIdx.x, b = blockIdx.y, Hkv = gridDim.x;
  const int64_t bh = int64_t(b) * Hkv + hk;
  if (blockIdx.z == 1) {
    const int64_t slot0 = bh * fc.slots + fc.meta[bh * 4 + 0];
    dec::first_candidates<1024>(fc.cscore + slot0, fc.cpos + slot0, fc.ccount[bh], fc.meta[bh * 4 + 2], fc.new_pos, fc.n_sink,
                                fc.cand + bh * dec::kCand);
    return;
  }
  const int nret = cnt[bh * 2], nevi = cnt[bh * 2 + 1];
  const int tid = threadIdx.x;
  const bool in_lds = nret < kGroupSlots;
  const double* us = ustar + bh * npad;
  const int32_t* tg = tgt + bh * npad;
  uint8_t* ps = pass + bh * npad;
  int32_t* gc = gcnt + bh * (npad + 1);
  int32_t* go = goff + bh * (npad + 1);
  int32_t* gu = gcur + bh * (npad + 1);
  int32_t* gs = gsrc + bh * npad;
  if (nevi == 0) {
    // no sources anywhere: merge_kernel reads the offsets of every slot, so they must say so
    for (int j = tid; j <= nret; j += blockDim.x) go[j] = 0;
    return;  // tau keeps its value (unset, NaN, after prompt encoding)
  }
  double part = 0.0;
#pragma unroll 4
  for (int i = tid; i < nevi; i += 1024) part += us[i];
  double tau = block_sum(part, red) / double(nevi);
  if (ema) {  // a step that evicts several tokens at once: Eq. 10 on their mean best similarity
    const double prev = tau_out[bh];
    if (!isnan(prev)) tau = __dadd_rn(__dmul_rn(beta, tau), __dmul_rn(1.0 - beta, prev));
    __syncthreads();  // every thread has read the previous value
  }
  if (tid == 0 && !(ema && !isnan(tau_force))) tau_out[bh] = tau;  // (a forced threshold leaves the EMA state alone)
  const double thr = isnan(tau_force) ? tau : tau_force;
  for (int j = tid; j <= nret; j += 1024) {
    if (in_lds) {
      slot_lds[j] = 0;
    } else {
      gc[j] = 0;
      gu[j] = 0;
    }
  }
  __syncthreads();
  // four tokens in flight per thread: the loop waits for memory once for them
  auto each_token = [&](auto f) {
    for (int i0 = tid; i0 < nevi; i0 += 4 * 1024) {
      double u[4];
      int t[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        u[k] = us[min(i0 + k * 1024, nevi - 1)];
        t[k] = tg[min(i0 + k * 1024, nevi - 1)];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + k * 1024 < nevi) f(i0 + k * 1024, u[k] >= thr, t[k]);
    }
  };
  each_token([&](int i, bool ok, int t) {
    ps[i] = ok ? 1 : 0;
    if (ok) atomicAdd(in_lds ? &slot_lds[t] : &gc[t], 1);
  });
  __syncthreads();
  // exclusive prefix of the counts over [0, nret]
  int base = 0;
  for (int j0 = 0; j0 <= nret; j0 += blockDim.x) {
    const int j = j0 + tid;
    const int v = j < nret ? (in_lds ? slot_lds[j] : gc[j]) : 0;
    // inclusive scan within the wavefront
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o, 64);
      if ((tid & 63) >= o) inc += t;
    }
    __syncthreads();
    if ((tid & 63) == 63) wa[tid >> 6] = inc;
    __syncthreads();
    int woff = 0, tot = 0;
    for (int i = 0; i < int(blockDim.x >> 6); ++i) {
      if (i < (tid >> 6)) woff += wa[i];
      tot += wa[i];
    }
    if (j <= nret) {
      go[j] = base + woff + inc - v;
      if (in_lds) slot_lds[j] = base + woff + inc - v;
    }
    base += tot;
  }
  __syncthreads();
  each_token([&](int i, bool ok, int t) {
    if (!ok) return;
    if (in_lds)
      gs[atomicAdd(&slot_lds[t], 1)] = i;
    else
      gs[go[t] + atomicAdd(&gu[t], 1)] = i;
  });
}

// PER consecutive elements of a row as one load / one store.
template <typename T, int PER>
struct RowBits {
  static_assert(PER * sizeof(T) == 4 || PER * sizeof(T) == 8, "one 4- or 8-byte access");
  typedef typename std::conditional<PER * sizeof(T) == 4, uint32_t, uint64_t>::type type;
};
template <typename T, int PER>
__device__ __forceinline__ typename RowBits<T, PER>::type load_row_bits(const T* p) {
  return *reinterpret_cast<const typename RowBits<T, PER>::type*>(p);
}
template <typename T, int PER>
__device__ __forceinline__ void widen(typename RowBits<T, PER>::type raw, double* out) {
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if constexpr (sizeof(T) == 2)
      out[i] = Elem<T>::to_f64(T(raw >> (16 * i)));
    else
      out[i] = Elem<T>::to_f64(__uint_as_float(uint32_t(raw >> (32 * i))));
  }
}
template <typename T, int PER>
__device__ __forceinline__ void load_elems(const T* p, double* out) {
  widen<T, PER>(load_row_bits<T, PER>(p), out);
}
template <typename T, int PER>
__device__ __forceinline__ void store_elems(T* p, const double* v, double z) {
  T tmp[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) tmp[i] = Elem<T>::from_f64(v[i] / z);
  if constexpr (PER * sizeof(T) == 4)
    *reinterpret_cast<uint32_t*>(p) = *reinterpret_cast<const uint32_t*>(tmp);
  else
    *reinterpret_cast<uint64_t*>(p) = *reinterpret_cast<const uint64_t*>(tmp);
}

// Merge (Eq. 11-12).  One wavefront per retained slot that has sources; lane i owns elements
// PER*i .. PER*i + PER - 1 of the row.  fp64, operation order of the definition: acc = e * k_c;
// for each source in ascending evicted order: w = exp(u), Z += w, acc += w * k_e; result
// acc / Z rounded once to the cache dtype.  Products and sums are kept unfused so the sequence
// is the one written in the formula.
// The source list of a slot is unordered, and its length varies widely (the keys nearest to a
// cluster centre collect hundreds of sources; a small budget lengthens every list).
//   up to 64 sources      one source per lane: the lanes rank their sources (count the smaller
//                         ones), fetch weight and position in parallel;
//   up to kMergeCap       the same ranking through LDS, the sources stored at their ranks, and then
//                         64 of them at a time as above;
//   beyond                the next source is extracted by a scan per step.
// The rows are then read kMergeBatch sources at a time in rank order.  A list is a chain of dependent
// loads, so what counts is how many lists are in flight: 16 KB of LDS per workgroup and rows held as
// they were loaded (with weights and positions in LDS and rows widened on arrival it was 32 KB and
// five workgroups per CU: 34.7 us at 32 heads x 4096 tokens, now 24.6 us; 174 -> 114 us at 32768).
constexpr int kMergeCap = 512;
constexpr int kMergeBatch = 8;
template <typename T, int D, bool AVERAGE>
__global__ __launch_bounds__(256) void merge_kernel(const T* __restrict__ K, View kv, const T* __restrict__ V, View vv,
                                                    const int32_t* __restrict__ evi, const int32_t* __restrict__ cnt,
                                                    const double* __restrict__ ustar, const int32_t* __restrict__ goff,
                                                    const int32_t* __restrict__ gsrc, const int32_t* __restrict__ meta,
                                                    T* __restrict__ cK, T* __restrict__ cV, int npad, int64_t slots) {
  __shared__ int s_src[4][kMergeCap], s_sorted[4][kMergeCap];
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int slot = blockIdx.x * 4 + w;  // < npad: both offsets below are inside the array
  const int nret = cnt[bh * 2];
  const int32_t* go = goff + bh * (npad + 1);  // exclusive prefix of the list sizes over [0, nret]
  const int off0 = go[slot], off1 = go[slot + 1];
  if (slot >= nret) return;
  const int ns = off1 - off0;
  if (ns == 0) return;
  const int32_t* src = gsrc + bh * npad + off0;
  const int32_t* el = evi + bh * npad;
  const double* us = ustar + bh * npad;
  const T* kb = K + b * kv.sb + hk * kv.sh;
  const T* vb = V + b * vv.sb + hk * vv.sh;
  constexpr int PER = D / 64;
  const int64_t dst = (bh * slots + meta[bh * 4 + 0] + slot) * D + lane * PER;
  // exp(1), the retained token's self-similarity weight; average merging weighs every member 1
  const double e1 = AVERAGE ? 1.0 : 2.718281828459045;
  auto weight = [&](double u) __attribute__((always_inline)) { return AVERAGE ? 1.0 : exp(u); };
  double ak[PER], av[PER];
  load_elems<T, PER>(cK + dst, ak);
  load_elems<T, PER>(cV + dst, av);
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    ak[p] = __dmul_rn(e1, ak[p]);
    av[p] = __dmul_rn(e1, av[p]);
  }
  double z = e1;
  auto add_source = [&](double wgt, const double* xk, const double* xv) {
    z = __dadd_rn(z, wgt);
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      ak[p] = __dadd_rn(ak[p], __dmul_rn(wgt, xk[p]));
      av[p] = __dadd_rn(av[p], __dmul_rn(wgt, xv[p]));
    }
  };
  // `count` sources, kMergeBatch rows in flight; the weight and position of source s are in lane at(s)
  auto stream = [&](int count, double wl, int pl, auto at) {
    for (int s0 = 0; s0 < count; s0 += kMergeBatch) {
      double wq[kMergeBatch];
      typename RowBits<T, PER>::type xk[kMergeBatch], xv[kMergeBatch];
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u) {
        const int owner = at(min(s0 + u, count - 1));
        wq[u] = lane_f64(wl, owner);
        const int pos = __builtin_amdgcn_readlane(pl, owner);
        xk[u] = load_row_bits<T, PER>(kb + int64_t(pos) * kv.sn + lane * PER);
        xv[u] = load_row_bits<T, PER>(vb + int64_t(pos) * vv.sn + lane * PER);
      }
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u)
        if (s0 + u < count) {
          double fk[PER], fv[PER];
          widen<T, PER>(xk[u], fk);
          widen<T, PER>(xv[u], fv);
          add_source(wq[u], fk, fv);
        }
    }
  };
  if (ns <= 64) {
    const bool have = lane < ns;
    const int mine = have ? src[lane] : 0x7FFFFFFF;
    const double wmine = have ? weight(us[mine]) : 0.0;
    const int pmine = have ? el[mine] : 0;
    int rank = 0;  // sources are distinct: the ranks are a permutation of 0 .. ns-1
    for (int i = 0; i < ns; ++i) rank += __builtin_amdgcn_readlane(mine, i) < mine ? 1 : 0;
    stream(ns, wmine, pmine, [&](int s) { return __ffsll((long long)__ballot(have && rank == s)) - 1; });
  } else if (ns <= kMergeCap) {
    for (int t = lane; t < ns; t += 64) s_src[w][t] = src[t];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int t = lane; t < ns; t += 64) {
      const int mine = s_src[w][t];
      int rank = 0;
      for (int i = 0; i < ns; ++i) rank += s_src[w][i] < mine ? 1 : 0;
      s_sorted[w][rank] = mine;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int t0 = 0; t0 < ns; t0 += 64) {
      const int mine = s_sorted[w][min(t0 + lane, ns - 1)];
      stream(min(64, ns - t0), weight(us[mine]), el[mine], [](int s) { return s; });
    }
  } else {
    int prev = -1;
    for (int s = 0; s < ns; ++s) {
      int cur = 0x7FFFFFFF;
      for (int t = lane; t < ns; t += 64) {
        const int r = src[t];
        if (r > prev && r < cur) cur = r;
      }
      cur = wave_min(cur);
      const double wgt = weight(us[cur]);
      const int64_t pos = el[cur];
      double xk[PER], xv[PER];
      load_elems<T, PER>(kb + pos * kv.sn + lane * PER, xk);
      load_elems<T, PER>(vb + pos * vv.sn + lane * PER, xv);
      add_source(wgt, xk, xv);
      prev = cur;
    }
  }
  store_elems<T, PER>(cK + dst, ak, z);
  store_elems<T, PER>(cV + dst, av, z);
}

}  // namespace

// ---------------------------------------------------------------------------------------------

hipError_t launch_select(d2o_ctx* c, int layer, int n, hipStream_t s, bool append) {
  const d2o_config& cf = c->cfg;
  const float* score = c->score_pre + size_t(layer) * cf.batch * cf.n_kv_heads * c->npad;
  const int bh = cf.batch * cf.n_kv_heads;
  int32_t* meta = c->meta + size_t(layer) * bh * 4;
  const dim3 grid(cf.n_kv_heads, cf.batch);
  KernelTimer kt(c, D2O_K_SELECT, s);
  if (append)
    select_kernel<double, false><<<grid, 1024, 0, s>>>(c->app_score, MetaPack{}, meta, nullptr, c->amb_cnt, c->sel_ret, c->sel_evi,
                                                       c->sel_cnt, n, c->app_n, c->npad, cf.n_sink);
  else if (bh <= kMetaPerLaunch)
    select_kernel<float, true><<<grid, 1024, 0, s>>>(score, pack_meta(c, layer, 0, bh), meta,
                                                     cf.cache_fp8 ? c->meta_stage + size_t(layer) * bh * 4 : nullptr, c->amb_cnt,
                                                     c->sel_ret, c->sel_evi, c->sel_cnt, n, nullptr, c->npad, cf.n_sink);
  else
    select_kernel<float, false><<<grid, 1024, 0, s>>>(score, MetaPack{}, meta, nullptr, c->amb_cnt, c->sel_ret, c->sel_evi,
                                                      c->sel_cnt, n, nullptr, c->npad, cf.n_sink);
  return hipGetLastError();
}

template <typename T>
static void run_gather(d2o_ctx* c, int layer, View K, View V, int max_budget, bool append, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const float* score = c->score_pre + size_t(layer) * cf.batch * cf.n_kv_heads * c->npad;
  const int32_t* meta = c->meta + size_t(layer) * cf.batch * cf.n_kv_heads * 4;
  int32_t* ccount = c->ccount + size_t(layer) * cf.batch * cf.n_kv_heads;
  const int rows = 256 / (cf.head_dim * int(sizeof(T)) / 16);
  const dim3 grid((max_budget + rows - 1) / rows, cf.n_kv_heads, cf.batch);
  if (append)
    gather_kernel<T, true><<<grid, 256, 0, s>>>((const T*)K.ptr, K, (const T*)V.ptr, V, score, c->app_score, c->app_pos,
                                                c->sel_ret, c->sel_cnt, meta, (T*)prompt_rows_K(c), (T*)prompt_rows_V(c), c->cscore,
                                                c->cpos, ccount, c->npad, cf.head_dim, cf.slots_per_seq,
                                                prompt_rows_meta(c, layer), prompt_rows_stride(c), c->invnorm);
  else
    gather_kernel<T, false><<<grid, 256, 0, s>>>((const T*)K.ptr, K, (const T*)V.ptr, V, score, nullptr, nullptr,
                                                 c->sel_ret, c->sel_cnt, meta, (T*)prompt_rows_K(c), (T*)prompt_rows_V(c), c->cscore,
                                                 c->cpos, ccount, c->npad, cf.head_dim, cf.slots_per_seq,
                                                 prompt_rows_meta(c, layer), prompt_rows_stride(c), c->invnorm);
}

static int max_evicted(const d2o_ctx* c, int layer, int n) {
  int m = 0;
  for (const auto& mt : c->layers[layer].meta) m = std::max(m, n - std::min(mt.budget, n));
  return m;
}

hipError_t launch_gather(d2o_ctx* c, int layer, View K, View V, int n, hipStream_t s, bool append) {
  const d2o_config& cf = c->cfg;
  int max_budget = 0;
  for (const auto& mt : c->layers[layer].meta) max_budget = std::max(max_budget, std::min(mt.budget, n));
  if (cf.dtype == D2O_BF16)
    run_gather<uint16_t>(c, layer, K, V, max_budget, append, s);
  else
    run_gather<float>(c, layer, K, V, max_budget, append, s);
  return hipGetLastError();
}

hipError_t launch_match(d2o_ctx* c, int layer, View K, int n, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const int me = max_evicted(c, layer, n);
  if (me == 0) return hipSuccess;
  // evicted rows per workgroup of match_refine (bf16: head_dim 128)
  const int refine_rows = 4 * (cf.dtype == D2O_BF16 ? refine_rows_per_wave<uint16_t, 128>() : refine_rows_per_wave<float, 128>());
  const dim3 gr((me + refine_rows - 1) / refine_rows, cf.n_kv_heads, cf.batch);
  if (cf.dtype == D2O_BF16) {
    const dim3 gf((me + 127) / 128, cf.n_kv_heads, cf.batch);
    {
      KernelTimer kt(c, D2O_K_MATCH_FILTER, s);
      // Up to a workgroup of 32 rows per CU: blocks of 128 rows would leave three CUs of four idle.
      const dim3 few((me + 31) / 32, cf.n_kv_heads, cf.batch);
      if (int64_t(few.x) * few.y * few.z <= 256)
        match_filter_few<<<few, 64 * kFewWaves, 0, s>>>(
            (const uint16_t*)K.ptr, K, (const uint16_t*)prompt_rows_K(c), prompt_rows_meta(c, layer), prompt_rows_stride(c),
            c->invnorm, c->sel_evi, c->sel_cnt, c->m_cand, c->m_thr, c->amb_list, c->amb_cnt, c->m_ncand, c->npad);
      else
        match_filter_bf16<false><<<gf, 256, 0, s>>>((const uint16_t*)K.ptr, K, (const uint16_t*)prompt_rows_K(c),
                                                    prompt_rows_meta(c, layer), prompt_rows_stride(c),
                                                    c->invnorm, c->sel_evi, c->sel_cnt, c->m_cand, c->m_thr, c->amb_list, c->amb_cnt,
                                                    c->m_ncand, c->m_clist, c->npad, 1);
      constexpr int kSplit = 8;
      match_filter_bf16<true><<<dim3(gf.x * kSplit, gf.y, gf.z), 256, 0, s>>>((const uint16_t*)K.ptr, K, (const uint16_t*)prompt_rows_K(c),
                                                 prompt_rows_meta(c, layer), prompt_rows_stride(c),
                                                 c->invnorm, c->sel_evi, c->sel_cnt, c->m_cand, c->m_thr, c->amb_list, c->amb_cnt,
                                                 c->m_ncand, c->m_clist, c->npad, kSplit);
    }
    KernelTimer kt(c, D2O_K_MATCH_REFINE, s);
    match_refine<uint16_t, 128><<<gr, 256, 0, s>>>((const uint16_t*)K.ptr, K, c->sel_ret, c->sel_evi, c->sel_cnt,
                                                   c->m_cand, c->m_ncand, c->m_clist, c->m_ustar, c->m_tgt, c->npad, 1);
  } else if (cf.head_dim == 64) {
    KernelTimer kt(c, D2O_K_MATCH_REFINE, s);
    match_refine<float, 64><<<gr, 256, 0, s>>>((const float*)K.ptr, K, c->sel_ret, c->sel_evi, c->sel_cnt, c->m_cand,
                                               c->m_ncand, c->m_clist, c->m_ustar, c->m_tgt, c->npad, 0);
  } else {
    KernelTimer kt(c, D2O_K_MATCH_REFINE, s);
    match_refine<float, 128><<<gr, 256, 0, s>>>((const float*)K.ptr, K, c->sel_ret, c->sel_evi, c->sel_cnt, c->m_cand,
                                                c->m_ncand, c->m_clist, c->m_ustar, c->m_tgt, c->npad, 0);
  }
  return hipGetLastError();
}

hipError_t launch_threshold_group(d2o_ctx* c, int layer, int n, int new_pos, hipStream_t s, bool append) {
  const d2o_config& cf = c->cfg;
  const size_t lo = size_t(layer) * cf.batch * cf.n_kv_heads;
  double* tau = c->ctau + lo;
  const FirstCandidates fc{c->cscore, c->cpos, c->ccount + lo, c->meta + lo * 4, c->ccand + lo * decode_candidates(),
                           cf.slots_per_seq, new_pos, cf.n_sink};
  threshold_group_kernel<<<dim3(cf.n_kv_heads, cf.batch, 2), 1024, 0, s>>>(c->m_ustar, c->m_tgt, c->sel_cnt, c->m_pass,
                                                                        c->g_cnt, c->g_off, c->g_cur, c->g_src, tau,
                                                                        c->npad, cf.tau_force, append ? 1 : 0, cf.beta, fc);
  return hipGetLastError();
}

template <typename T, int D>
static void run_merge(d2o_ctx* c, const int32_t* meta, View K, View V, int max_budget, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const dim3 grid((max_budget + 3) / 4, cf.n_kv_heads, cf.batch);
  if (cf.merge_average)
    merge_kernel<T, D, true><<<grid, 256, 0, s>>>((const T*)K.ptr, K, (const T*)V.ptr, V, c->sel_evi, c->sel_cnt,
                                                  c->m_ustar, c->g_off, c->g_src, meta, (T*)prompt_rows_K(c), (T*)prompt_rows_V(c),
                                                  c->npad, prompt_rows_stride(c));
  else
    merge_kernel<T, D, false><<<grid, 256, 0, s>>>((const T*)K.ptr, K, (const T*)V.ptr, V, c->sel_evi, c->sel_cnt,
                                                   c->m_ustar, c->g_off, c->g_src, meta, (T*)prompt_rows_K(c), (T*)prompt_rows_V(c),
                                                   c->npad, prompt_rows_stride(c));
}

hipError_t launch_merge(d2o_ctx* c, int layer, View K, View V, int n, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  if (max_evicted(c, layer, n) == 0) return hipSuccess;
  int max_budget = 0;
  for (const auto& mt : c->layers[layer].meta) max_budget = std::max(max_budget, std::min(mt.budget, n));
  const int32_t* meta = prompt_rows_meta(c, layer);  // the merge kernel touches rows only
  KernelTimer kt(c, D2O_K_MERGE, s);
  if (cf.dtype == D2O_BF16)
    run_merge<uint16_t, 128>(c, meta, K, V, max_budget, s);
  else if (cf.head_dim == 64)
    run_merge<float, 64>(c, meta, K, V, max_budget, s);
  else
    run_merge<float, 128>(c, meta, K, V, max_budget, s);
  return hipGetLastError();
}

}  // namespace d2o
