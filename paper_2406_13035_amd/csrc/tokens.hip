// Token-level operation after prompt encoding (Sec. 4.2): selection (Eq. 7-8), compaction into
// the cache, nearest-neighbour matching (Eq. 9), the initial threshold (Eq. 10, t = 0) and the
// similarity-weighted merge (Eq. 11-12).
//
// Every decision (top-N membership, arg-max of the cosine, threshold test) is taken on exact
// integer keys or in fp64 with the operation order of the defining formulas, so that index
// outputs do not depend on reduction shapes; the bf16 matrix-core product of the matching filters
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
  if (tid == 0) amb_cnt[bh] = 0;  // (counted up by the matching filters)
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

// The place of a workgroup in a one-dimensional launch of several workgroups per (sequence, KV head), the heads fastest:
// with a head count that is a multiple of the XCD count all workgroups of a head, which read the same retained
// keys, run on one XCD and share its L2.
struct HeadGrid {
  int Hkv, heads;  // KV heads, and KV heads of all sequences
  __device__ __forceinline__ int index() const { return int(blockIdx.x) % heads; }
  __device__ __forceinline__ int head() const { return index() % Hkv; }
  __device__ __forceinline__ int sequence() const { return index() / Hkv; }
  __device__ __forceinline__ int block() const { return int(blockIdx.x) / heads; }
  __device__ __forceinline__ int blocks() const { return int(gridDim.x) / heads; }
};

// Candidate filter on the matrix cores.  A workgroup owns 128 evicted rows (4 wavefronts x 32,
// the stationary B operand) and streams the retained keys, read contiguously from the cache
// region they were compacted into, in double-buffered tiles of 64 through LDS (the A operand),
// so each lane owns one evicted row and sees 16 retained keys per MFMA tile.  Per row, the best and
// second-best fp32 cosine and the best's retained rank.  A row whose two best values differ by less than
// kAmbiguous is flagged and its acceptance threshold (best - kAmbiguous, in the un-normalised domain) is stored, for
// match_flagged; the others have one candidate, whose exact similarity the two lanes that hold the row form
// at once.  (As a launch of its own, which read the evicted rows again, that took 19 us at 32 heads x 4096 tokens, a
// fifth kept, and 153 at 32768, a tenth kept.)
// The filter is bound by the vector ALU (68 instructions per 32 x 32 sub-tile and wavefront beside 8 products), as
// long as no wavefront waits for LDS: with the operands and inverse norms requested half a sub-tile ahead and the
// padding confined to the last tile, at four wavefronts per SIMD, 940 -> 867 us (32768 tokens, 32 heads, a tenth
// kept), 37 -> 34 (4096, a fifth), 54 -> 41 (256 of 2304 rows leave); with the exact similarities 864 and 40 (two of the 128
// registers are spilled over the loop, 12 bytes per lane).
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

// The margin of a row's best two, in the un-normalised domain (ie: the row's inverse norm), and whether they are too close;
// also true for NaN / equal / zero norm, and where the best is no key: padding wins where no retained key has a value (all of
// them are NaN), and the values of the padding differ among themselves by far more than the margin.
__device__ __forceinline__ float margin_of(float ie) { return ie > 0.f ? kAmbiguous / ie : INFINITY; }
__device__ __forceinline__ bool is_ambiguous(float best, float second, int bi, int nret, float ie) {
  return bi >= nret || !(best - second >= margin_of(ie));
}
__device__ __forceinline__ void flag_row(float best, float ie, int erank, int epos, int64_t base, int64_t bh,
                                         FlaggedRow* amb_list, int32_t* amb_cnt) {
  amb_list[base + atomicAdd(&amb_cnt[bh], 1)] = FlaggedRow{erank, epos, best - margin_of(ie), 0};
}

// Exact similarity in fp64, operation order of Eq. 9 as written: dot / (|k_i| * |k_j|), 0 when
// a norm is 0.  Products of bf16 values are exact in fp64 and their sums stay
// exact at these magnitudes; the order of additions is the same everywhere all the same: eight neighbouring
// elements one after the other, then neighbouring sums in pairs.
struct DotNorms {
  double dot, ne, nr;  // evicted key . retained key, and their squared norms
};
__device__ __forceinline__ DotNorms operator+(const DotNorms& a, const DotNorms& b) {
  return DotNorms{a.dot + b.dot, a.ne + b.ne, a.nr + b.nr};
}
__device__ __forceinline__ DotNorms dot_of_eight(const u32x4& x, const u32x4& y) {
  DotNorms s{0.0, 0.0, 0.0};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double a = double(__uint_as_float(e & 1 ? x[e / 2] & 0xFFFF0000u : x[e / 2] << 16));
    const double b = double(__uint_as_float(e & 1 ? y[e / 2] & 0xFFFF0000u : y[e / 2] << 16));
    s.dot = fma(a, b, s.dot);
    s.ne = fma(a, a, s.ne);
    s.nr = fma(b, b, s.nr);
  }
  return s;
}
__device__ __forceinline__ double cosine(const DotNorms& s) {
  const double den = sqrt(s.ne) * sqrt(s.nr);
  return den > 0.0 ? s.dot / den : 0.0;
}
// By sixteen neighbouring lanes, eight elements each.
__device__ __forceinline__ double cosine_by_16(const u32x4& x, const u32x4& y) {
  const DotNorms s = dot_of_eight(x, y);
  return cosine(DotNorms{row16_sum(s.dot), row16_sum(s.ne), row16_sum(s.nr)});
}
// By lanes l and l + 32, which hold elements 16 ks + 8 (l / 32) .. of both keys, as the matrix instruction's operands.
__device__ __forceinline__ double cosine_by_2(const bf16x8 (&be)[8], const u32x4 (&y)[8]) {
  auto part = [&](int ks) {
    const DotNorms s = dot_of_eight(__builtin_bit_cast(u32x4, be[ks]), y[ks]);
    return DotNorms{sum_halves(s.dot), sum_halves(s.ne), sum_halves(s.nr)};
  };
  auto four = [&](int ks) { return (part(ks) + part(ks + 1)) + (part(ks + 2) + part(ks + 3)); };
  return cosine(four(0) + four(4));
}
// (a non-finite key: no cosine compares above the start, and no threshold is reached)
__device__ __forceinline__ void store_match(double u, int j, int64_t at, double* ustar, int32_t* tgt) {
  const bool none = !(u > -2.0);
  ustar[at] = none ? __longlong_as_double(0x7FF8000000000000ll) : u;
  tgt[at] = none ? 0 : j;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void match_filter_bf16(const uint16_t* __restrict__ K, View kv,
                                                         const uint16_t* __restrict__ cK,
                                                         const int32_t* __restrict__ meta, int64_t slots,
                                                         const float* __restrict__ invn,
                                                         const int32_t* __restrict__ evi,
                                                         const int32_t* __restrict__ cnt,
                                                         FlaggedRow* __restrict__ amb_list,
                                                         int32_t* __restrict__ amb_cnt, double* __restrict__ ustar,
                                                         int32_t* __restrict__ tgt, int npad, HeadGrid hg) {
  constexpr int kTile = 64;     // retained keys per LDS tile
  constexpr int NCH = kTile * 16 / 256;  // 16-byte chunks of a tile per thread
  __shared__ __attribute__((aligned(16))) uint16_t Rs[2][kTile * kLdM];
  __shared__ __attribute__((aligned(16))) float rin[2][kTile];    // 1/|k| of the staged retained keys
  __shared__ __attribute__((aligned(16))) float rbias[2][kTile];  // 0, or -3e38 for padding rows (finite: the low
                                                                  // mantissa bits of a value get overwritten below)
  const int hk = hg.head(), b = hg.sequence();
  const int64_t bh = hg.index();
  const int nret = cnt[bh * 2], nevi = cnt[bh * 2 + 1];
  const int e0 = hg.block() * 128;
  if (e0 >= nevi) return;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 31, h = lane >> 5;
  const uint16_t* kb = K + b * kv.sb + hk * kv.sh;
  // the retained keys, in retained order, already sit contiguously in the layer's cache
  // region (compaction runs first; merging, which changes them, runs after the matching)
  const uint16_t* rk = cK + (bh * slots + meta[bh * 4 + 0]) * 128;
  const int32_t* el = evi + bh * npad;
  const float* inl = invn + bh * npad;  // by retained rank
  const int epos = el[min(e0 + w * 32 + m, nevi - 1)];
  bf16x8 be[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    be[ks] = *reinterpret_cast<const bf16x8*>(kb + int64_t(epos) * kv.sn + ks * 16 + h * 8);
  BestTwo two;
  // Tiles travel global -> registers -> LDS: the next tile is requested when work on a tile
  // starts and written to the other LDS buffer when it ends.
  u32x4 rg[NCH];
  float rv = 0.f;
  const int tend = (nret + kTile - 1) / kTile;
  const int tfull = nret / kTile;  // the first tile that is not full
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
      two.take(tv, r0 + st * 32);
    };
    // (two sub-tiles as two independent accumulation chains need 160 registers and cost a
    // wavefront per SIMD: slower)
    post(mma(0), 0);
    if (!padded || nret - r0 > 32) post(mma(1), 1);
    if (t + 1 < tend) stage(buf ^ 1);
    __syncthreads();
  };
  issue(0);
  stage(0);
  __syncthreads();
#pragma unroll 1
  for (int t = 0; t < tfull; ++t) one_tile(t, std::false_type{});
  if (tfull < tend) one_tile(tfull, std::true_type{});
  // combine the two lane halves that share an evicted row
  float best = two.m1, second = two.m2;
  int bi = two.rank(h);
  join_best(best, second, bi, __shfl_xor(best, 32, 64), __shfl_xor(second, 32, 64), __shfl_xor(bi, 32, 64));
  const float ie = evicted_norm(be);
  const int row = e0 + w * 32 + m;
  const bool live = row < nevi;
  const int erank = min(row, nevi - 1);
  const bool amb = is_ambiguous(best, second, bi, nret, ie);  // (both lanes agree; unless it is, they have the same candidate)
  u32x4 y[8];
  const uint16_t* yrow = rk + int64_t(amb ? 0 : bi) * 128 + h * 8;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) y[ks] = *reinterpret_cast<const u32x4*>(yrow + ks * 16);
  const double u = cosine_by_2(be, y);
  if (h == 0 && live) {
    if (amb)
      flag_row(best, ie, erank, el[erank], bh * npad, bh, amb_list, amb_cnt);
    else
      store_match(u, bi, bh * npad + erank, ustar, tgt);
  }
}

// A wavefront's way through the retained keys for 32 evicted rows, whose operands it holds: the 32-key sub-tiles w, w + STEP,
// ... come in whole lines one ahead and pass through the wavefront's own LDS (as the operands themselves, 32 bytes of every
// row per load, a line came from the L2 four times over), with their inverse norms.  post(s, j): the sub-tile's products,
// register r of key 32 j + (r / 4) 8 + 4 h + r % 4.  Same values as in match_filter_bf16, in the same order of products.
template <int STEP, typename Post>
__device__ __forceinline__ void sweep_keys(const uint16_t* rk, const float* inl, int nret, int w, int lane,
                                           const bf16x8 (&be)[8], uint16_t* tile, float* rin, Post post) {
  const int m = lane & 31, h = lane >> 5, nsub = (nret + 31) / 32;
  if (w >= nsub) return;
  u32x4 rg[8];
  float norm;
  // (rows and norms past the last one: zero)
  const __amdgpu_buffer_rsrc_t norms = buffer_of(inl, uint32_t(nret) * 4);
  auto request = [&](int j) {
    const int js = __builtin_amdgcn_readfirstlane(j), rows = max(min(nret - js * 32, 32), 0);
    const __amdgpu_buffer_rsrc_t keys = buffer_of(rk + int64_t(js) * 32 * 128, uint32_t(rows) * 256);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      rg[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(keys, lane * 16 + i * 1024, 0, 0));
    norm = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(norms, (js * 32 + m) * 4, 0, 0));
  };
  // (within the wavefront; LDS serves its requests in order, so the hand-overs need compiler ordering only)
  auto hand_over = []() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  request(w);
#pragma unroll 1
  for (int j = w; j < nsub; j += STEP) {
    hand_over();
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(tile + (i * 4 + (lane >> 4)) * kLdM + (lane & 15) * 8) = rg[i];
    if (h == 0) rin[m] = norm;
    hand_over();
    if (j + STEP < nsub) request(j + STEP);
    f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(tile + m * kLdM + ks * 16 + h * 8), be[ks], s, 0, 0, 0);
    post(s, j);
  }
}

// The filter for launches of few rows: 32 evicted rows per workgroup, whose wavefronts take the sub-tiles
// in turn and join their best two at the end.  A launch of few rows leaves most of the chip idle in blocks of 128; from
// two workgroups per CU on those, which read the keys a quarter as often, are the faster ones (512 rows against 128 keys 18.4
// where this takes 20.4, 800 against 200 18.5 where it takes 31).  256 rows against 2048 keys, 32 heads: 17 us with the exact
// similarities, where the operands came straight from memory 23 without.
constexpr int kFewWaves = 4;
__global__ __launch_bounds__(64 * kFewWaves) void match_filter_few(const uint16_t* __restrict__ K, View kv,
                                                                   const uint16_t* __restrict__ cK,
                                                                   const int32_t* __restrict__ meta, int64_t slots,
                                                                   const float* __restrict__ invn,
                                                                   const int32_t* __restrict__ evi,
                                                                   const int32_t* __restrict__ cnt,
                                                                   FlaggedRow* __restrict__ amb_list,
                                                                   int32_t* __restrict__ amb_cnt,
                                                                   double* __restrict__ ustar,
                                                                   int32_t* __restrict__ tgt, int npad, HeadGrid hg) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[kFewWaves][32 * kLdM];
  __shared__ __attribute__((aligned(16))) float rin[kFewWaves][32];  // of the wavefront's sub-tile
  __shared__ float best_s[kFewWaves][32], second_s[kFewWaves][32];
  __shared__ int rank_s[kFewWaves][32];
  const int hk = hg.head(), b = hg.sequence();
  const int64_t bh = hg.index();
  const int nret = cnt[bh * 2], nevi = cnt[bh * 2 + 1];
  const int e0 = hg.block() * 32;
  if (e0 >= nevi) return;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 31, h = lane >> 5;
  const uint16_t* rk = cK + (bh * slots + meta[bh * 4 + 0]) * 128;
  const uint16_t* kb = K + b * kv.sb + hk * kv.sh;
  const int erank = min(e0 + m, nevi - 1);
  const int epos = evi[bh * npad + erank];
  const uint16_t* erow = kb + int64_t(epos) * kv.sn;
  bf16x8 be[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) be[ks] = *reinterpret_cast<const bf16x8*>(erow + ks * 16 + h * 8);
  BestTwo two;
  sweep_keys<kFewWaves>(rk, invn + bh * npad, nret, w, lane, be, tile[w], rin[w], [&](const f32x16& s, int j) {
    float tv[16];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const f32x4 ri = *reinterpret_cast<const f32x4*>(&rin[w][g4 * 8 + h * 4]);
#pragma unroll
      for (int i = 0; i < 4; ++i) tv[g4 * 4 + i] = s[g4 * 4 + i] * ri[i];
    }
    if (j * 32 + 32 > nret) {  // zeros past the end: the lowest value
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (j * 32 + (r >> 2) * 8 + h * 4 + (r & 3) >= nret) tv[r] = -3.0e38f;
    }
    two.take(tv, j * 32);
  });
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
  if (tid < 32) {
#pragma unroll
    for (int u = 1; u < kFewWaves; ++u) join_best(best, second, bi, best_s[u][tid], second_s[u][tid], rank_s[u][tid]);
    const bool live = e0 + tid < nevi, amb = is_ambiguous(best, second, bi, nret, ie);
    if (live && amb) flag_row(best, ie, erank, epos, bh * npad, bh, amb_list, amb_cnt);
    rank_s[0][tid] = live && !amb ? bi : -1;
  }
  __syncthreads();
  // the exact similarities, sixteen lanes per row
#pragma unroll
  for (int i = 0; i < 32; i += kFewWaves * 4) {
    const int r = i + tid / 16, j = rank_s[0][r];
    const int at = evi[bh * npad + min(e0 + r, nevi - 1)];
    const u32x4 x = *reinterpret_cast<const u32x4*>(kb + int64_t(at) * kv.sn + tid % 16 * 8);
    const u32x4 y = *reinterpret_cast<const u32x4*>(rk + int64_t(max(j, 0)) * 128 + tid % 16 * 8);
    const double u = cosine_by_16(x, y);
    if (tid % 16 == 0 && j >= 0) store_match(u, j, bh * npad + e0 + r, ustar, tgt);
  }
}

// The flagged rows (a list in no particular order; the rows are independent of each other).  A workgroup takes 32 or 8 of
// them at a time: its wavefronts sweep the retained keys again and list, in LDS, every key whose fp32
// cosine reaches the row's threshold (the best value among them: the arithmetic is the first sweep's), up to kMaxCand;
// then sixteen lanes per row decide among them exactly, first maximum in ascending retained order.  A row with more of
// them, or none (a zero norm, a key that is not finite), is searched exhaustively by its wavefront.  Half a
// percent of the rows is flagged, so the launch has a few workgroups per head, and what bounds
// it is the instructions of one wavefront: hits as bits instead of sixteen branches, addresses through buffer
// descriptors, eight wavefronts (sixteen share the SIMDs and spill: 8.8 -> 16.5 us).  32 heads x 4096 tokens, a fifth kept, 8.8 us;
// 32768, a tenth kept, 19.8; as a sweep in blocks of 128 rows by eight key ranges, most of them empty, 11 and 44.
// Where many rows are flagged (repeated keys, zeros), all workgroups share what lies beyond each head's first blocks; where few
// are, a block has a row per wavefront, as the exhaustive search is a wavefront's own.  (With the head's own workgroups only and
// blocks of 32, one head of 32768 tokens, a tenth kept: every row tied in pairs 835 us, now 73, in nines 43.5 and 3.1 ms, a tenth
// of the evicted keys zero 4632 and 770 us; one of 4096 with a tenth zero 111 and 37.)
constexpr int kFlaggedWaves = 8;
__global__ __launch_bounds__(64 * kFlaggedWaves) void match_flagged(const uint16_t* __restrict__ K, View kv,
                                                                    const uint16_t* __restrict__ cK,
                                                                    const int32_t* __restrict__ meta, int64_t slots,
                                                                    const float* __restrict__ invn,
                                                                    const int32_t* __restrict__ cnt,
                                                                    const FlaggedRow* __restrict__ amb_list,
                                                                    const int32_t* __restrict__ amb_cnt,
                                                                    double* __restrict__ ustar, int32_t* __restrict__ tgt,
                                                                    int npad, HeadGrid hg) {
  static_assert(kFlaggedWaves * 4 == 32, "sixteen lanes per row");
  constexpr int D = 128;
  __shared__ __attribute__((aligned(16))) uint16_t tile[kFlaggedWaves][32 * kLdM];
  __shared__ __attribute__((aligned(16))) float rin[kFlaggedWaves][32];  // of the wavefront's sub-tile
  __shared__ int ncand[32], clist[32][kMaxCand];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, m = lane & 31, h = lane >> 5;
  const int rr = w + lane / 16 * kFlaggedWaves, tc = tid % 16;  // the row of the exact comparison
  // ---- a head's own workgroups take its first blocks of rows, as many for every head; where a head has more, all
  //      workgroups share what is left of all heads
  int most = 0, least = 0x7FFFFFFF;  // flagged rows of a head
  for (int x = lane; x < hg.heads; x += 64) {
    most = max(most, amb_cnt[x]);
    least = min(least, amb_cnt[x]);
  }
  const int nblk = hg.blocks();
  const bool more = __any(most > nblk * 32);
  int rounds = 1;  // of a head's own workgroups
  if (more) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) least = min(least, __shfl_xor(least, o, 64));
    rounds = max(__builtin_amdgcn_readfirstlane(least) / (nblk * 32), 1);
  }
  // the head in work
  int64_t bh;
  int namb, nret;
  const uint16_t *rk, *kb;
  const FlaggedRow* list;
  auto take_head = [&](int x) {
    bh = x;
    namb = amb_cnt[x];
    nret = cnt[bh * 2];
    rk = cK + (bh * slots + meta[bh * 4 + 0]) * D;
    kb = K + x / hg.Hkv * kv.sb + x % hg.Hkv * kv.sh;
    list = amb_list + bh * npad;
  };
  take_head(hg.index());
  int group = namb <= 8 * min(nblk, 256 / hg.heads) ? 8 : 32;  // rows of a block: one per wavefront where there is a CU for each
  int e0 = hg.block() * group;
  int at = 0, before = 0;  // the rest: the 64 heads in turn, and the blocks of the heads before them
#pragma unroll 1
  for (int i = blockIdx.x, round = 1;;) {
    const int end = min(namb, e0 + group);
    if (e0 < end) {
      const FlaggedRow fr = list[min(e0 + m, end - 1)], own = list[min(e0 + rr, end - 1)];
      const float mythr = e0 + m < end ? fr.thr : INFINITY;
      const bool valid = e0 + rr < end;
      const uint16_t* erow = kb + int64_t(fr.pos) * kv.sn;
      bf16x8 be[8];
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) be[ks] = *reinterpret_cast<const bf16x8*>(erow + ks * 16 + h * 8);
      const u32x4 x = *reinterpret_cast<const u32x4*>(kb + int64_t(own.pos) * kv.sn + tc * 8);
      if (tid < 32) ncand[tid] = 0;
      __syncthreads();
      sweep_keys<kFlaggedWaves>(rk, invn + bh * npad, nret, w, lane, be, tile[w], rin[w], [&](const f32x16& s, int j) {
        uint32_t hits = 0;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const f32x4 ri = *reinterpret_cast<const f32x4*>(&rin[w][g4 * 8 + h * 4]);
#pragma unroll
          for (int i = 0; i < 4; ++i) hits |= s[g4 * 4 + i] * ri[i] >= mythr ? 1u << (g4 * 4 + i) : 0u;
        }
        while (hits) {
          const int r = __ffs(hits) - 1, key = j * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
          hits &= hits - 1;
          const int k = key < nret ? atomicAdd(&ncand[m], 1) : kMaxCand;
          if (k < kMaxCand) clist[m][k] = key;
        }
      });
      __syncthreads();
      // ---- exactly: sixteen lanes per row, two candidates in flight
      const int listed = valid ? ncand[rr] : 0, ncd = listed <= kMaxCand ? listed : 0;
      double best = -2.0;
      int bj = 0;
      int nloop = max(ncd, __shfl_xor(ncd, 16, 64));
      nloop = max(nloop, __shfl_xor(nloop, 32, 64));
      for (int q = 0; q < nloop; q += 2) {
        int j[2];
        u32x4 y[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          j[i] = q + i < ncd ? clist[rr][q + i] : 0;
          y[i] = *reinterpret_cast<const u32x4*>(rk + int64_t(j[i]) * D + tc * 8);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const double u = cosine_by_16(x, y[i]);
          if (q + i < ncd && (u > best || (u == best && j[i] < bj))) {
            best = u;
            bj = j[i];
          }
        }
      }
      unsigned long long todo = __ballot(valid && ncd == 0 && tc == 0);
      while (todo) {  // one row at a time, the wavefront's lanes striding over the retained keys
        const int src = __ffsll((long long)todo) - 1;  // first lane of the row to serve
        todo &= todo - 1;
        double* ke = reinterpret_cast<double*>(tile[w]);  // the row as fp64
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double ne = 0.0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double v = double(__uint_as_float(e & 1 ? x[e / 2] & 0xFFFF0000u : x[e / 2] << 16));
          if (lane / 16 == src / 16) ke[tc * 8 + e] = v;
          ne = fma(v, v, ne);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const double sne = sqrt(lane_f64(row16_sum(ne), src));
        double fb = -2.0;
        int fj = 0x7FFFFFFF;
        for (int j = lane; j < nret; j += 64) {
          double dot = 0.0, nr = 0.0;
#pragma unroll 1
          for (int c = 0; c < D; c += 8) {
            const u32x4 y = *reinterpret_cast<const u32x4*>(rk + int64_t(j) * D + c);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const double v = double(__uint_as_float(e & 1 ? y[e / 2] & 0xFFFF0000u : y[e / 2] << 16));
              dot = fma(ke[c + e], v, dot);
              nr = fma(v, v, nr);
            }
          }
          const double den = sne * sqrt(nr);
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
      if (tc == 0 && valid) store_match(best, bj, bh * npad + own.erank, ustar, tgt);
      __syncthreads();  // the lists are read before they are emptied
    }
    if (!more) return;
    if (round++ < rounds) {
      e0 += nblk * 32;
      continue;
    }
    // the block i of what is left of the heads, of 64 heads at a time
    int last, total;  // blocks up to and with the lane's head
    for (;; at += 64, before += total) {
      if (at >= hg.heads) return;
      last = at + lane < hg.heads ? max((amb_cnt[at + lane] + 31) / 32 - nblk * rounds, 0) : 0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(last, o, 64);
        if (lane >= o) last += t;
      }
      total = __builtin_amdgcn_readlane(last, 63);
      if (i - before < total) break;
    }
    const int x = __popcll(__ballot(last <= i - before));
    take_head(at + x);
    group = 32;
    e0 = (nblk * rounds + i - before - (x > 0 ? __builtin_amdgcn_readlane(last, max(x - 1, 0)) : 0)) * 32;
    i += gridDim.x;
  }
}

// fp32: the exact search over all retained keys (no filter: 24 bits of a product are not decided by fp32 sums).  One evicted row
// per wavefront, whose lanes stride over the retained keys, first maximum in ascending retained order; the
// sums run over four neighbouring elements, the evicted key's norm over sixteen or 32 lanes.
template <int D>
__global__ __launch_bounds__(256) void match_search_f32(const float* __restrict__ K, View kv, const int32_t* __restrict__ ret,
                                                        const int32_t* __restrict__ evi, const int32_t* __restrict__ cnt,
                                                        double* __restrict__ ustar, int32_t* __restrict__ tgt, int npad) {
  constexpr int TPR = D / 4;  // lanes that share the evicted row, 16 bytes each
  __shared__ double ke[4][D];
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int nret = cnt[bh * 2], nevi = cnt[bh * 2 + 1];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, tc = lane % TPR;
  const int erank = blockIdx.x * 4 + w;
  if (erank >= nevi) return;
  const float* kb = K + b * kv.sb + hk * kv.sh;
  const int32_t* rl = ret + bh * npad;
  const float4 x = *reinterpret_cast<const float4*>(kb + int64_t(evi[bh * npad + erank]) * kv.sn + tc * 4);
  const double xs[4] = {x.x, x.y, x.z, x.w};
  double ne = 0.0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    ne = fma(xs[e], xs[e], ne);
    if (lane < TPR) ke[w][tc * 4 + e] = xs[e];
  }
  ne = row16_sum(ne);
  if constexpr (TPR == 32) ne += __shfl_xor(ne, 16, 64);
  const double sne = sqrt(ne);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  double fb = -2.0;
  int fj = 0x7FFFFFFF;
  for (int j = lane; j < nret; j += 64) {
    const float* rr = kb + int64_t(rl[j]) * kv.sn;
    double dot = 0.0, nr = 0.0;
#pragma unroll 4
    for (int c = 0; c < D; c += 4) {
      const float4 y = *reinterpret_cast<const float4*>(rr + c);
      const double ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        dot = fma(ke[w][c + e], ys[e], dot);
        nr = fma(ys[e], ys[e], nr);
      }
    }
    const double den = sne * sqrt(nr);
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
  if (lane == 0) store_match(fb, fj, bh * npad + erank, ustar, tgt);
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
  if (cf.dtype == D2O_BF16) {
    const int heads = cf.batch * cf.n_kv_heads;
    const HeadGrid hg{cf.n_kv_heads, heads};
    const uint16_t *k = (const uint16_t*)K.ptr, *rows = (const uint16_t*)prompt_rows_K(c);
    const int32_t* meta = prompt_rows_meta(c, layer);
    const int64_t stride = prompt_rows_stride(c);
    {
      KernelTimer kt(c, D2O_K_MATCH_FILTER, s);
      // Up to a workgroup of 32 rows per CU: blocks of 128 rows would leave three CUs of four idle.
      const int64_t few = int64_t((me + 31) / 32) * heads;
      if (few <= 256)
        match_filter_few<<<int(few), 64 * kFewWaves, 0, s>>>(k, K, rows, meta, stride, c->invnorm, c->sel_evi, c->sel_cnt,
                                                             c->amb_list, c->amb_cnt, c->m_ustar, c->m_tgt, c->npad, hg);
      else
        match_filter_bf16<<<(me + 127) / 128 * heads, 256, 0, s>>>(k, K, rows, meta, stride, c->invnorm, c->sel_evi, c->sel_cnt,
                                                                   c->amb_list, c->amb_cnt, c->m_ustar, c->m_tgt, c->npad, hg);
    }
    KernelTimer kt(c, D2O_K_MATCH_REFINE, s);
    // Sixteen workgroups per head, or two for every CU where few heads leave the chip idle (one fits a CU at a time).
    const int per_head = std::min((me + 31) / 32, std::max(16, 512 / heads));
    match_flagged<<<per_head * heads, 64 * kFlaggedWaves, 0, s>>>(
        k, K, rows, meta, stride, c->invnorm, c->sel_cnt, c->amb_list, c->amb_cnt, c->m_ustar, c->m_tgt, c->npad, hg);
  } else {
    const dim3 grid((me + 3) / 4, cf.n_kv_heads, cf.batch);
    KernelTimer kt(c, D2O_K_MATCH_REFINE, s);
    if (cf.head_dim == 64)
      match_search_f32<64><<<grid, 256, 0, s>>>((const float*)K.ptr, K, c->sel_ret, c->sel_evi, c->sel_cnt, c->m_ustar, c->m_tgt, c->npad);
    else
      match_search_f32<128><<<grid, 256, 0, s>>>((const float*)K.ptr, K, c->sel_ret, c->sel_evi, c->sel_cnt, c->m_ustar, c->m_tgt, c->npad);
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
