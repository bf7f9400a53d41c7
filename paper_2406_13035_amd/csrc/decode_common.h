// Building blocks of the decode-step kernels in csrc/decode.hip: kernel arguments, element
// conversions, the orders in which matches and evictions are decided, and the step's closing
// arithmetic (Eq. 9-12 with one source).  Header-only; not part of the C ABI.
#pragma once

#include "d2o_internal.h"
#include "device_utils.h"

namespace d2o {
namespace dec {

// Eviction candidates whose similarities ride along with the attention pass.  One: the token
// with the lowest score after a step is, with very few exceptions, the one evicted at the next
// (scores only grow, and the lowest tokens are the ones that receive next to no attention); on
// the benchmark workloads no eviction of 5 x 10^5 to 2 x 10^6 head-steps took another token.
// Every further candidate costs the K pass another fp64 dot product per cache row (with three,
// configuration 4 ran 6 % and an fp8 cache 11 % slower); a miss costs one head a second pass
// over its keys.
constexpr int kCand = 1;
constexpr int kMaxLayersPerCall = 64;
// Doubles per sub-chunk record: the G softmax maxima, the G exp-sums, then per candidate its
// best cosine, that key's slot and its position; rounded up to a multiple of eight (64 bytes).
__host__ __device__ constexpr int rec_doubles(int G) { return (2 * G + 3 * kCand + 7) / 8 * 8; }
constexpr int kPiece = 64;              // bytes of a cache row staged per LDS round
constexpr int kPitch = kPiece + 16;     // LDS pitch of a staged row piece (20 words: sixteen lanes that read sixteen
                                        // consecutive rows, and four lanes that write a row, meet all banks once)
// A wavefront's 64 rows are staged in four sets of sixteen, row s + 4 b + 16 i as row 4 b + i of set s; 16 words
// between the sets put consecutive rows on different banks for the writing lanes.
constexpr int kSetBytes = 16 * kPitch + 64;
constexpr int kWaveStage = 4 * kSetBytes;
constexpr int kStageBytes = 4 * kWaveStage;
constexpr int kSub = 64;                // rows one wavefront handles at a time (lane = row)

struct DecodeArgs {
  int32_t* ccount;
  int32_t* ctotal;    // [L][B][Hkv] entries (count + 1) of a head that decode_attend leaves to the split kernels, else 0
  double* ctau;
  const int32_t* meta;
  void* cK;
  void* cV;
  int8_t* cKe;        // fp8 cache only: the power of two of every K row, [B][Hkv][slots]
  int8_t* cVe;        // the same for V
  double* cscore;
  int32_t* cpos;
  int32_t* cand;      // [L][B][Hkv][kCand] candidate slots for this step, -1 = none
  uint32_t* ticket;   // [L][B][Hkv] finished chunks of the running step
  uint32_t* cmiss;    // [L][B][Hkv] evictions whose token was not among the predicted candidates (since the last reset)
  double* elog;       // [chunk][B][Hkv][G][256] exp(logit - sub-chunk max)
  double* rec;        // [chunk][B][Hkv][4][rec_doubles(G)] per sub-chunk record: [0..G) softmax maxima of the
                      // query heads, [G..2G) exp-sums relative to them, [2G..2G+kCand) the candidates' best
                      // cosine, [2G+kCand..2G+2kCand) its slot (-1 none), [2G+2kCand..2G+3kCand) its position; written with one store
  float* pacc;        // [chunk][B][Hkv][G][d] partial outputs, relative to the chunk's softmax maximum
  int32_t* ev_evicted;
  int32_t* ev_target;
  double* ev_ustar;
  int64_t slots;
  int layer0, nl, B, Hkv, G, new_pos, n_sink, out_f32, merge_average;
  int big_rows;       // heads with more entries are closed by the split kernels, not by their last workgroup
  int part_chunks;    // chunks per workgroup of decode_close_part
  double* part;       // [chunk][B][Hkv][kPartRecDoubles] part records (at a part's first chunk)
  double* hnorm;      // [L][B][Hkv][16] of a head closed in parts: [0..G) softmax maxima, [G..2G) exact normalisers
  double beta, tau_force;
  int32_t lay_off[kMaxLayersPerCall + 1];  // first flat chunk-group index of each entry of lay_id
  int32_t lay_id[kMaxLayersPerCall];       // layers of the call (relative), most chunks first
};

template <typename T>
__device__ __forceinline__ void cvt16(const u32x4& v, double* out);  // 16 bytes -> 8 or 4 doubles
template <>
__device__ __forceinline__ void cvt16<uint16_t>(const u32x4& v, double* out) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[2 * i] = double(__uint_as_float(v[i] << 16));
    out[2 * i + 1] = double(__uint_as_float(v[i] & 0xFFFF0000u));
  }
}
template <>
__device__ __forceinline__ void cvt16<float>(const u32x4& v, double* out) {
#pragma unroll
  for (int i = 0; i < 4; ++i) out[i] = double(__uint_as_float(v[i]));
}
template <>
__device__ __forceinline__ void cvt16<uint8_t>(const u32x4& v, double* out) {  // sixteen fp8 codes, without the row's power of two
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[4 * i] = double(__builtin_amdgcn_cvt_f32_fp8(int(v[i]), 0));
    out[4 * i + 1] = double(__builtin_amdgcn_cvt_f32_fp8(int(v[i]), 1));
    out[4 * i + 2] = double(__builtin_amdgcn_cvt_f32_fp8(int(v[i]), 2));
    out[4 * i + 3] = double(__builtin_amdgcn_cvt_f32_fp8(int(v[i]), 3));
  }
}

// 8 or 16 bytes of consecutive elements held as raw bits.
template <int BYTES> struct RawBits;
template <> struct RawBits<16> { typedef u32x4 type; };
template <> struct RawBits<8> { typedef u32x2 type; };
// 16, or BYTES, bytes per lane of a stream that is read once (non-temporal), `off` bytes into the buffer; zero past its end.
constexpr int kStreamPolicy = 2;
__device__ __forceinline__ u32x4 stream16(__amdgpu_buffer_rsrc_t src, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(src, int(off), 0, kStreamPolicy));
}
template <int BYTES>
__device__ __forceinline__ typename RawBits<BYTES>::type stream_raw(__amdgpu_buffer_rsrc_t src, uint32_t off) {
  if constexpr (BYTES == 16) return stream16(src, off);
  else return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(src, int(off), 0, kStreamPolicy));
}
// The partial results of a step are laid out chunk-major: [layer's chunk offset + chunk]
// [sequence][KV head]...  Workgroups are dispatched head-fastest, so the results that are written
// at about the same time are neighbours in memory (per-head contiguous arrays scatter them; a
// streaming probe with this kernel's store pattern lost 6.2 -> 5.0 TB/s of read rate to the
// scattered form and 6.2 -> 5.3 to this one).
__device__ __forceinline__ int64_t sub_index(const DecodeArgs& a, int64_t bh, int chunk0, int c) {  // sub-chunk c of the head
  return ((int64_t(chunk0) + (c >> 2)) * (a.B * a.Hkv) + bh) * 4 + (c & 3);
}
__device__ __forceinline__ int64_t chunk_index(const DecodeArgs& a, int64_t bh, int chunk0, int chunk) {  // chunk of the head
  return (int64_t(chunk0) + chunk) * (a.B * a.Hkv) + bh;
}
__device__ __forceinline__ int64_t elog_index(const DecodeArgs& a, int64_t bh, int chunk0, int G, int g, int j) {  // slot j
  return (((int64_t(chunk0) + (j >> 8)) * (a.B * a.Hkv) + bh) * G + g) * kChunk + (j & (kChunk - 1));
}

// Place of element c of operand vector v (queries, then candidate keys) in the LDS table: the order in
// which the lanes of the K pass's matrix instructions fetch it.  A row piece of 64 bytes is four
// parts of 16 (k = 0..3); two consecutive elements of every part and vector form a step.
template <typename T, int NV>
__host__ __device__ constexpr int operand_index(int v, int c) {
  constexpr int EP = kPiece / int(sizeof(T)), EL = 16 / int(sizeof(T));
  const int p = c / EP, k = c % EP / EL, e = c % EL;
  return (((p * (EL / 2) + e / 2) * NV + v) * 4 + k) * 2 + (e & 1);
}
// Elements 2 i and 2 i + 1 of 16 bytes of a row (fp8 codes: without the row's power of two).
template <typename T>
__device__ __forceinline__ void pair_f64(const u32x4& r, int i, double& x0, double& x1) {
  if constexpr (sizeof(T) == 1) {
    const int wd = int(r[i / 2]);
    const auto two = i & 1 ? __builtin_amdgcn_cvt_pk_f32_fp8(wd, true) : __builtin_amdgcn_cvt_pk_f32_fp8(wd, false);
    x0 = double(two[0]);
    x1 = double(two[1]);
  } else if constexpr (sizeof(T) == 2) {
    x0 = double(__uint_as_float(r[i] << 16));
    x1 = double(__uint_as_float(r[i] & 0xFFFF0000u));
  } else {
    x0 = double(__uint_as_float(r[2 * i]));
    x1 = double(__uint_as_float(r[2 * i + 1]));
  }
}

// Data that one workgroup of decode_attend hands to another (the head's last workgroup) goes
// through agent-scope stores and loads: they write through / read around the per-XCD L2, so
// the hand-over needs no L2 write-back (a release fence at agent scope writes the whole L2
// back, once per workgroup, which costs more than the attention pass itself).
template <typename U>
__device__ __forceinline__ void st_agent(U* p, U v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename U>
__device__ __forceinline__ U ld_agent(const U* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float4 ld_agent4(const float* p) {  // 16 bytes as two 8-byte loads
  const uint64_t lo = ld_agent(reinterpret_cast<const uint64_t*>(p));
  const uint64_t hi = ld_agent(reinterpret_cast<const uint64_t*>(p) + 1);
  return make_float4(__uint_as_float(uint32_t(lo)), __uint_as_float(uint32_t(lo >> 32)),
                     __uint_as_float(uint32_t(hi)), __uint_as_float(uint32_t(hi >> 32)));
}

// Which entry of the call's layer list a flat chunk index belongs to (block-uniform), that entry's
// layer, first index and number of chunks.  The list is sorted by size, so the workgroups dispatched last belong to the
// smallest caches.  Unused entries of lay_off hold INT_MAX.  Every lane looks at one entry: three vector
// loads of the kernel arguments and a count of the lanes whose entry starts at or before x.  (As
// 63 scalar compares this was 186 vector and 300 scalar instructions per wavefront, a twelfth of
// the vector instructions of a chunk of the fp8 cache, whose launch is bound by their issue.)
struct LayerEntry {
  int first, layer, chunks;
};
__device__ __forceinline__ LayerEntry find_entry(const DecodeArgs& a, int x) {
  static_assert(kMaxLayersPerCall == 64, "an entry per lane");
  const int lane = threadIdx.x & 63, off = a.lay_off[lane], next = a.lay_off[lane + 1], id = a.lay_id[lane];
  const int e = __popcll(__ballot(x >= off)) - 1;  // (lay_off[0] is 0)
  const int first = __builtin_amdgcn_readlane(off, e);
  return LayerEntry{first, __builtin_amdgcn_readlane(id, e), __builtin_amdgcn_readlane(next, e) - first};
}

// (u larger, then position smaller) wins; slot < 0 means "no entry".
struct Best {
  double u;
  int pos, slot;
};
__device__ __forceinline__ bool better_match(double u, int p, int s, const Best& b) {
  return s >= 0 && (b.slot < 0 || u > b.u || (u == b.u && p < b.pos));
}
// Wavefront arg-max of that order for one entry per lane whose positions are all different and
// whose u is never below -1 (a cosine): largest u, then smallest position, then that lane's slot.
__device__ __forceinline__ Best fast_wave_best_match(double u, int pos, int slot) {
  const bool live = slot >= 0;
  const double umax = fast_wave_max(live ? u : -INFINITY);
  const bool top = live && u == umax;
  const int pmin = fast_wave_min(top ? pos : 0x7FFFFFFF);
  const unsigned long long who = __ballot(top && pos == pmin);
  if (who == 0ull) return Best{0.0, 0, -1};
  const int src = __ffsll((long long)who) - 1;
  return Best{umax, pmin, __builtin_amdgcn_readlane(slot, src)};
}
// (score smaller, then position larger) wins: the order in which tokens are evicted.
__device__ __forceinline__ bool evicts_before(double s, int p, int sl, const Best& b) {
  return sl >= 0 && (b.slot < 0 || s < b.u || (s == b.u && p > b.pos));
}
// Wavefront-wide first of that order, for one entry per lane whose positions are all different.
__device__ __forceinline__ Best fast_wave_first_evicted(const Best& b) {
  const bool live = b.slot >= 0;
  const double smin = -fast_wave_max(live ? -b.u : -INFINITY);
  const bool top = live && b.u == smin;
  const int pmax = -fast_wave_min(top ? -b.pos : 0x7FFFFFFF);
  const unsigned long long who = __ballot(top && b.pos == pmax);
  if (who == 0ull) return Best{0.0, 0, -1};
  const int src = __ffsll((long long)who) - 1;
  return Best{smin, pmax, __builtin_amdgcn_readlane(b.slot, src)};
}
// The eviction candidates of the first generation step of one head, chosen after prompt
// compression by a workgroup of NT threads: the kCand lowest scores among the cached tokens that are evictable when token
// `new_pos` arrives (Eq. 7-8 on count + 1 entries: neither sink nor inside the recent window).
// A prediction like the one every step makes for the next: a miss costs that step's closing
// workgroup a second pass over the keys and nothing else.
template <int NT>
__device__ __forceinline__ void first_candidates(const double* __restrict__ cscore, const int32_t* __restrict__ cpos,
                                                 int total, int recent, int new_pos, int n_sink, int32_t* __restrict__ cand) {
  constexpr int NW = NT / 64;
  __shared__ Best ex[NW];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  Best low[kCand + 1];
#pragma unroll
  for (int i = 0; i <= kCand; ++i) low[i] = Best{0.0, 0, -1};
  for (int j0 = tid; j0 < total; j0 += 4 * NT) {  // four entries in flight per thread
    double sc[4];
    int ps[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      sc[u] = cscore[min(j0 + u * NT, total - 1)];
      ps[u] = cpos[min(j0 + u * NT, total - 1)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + u * NT, p = ps[u];
      if (j < total && p >= n_sink && p <= new_pos - recent && evicts_before(sc[u], p, j, low[kCand - 1])) {
        low[kCand - 1] = Best{sc[u], p, j};
#pragma unroll
        for (int i = kCand - 1; i > 0; --i)
          if (evicts_before(low[i].u, low[i].pos, low[i].slot, low[i - 1])) {
            const Best t = low[i - 1];
            low[i - 1] = low[i];
            low[i] = t;
          }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kCand; ++r) {  // repeated block-wide extraction of the first in eviction order
    Best h = fast_wave_first_evicted(low[0]);
    __syncthreads();
    if (lane == 0) ex[w] = h;
    __syncthreads();
    h = ex[0];
#pragma unroll
    for (int i = 1; i < NW; ++i)
      if (evicts_before(ex[i].u, ex[i].pos, ex[i].slot, h)) h = ex[i];
    if (tid == 0) cand[r] = h.slot;
    if (h.slot >= 0 && low[0].slot == h.slot) {  // the owner pops its head
#pragma unroll
      for (int i = 0; i < kCand; ++i) low[i] = low[i + 1];
    }
  }
}

// This thread's elements of the two rows a step merges, the evicted one (ke, ve) and its match (kt, vt),
// as they were before the step; fp8 cache: with the rows' powers of two.  (Agent-scope loads: either may be
// the new token's row, written by another workgroup of the launch.)
template <typename T>
struct MergeRows {
  T ke, ve, kt, vt;
  int xke, xve, xkt, xvt;
};
template <typename T, int D>
__device__ __forceinline__ MergeRows<T> load_merge_rows(const DecodeArgs& a, int64_t slot0, int es, int bs) {
  MergeRows<T> r{};
  const int e = max(es, 0), t = max(bs, 0);
  if (threadIdx.x < D) {
    const T* Kc = static_cast<const T*>(a.cK) + slot0 * D + threadIdx.x;
    const T* Vc = static_cast<const T*>(a.cV) + slot0 * D + threadIdx.x;
    r.ke = ld_agent(Kc + int64_t(e) * D);
    r.ve = ld_agent(Vc + int64_t(e) * D);
    r.kt = ld_agent(Kc + int64_t(t) * D);
    r.vt = ld_agent(Vc + int64_t(t) * D);
  }
  if constexpr (sizeof(T) == 1) {
    r.xke = ld_agent(a.cKe + slot0 + e);
    r.xve = ld_agent(a.cVe + slot0 + e);
    r.xkt = ld_agent(a.cKe + slot0 + t);
    r.xvt = ld_agent(a.cVe + slot0 + t);
  }
  return r;
}
// Eq. 9 arg-max result -> Eq. 10 threshold, Eq. 11-12 merge with one source, slot bookkeeping.
// Called by every thread of a workgroup (at least D threads) with block-uniform arguments.
// (es, ep): the evicted slot and its position; (best, bp, bs): its match; told: the head's threshold
// before the step; (kl, vl): this thread's element of the last slot's row as it was before the step;
// (sl, pl): that slot's updated score and its position; mr: the two rows to merge.
template <typename T, int D>
__device__ __forceinline__ void finish_head(const DecodeArgs& a, int64_t lbh, int64_t slot0, int es, int ep, int total,
                                            double best, int bp, int bs, double told, T kl, T vl, double sl,
                                            int pl, const MergeRows<T>& mr, double* red) {
  T* Kc = static_cast<T*>(a.cK) + slot0 * D;
  T* Vc = static_cast<T*>(a.cV) + slot0 * D;
  const int tid = threadIdx.x, last = total - 1;
  bool do_merge;  // (never without a match: no cosine of a non-finite key compares above another)
  if (isnan(a.tau_force)) {
    const double tnew = isnan(told) ? best : __dadd_rn(__dmul_rn(a.beta, best), __dmul_rn(1.0 - a.beta, told));
    do_merge = bs >= 0 && best >= tnew;
    if (tid == 0) a.ctau[lbh] = tnew;
  } else {
    do_merge = bs >= 0 && best >= a.tau_force;
  }
  if (tid == 0) {
    a.ev_evicted[lbh] = ep;
    a.ev_target[lbh] = do_merge ? bp : -1;
    a.ev_ustar[lbh] = best;
    a.ccount[lbh] = last;
  }
  // exp(1), the retained token's self-similarity weight; average merging weighs both rows 1
  const double e1 = a.merge_average ? 1.0 : 2.718281828459045;
  const double w = a.merge_average ? 1.0 : exp(best);
  const double z = __dadd_rn(e1, w);
  if constexpr (sizeof(T) == 1) {
    // fp8 cache: rows are codes times the row's power of two.  The merged row is rounded to the
    // cache's logical type (bf16) and encoded again with a power of two of its own, which takes
    // its largest magnitude: a reduction over the workgroup (`red`: one double per wavefront).
    int8_t* Ke = a.cKe + slot0;
    int8_t* Ve = a.cVe + slot0;
    int ekl = ld_agent(Ke + last), evl = ld_agent(Ve + last);  // the last row's powers of two travel with its codes
    if (do_merge) {
      double km = 0.0, vm = 0.0;
      if (tid < D) {
        const double ke = Elem<T>::to_f64(mr.ke) * pow2_f64(mr.xke), ve = Elem<T>::to_f64(mr.ve) * pow2_f64(mr.xve);
        const double kt = Elem<T>::to_f64(mr.kt) * pow2_f64(mr.xkt), vt = Elem<T>::to_f64(mr.vt) * pow2_f64(mr.xvt);
        const double kk = __dadd_rn(__dmul_rn(e1, kt), __dmul_rn(w, ke));
        const double vv = __dadd_rn(__dmul_rn(e1, vt), __dmul_rn(w, ve));
        km = Elem<uint16_t>::to_f64(Elem<uint16_t>::from_f64(kk / z));
        vm = Elem<uint16_t>::to_f64(Elem<uint16_t>::from_f64(vv / z));
      }
      const double ak = wave_max(fabs(km)), av = wave_max(fabs(vm));
      __syncthreads();
      if ((tid & 63) == 0) {
        red[tid >> 6] = ak;
        red[4 + (tid >> 6)] = av;
      }
      __syncthreads();
      const int ek = fp8_row_exponent(fmax(fmax(red[0], red[1]), fmax(red[2], red[3])));
      const int ev = fp8_row_exponent(fmax(fmax(red[4], red[5]), fmax(red[6], red[7])));
      const T kc = fp8_encode(ldexp(km, -ek)), vc = fp8_encode(ldexp(vm, -ev));
      if (bs == last) {  // the merged row is the one that moves into the hole
        kl = kc;
        vl = vc;
        ekl = ek;
        evl = ev;
      } else {
        if (tid < D) {
          Kc[int64_t(bs) * D + tid] = kc;
          Vc[int64_t(bs) * D + tid] = vc;
        }
        if (tid == 0) {
          Ke[bs] = int8_t(ek);
          Ve[bs] = int8_t(ev);
        }
      }
    }
    if (es != last) {  // the last slot fills the hole
      if (tid < D) {
        Kc[int64_t(es) * D + tid] = kl;
        Vc[int64_t(es) * D + tid] = vl;
      }
      if (tid == 0) {
        Ke[es] = int8_t(ekl);
        Ve[es] = int8_t(evl);
      }
    }
  } else {
    if (tid < D) {
      if (do_merge) {
        const double kk = __dadd_rn(__dmul_rn(e1, Elem<T>::to_f64(mr.kt)), __dmul_rn(w, Elem<T>::to_f64(mr.ke)));
        const double vv = __dadd_rn(__dmul_rn(e1, Elem<T>::to_f64(mr.vt)), __dmul_rn(w, Elem<T>::to_f64(mr.ve)));
        const T km = Elem<T>::from_f64(kk / z), vm = Elem<T>::from_f64(vv / z);
        if (bs == last) {  // the merged row is the one that moves into the hole
          kl = km;
          vl = vm;
        } else {
          Kc[int64_t(bs) * D + tid] = km;
          Vc[int64_t(bs) * D + tid] = vm;
        }
      }
      if (es != last) {  // the last slot fills the hole
        Kc[int64_t(es) * D + tid] = kl;
        Vc[int64_t(es) * D + tid] = vl;
      }
    }
  }
  if (es != last && tid == 0) {
    a.cscore[slot0 + es] = sl;
    a.cpos[slot0 + es] = pl;
  }
}

// Sum over each group of N consecutive lanes (8, 16 or 32); every lane of the group gets it.
template <int N>
__device__ __forceinline__ double lane_group_sum(double v) {
  static_assert(N == 8 || N == 16 || N == 32, "lanes that share a row");
  v += dpp_f64<kDppXor1>(v);
  v += dpp_f64<kDppXor2>(v);
  v += dpp_f64<kDppHalfMirror>(v);
  if constexpr (N >= 16) v += dpp_f64<kDppMirror>(v);
  if constexpr (N == 32) v += __shfl_xor(v, 16, 64);
  return v;
}
// Cosine of the evicted key against every other row of the head (Eq. 9) by the whole workgroup;
// returns the arg-max per wavefront-reduced lane (the caller reduces over the wavefronts).
// ke: D doubles of shared memory, red: one double per wavefront.  NT = threads of the workgroup.
template <typename T, int D, int NT = 256>
__device__ __forceinline__ Best scan_matches(const DecodeArgs& a, int64_t slot0, int es, int total, double* ke,
                                             double* red) {
  constexpr int kVec = 16 / sizeof(T);
  constexpr int TPR = D / kVec;
  constexpr int RPP = NT / TPR;
  const int tid = threadIdx.x;
  const T* Kc = static_cast<const T*>(a.cK) + slot0 * D;
  double part = 0.0;
  __syncthreads();
  if (tid < D) {
    double x = Elem<T>::to_f64(Kc[int64_t(es) * D + tid]);
    if constexpr (sizeof(T) == 1) x *= pow2_f64(a.cKe[slot0 + es]);
    ke[tid] = x;
    part = x * x;
  }
  const double sne = sqrt(block_sum(part, red));
  const int tr = tid / TPR, tc = (tid % TPR) * kVec;
  Best m{0.0, 0, -1};
  // Four rows per group of TPR lanes are in flight (one at a time, 10000 rows took 0.5 ms); lane k of a
  // group then takes row k to its cosine, so that the square root and the division serve four rows.
  constexpr int U = 4;
  static_assert(TPR >= U, "a lane per row");
  const int own = min(tid % TPR, U - 1);
#pragma unroll 1
  for (int r0 = 0; r0 < total; r0 += U * RPP) {
    u32x4 raw[U];
#pragma unroll
    for (int k = 0; k < U; ++k)
      raw[k] = *reinterpret_cast<const u32x4*>(Kc + int64_t(min(r0 + k * RPP + tr, total - 1)) * D + tc);
    const int j = r0 + own * RPP + tr, jc = min(j, total - 1);
    const int p = a.cpos[slot0 + jc];
    double dot = 0.0, nr = 0.0;
#pragma unroll
    for (int k = 0; k < U; ++k) {
      double x[kVec], dk = 0.0, nk = 0.0;
      cvt16<T>(raw[k], x);
#pragma unroll
      for (int e = 0; e < kVec; ++e) {
        dk = fma(x[e], ke[tc + e], dk);
        nk = fma(x[e], x[e], nk);
      }
      dk = lane_group_sum<TPR>(dk);
      nk = lane_group_sum<TPR>(nk);
      dot = own == k ? dk : dot;
      nr = own == k ? nk : nr;
      __builtin_amdgcn_sched_barrier(0);  // one row after the other (registers)
    }
    if constexpr (sizeof(T) == 1) {  // the row's power of two: exact on sums that are exact
      const double sc = pow2_f64(a.cKe[slot0 + jc]);
      dot *= sc;
      nr *= sc * sc;
    }
    const double den = sne * sqrt(nr);
    const double u = den > 0.0 ? dot / den : 0.0;
    if (j < total && j != es && (tid % TPR) < U && better_match(u, p, j, m)) m = Best{u, p, j};
  }
  return m;
}


// Best match of candidate 0 over the workgroup's four wavefronts (their results are in LDS).
__device__ __forceinline__ Best candidate_match(const double* wcm_u, const int2* wcm_ps, int ci) {
  Best m{wcm_u[ci], wcm_ps[ci].x, wcm_ps[ci].y};
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    const int2 q = wcm_ps[i * kCand + ci];
    if (better_match(wcm_u[i * kCand + ci], q.x, q.y, m)) m = Best{wcm_u[i * kCand + ci], q.x, q.y};
  }
  return m;
}

// An entry more for the kCand + 1 first in eviction order.
__device__ __forceinline__ void insert_entry(Best (&a)[kCand + 1], const Best& x) {
  if (evicts_before(x.u, x.pos, x.slot, a[kCand])) {
    a[kCand] = x;
#pragma unroll
    for (int i = kCand; i > 0; --i)
      if (evicts_before(a[i].u, a[i].pos, a[i].slot, a[i - 1])) {
        const Best t = a[i - 1];
        a[i - 1] = a[i];
        a[i] = t;
      }
  }
}
// The two first of two sorted lists of two (no entry is in both): half the comparisons of two insertions.
__device__ __forceinline__ void join_entries(Best (&a)[2], const Best (&b)[2]) {
  auto pick = [](bool first, const Best& x, const Best& y) {
    return Best{first ? x.u : y.u, first ? x.pos : y.pos, first ? x.slot : y.slot};
  };
  const bool front = evicts_before(b[0].u, b[0].pos, b[0].slot, a[0]);
  const Best x = pick(front, a[0], b[0]), y = pick(front, b[1], a[1]);
  a[0] = pick(front, b[0], a[0]);
  a[1] = pick(evicts_before(x.u, x.pos, x.slot, y), x, y);
}
// The kCand + 1 first of the lists of a wavefront's lanes, in eviction order; `low` is used up.
__device__ __forceinline__ void wave_first_entries(Best (&low)[kCand + 1], Best (&out)[kCand + 1]) {
#pragma unroll
  for (int r = 0; r <= kCand; ++r) {
    out[r] = fast_wave_first_evicted(low[0]);
    if (out[r].slot >= 0 && low[0].slot == out[r].slot) {  // the owner pops its head
#pragma unroll
      for (int i = 0; i < kCand; ++i) low[i] = low[i + 1];
      low[kCand].slot = -1;
    }
  }
}

// The end of a head's closing work, by a workgroup of 256 threads, with block-uniform arguments: `ev`, the first evicted
// entry of the head; `nx`, the lowest entries evictable at the next step, in eviction order (`ev` may be among
// them); `cm`, this step's candidates' matches; the last slot's
// updated score and position (sred[4], ired[8]) and its row as it was before the step
// (`park_kv`: K at [0, D), V at [256, 256 + D)).  `mr` holds the rows of candidate 0 and of its best
// match (requested before the score pass, so that a step that evicts this candidate, which is the
// normal case, waits for no memory here).  The function writes the next step's
// candidates, resets the head's ticket, finds the merge target (from the candidates' results,
// else by a pass over the head's keys) and finishes the step.
template <typename T, int D>
__device__ __forceinline__ void close_head(const DecodeArgs& a, int64_t lbh, int64_t slot0, int total, bool evict,
                                           Best ev, const Best (&nx)[kCand + 1], const int (&cl)[kCand],
                                           const Best (&cm)[kCand], double told, double* sred, int* ired, double* dred,
                                           const T* park_kv, MergeRows<T> mr) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int last = total - 1;
  const double s_last = sred[4];
  const int p_last = ired[8];
  // (a candidate always exists: total > budget >= T + M; but where every score is NaN none compares below
  // another and the slot is -1: the new token leaves then)
  if (ev.slot < 0) {
    ev.slot = last;
    ev.pos = p_last;
  }
  const int es = evict ? ev.slot : -1;
  int ci = -1;
#pragma unroll
  for (int i = kCand - 1; i >= 0; --i)
    if (es >= 0 && cl[i] == es) ci = i;
  if (tid == 0) {  // the next step's candidates (every thread holds this step's list in registers)
    int k = 0;
#pragma unroll
    for (int r = 0; r <= kCand; ++r) {
      int s = nx[r].slot;
      if (k >= kCand || s < 0 || s == es) continue;
      if (es >= 0 && s == last) s = es;  // the last slot is about to move into the freed one
      a.cand[lbh * kCand + k++] = s;
    }
    for (; k < kCand; ++k) a.cand[lbh * kCand + k] = -1;
    st_agent(&a.ticket[lbh], 0u);
  }
  if (!evict) {
    if (tid == 0) {
      a.ccount[lbh] = total;
      a.ev_evicted[lbh] = -1;
      a.ev_target[lbh] = -1;
      a.ev_ustar[lbh] = __longlong_as_double(0x7FF8000000000000ll);
    }
    return;
  }
  Best m{0.0, 0, -1};
  if (ci < 0) {
    // Not foreseen (the first step after a cache import, or a candidate overtaken by a token
    // outside the list): a second pass over the head's keys.
    if (tid == 0) a.cmiss[lbh] += 1u;
    // (the new token's row and position were written by another workgroup of the launch: they are read after this)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    m = scan_matches<T, D>(a, slot0, es, total, dred, sred);
    m = fast_wave_best_match(m.u, m.pos, m.slot);
    lds_barrier();
    if (lane == 0) {
      sred[w] = m.u;
      ired[w] = m.pos;
      ired[4 + w] = m.slot;
    }
    lds_barrier();
    m = Best{sred[0], ired[0], ired[4]};
#pragma unroll
    for (int i = 1; i < 4; ++i)
      if (better_match(sred[i], ired[i], ired[4 + i], m)) m = Best{sred[i], ired[i], ired[4 + i]};
  } else {
#pragma unroll
    for (int i = 0; i < kCand; ++i)
      if (i == ci) m = cm[i];
  }
  if (ci != 0) mr = load_merge_rows<T, D>(a, slot0, es, m.slot);
  T kl = T(), vl = T();
  if (tid < D) {
    kl = park_kv[tid];
    vl = park_kv[256 + tid];
  }
  finish_head<T, D>(a, lbh, slot0, es, ev.pos, total, m.u, m.pos, m.slot, told, kl, vl, s_last, p_last, mr, sred);
}

// The two launches that close the heads with more than a.big_rows entries (decode_split.hip).
// `max_chunks[i]`: the chunks the largest head of the call's layer i can occupy in this step.
hipError_t launch_decode_split(d2o_ctx* c, const DecodeArgs& attend, const int* max_chunks, int nl, View out,
                               hipStream_t s);

}  // namespace dec

}  // namespace d2o
