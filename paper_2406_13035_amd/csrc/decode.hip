// One generation step over the compressed cache (Sec. 3 Eq. 2-3; Sec. 4.2 Eq. 6-12), for a
// range of layers in one launch (two more for very large heads).  The step reads every K and V row of
// every layer exactly once:
//
//   decode_attend   one workgroup per chunk of 256 slots, each of its four wavefronts working
//                   alone on 64 of them.  It lays out, in fp64 in LDS, the vectors that every cache key is
//                   multiplied with: the G queries and the keys of kCand eviction candidates chosen at the
//                   end of the previous step; the wavefront whose rows the new token's k, v fall among
//                   writes them into the free slot (score 0, its position).  (A launch of its own for
//                   both, before this one, cost a step 5 to 12 us: one layer per call, 32 layers took
//                   984 us instead of 875, a step of a 128-entry fp32 cache 17.1 instead of 15.1.)
//                   K pass: the keys go through LDS, and four lanes share
//                   four cache rows, a quarter of every 64 bytes each; they form, in fp64, the G
//                   logits, the dot products with the candidate keys and the rows' squared norms.
//                   Then, one row per lane, the softmax
//                   statistics of the 64 rows, the candidates' best cosine among them (Eq. 9),
//                   and the partial P V in fp32 on the matrix core.
//                   The last workgroup of a head to finish (a ticket counter, no waiting)
//                   closes the head: output rows, exact fp64 normaliser, score update (Eq. 6,
//                   generation case), the token to evict (Eq. 7-8: lowest score outside sinks
//                   and the recent window; equal scores evict the later position) and the
//                   candidates of the next step (the lowest scores that remain).  When the
//                   evicted token is one of this step's candidates, which is the normal case,
//                   its similarities are already there; otherwise (the first step after a cache
//                   import, or a candidate overtaken by a token outside the list) the same
//                   workgroup makes a second pass over the head's keys.  Then: arg-max (ties:
//                   earlier position), EMA threshold (Eq. 10, update first, then test), merge
//                   or discard (Eq. 11-12 with one source), and the last slot moves into the
//                   freed one.
//
// All decision-bearing arithmetic - logits, softmax normaliser, score accumulation, eviction
// arg-min, cosine arg-max, EMA threshold, merge - is fp64 in the operation order of the
// defining formulas; only the attention output (P V) accumulates in fp32.
// Slots are physically unordered; a token's identity is its position.
#include <algorithm>
#include <type_traits>

#include "decode_common.h"

namespace d2o {

// Scratch memory of d2o_decode_step_static: the partial results of one generation step, for callers
// that cannot hand over (or allocate) a scratch workspace.  One copy per GPU, held from the moment the library's code is loaded on it until the process ends.
// In host code the array's name is only a handle: the device address comes from
// hipGetSymbolAddress, once per device, and is what kernels and launchers are given.
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
unsigned char* g_static_scratch[kMaxDevices] = {};  // device address of `scratch` per device (0: not looked up yet)

}  // namespace

// Device address of the static scratch array on the current device (looked up on the first
// call per device; allocates nothing: the array is part of the loaded code object).
hipError_t static_scratch_address(unsigned char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  unsigned char* p = __atomic_load_n(&g_static_scratch[dev], __ATOMIC_ACQUIRE);
  if (!p) {
    void* sym = nullptr;
    e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!sym) return hipErrorInvalidSymbol;
    p = static_cast<unsigned char*>(sym);
    __atomic_store_n(&g_static_scratch[dev], p, __ATOMIC_RELEASE);  // every thread would store the same address
  }
  *out = p;
  return hipSuccess;
}

namespace {

using namespace dec;

// The type of q, k_new, v_new and (unless fp32 is asked for) of the outputs: the cache's own
// type, or bf16 when the cache holds fp8 codes.
template <typename T>
struct TensorType {
  typedef typename std::conditional<sizeof(T) == 1, uint16_t, T>::type type;
};

// This lane's share of a vector of D elements (elements E lane .. E lane + E - 1, E = D / 64) as loaded and as fp64.
template <typename U, int D>
struct LaneShare {
  static constexpr int E = D / 64;
  typedef typename std::conditional<E * sizeof(U) == 2, uint16_t, typename std::conditional<E * sizeof(U) == 4, uint32_t, uint64_t>::type>::type Bits;
  static __device__ __forceinline__ Bits load(const U* p, int lane) { return *reinterpret_cast<const Bits*>(p + E * lane); }
  static __device__ __forceinline__ void widen(Bits b, double (&x)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if constexpr (sizeof(U) == 4)
        x[e] = double(__uint_as_float(uint32_t(b >> (32 * e))));
      else
        x[e] = Elem<U>::to_f64(U(b >> (8 * int(sizeof(U)) * e)));
    }
  }
};

// Sum of the squares of a key's elements, E neighbours per lane.  Squares of bf16 elements and fp8 codes add up exactly in any
// order; those of fp32 elements do not, and where a candidate is the twin of its match a last bit of its norm can
// decide the threshold test (both 1 but for rounding), so their order is held (BY_HALVES): elements 32, 16, 8, 4, 2
// and 1 apart in every 64 of them.
template <bool BY_HALVES, int E>
__device__ __forceinline__ double square_sum(const double (&x)[E]) {
  if constexpr (!BY_HALVES) {
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) s = fma(x[e], x[e], s);
    return fast_wave_sum(s);
  } else if constexpr (E == 1) {
    const double s = x[0] * x[0];
    return half_wave_sum(s + __shfl_xor(s, 32, 64));
  } else {
    static_assert(E == 2, "one or two elements per lane");
    const double s = half_wave_sum(x[0] * x[0]) + half_wave_sum(x[1] * x[1]);
    return lane_f64(s, 0) + lane_f64(s, 32);
  }
}

// Softmax maximum and exact normaliser sum_j exp(s_j - max) of each query head of one head, from
// its sub-chunk records (fixed summation tree), by one workgroup of 256 threads of the launch
// that wrote the records; result: hn[g] = maximum, hn[G + g] = normaliser.
template <int G>
__device__ __forceinline__ void head_normaliser(const DecodeArgs& a, int64_t bh, int ch0, int nsub, double* hn,
                                                double* dred, double* sred) {
  constexpr int kRec = rec_doubles(G);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  double Mg[G], part[G];
#pragma unroll
  for (int g = 0; g < G; ++g) Mg[g] = -INFINITY;
  for (int c = tid; c < nsub; c += 256) {
    const int64_t x = sub_index(a, bh, ch0, c) * kRec;
#pragma unroll
    for (int g = 0; g < G; ++g) Mg[g] = fmax(Mg[g], ld_agent(&a.rec[x + g]));
  }
#pragma unroll
  for (int g = 0; g < G; ++g) Mg[g] = fast_wave_max(Mg[g]);
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) dred[w * G + g] = Mg[g];
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < G; ++g) {
    Mg[g] = fmax(fmax(dred[g], dred[G + g]), fmax(dred[2 * G + g], dred[3 * G + g]));
    part[g] = 0.0;
  }
  for (int c = tid; c < nsub; c += 256) {
    const int64_t x = sub_index(a, bh, ch0, c) * kRec;
#pragma unroll
    for (int g = 0; g < G; ++g) part[g] += ld_agent(&a.rec[x + G + g]) * exp(ld_agent(&a.rec[x + g]) - Mg[g]);
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const double wg = fast_wave_sum(part[g]);
    __syncthreads();
    if (lane == 0) sred[w] = wg;
    __syncthreads();
    if (tid == 0) {
      hn[g] = Mg[g];
      hn[G + g] = ((sred[0] + sred[1]) + sred[2]) + sred[3];
    }
  }
}

// Closing work of a head, by one workgroup of 256 threads: combine the sub-chunks, update the
// scores, choose the evicted token and the next candidates, find the merge target and finish the
// step.  What bounds it is its chain of memory round trips and workgroup-wide exchanges, so every
// load whose address does not depend on a result of this function is issued before the first of
// the reductions - the records, and the first batches of partial rows and of scores with their
// exp-logits - and the rows that a merge needs when the candidate is evicted as soon as the
// candidate's match is known.  (With each of them requested where it is used, and an exchange per
// evicted token and candidate, a head of 80 to 1900 entries took 18000 to 24700 cycles to close;
// issued one layer per call, 32 layers take 8 % less now, and a step of a 128-entry fp32 cache
// 17.5 instead of 19.2 us.  With two batches of the score pass in flight, the partial rows of all query heads
// requested together and one list of lowest scores instead of two, a layer of 8 heads of 5000
// entries takes 73 instead of 77 us, two steps of 24 layers with eight query heads per KV head 228 instead of 236.)
// With the normaliser, the factors and the match formed by every wavefront for itself where a head has at most 64
// sub-chunks, the matches' positions in the records and two instead of three reductions at the end, 32 layers one per call take
// 833 instead of 874 us, a step of a 128-entry fp32 cache 13.8 instead of 15.3; with such a head's output rows by a wavefront
// each, straight from registers, 812 and 12.6.  Calls of many layers hide most of the closing work: both changes together are
// 1500 -> 1495 us for two steps of 32 layers of 16 sequences, four query heads per KV head, and 845 -> 838 for one long context.
template <typename T, typename OT, int D, int G>
__device__ __forceinline__ void head_tail(const DecodeArgs& a, OT* __restrict__ out, const View& ov, int li, int b,
                                          int hk, int64_t lbh, int64_t slot0, int ch0, int total, int nsub, double* sred,
                                          int* ired, float* fred, double* dred, unsigned char* park) {
  constexpr int kRec = rec_doubles(G);
  constexpr int U = G >= 8 ? 1 : G >= 4 ? 2 : G >= 2 ? 4 : 6;  // slots per thread and batch of the score pass, of which two are in flight
  constexpr int C4 = D / 4;                           // threads across an output row (four columns each)
  constexpr int RG = 256 / C4;                        // groups of threads that share the sub-chunks
  // partial rows of each query head in flight per thread: four in all, or one each (eight query heads with
  // four rows each, one layer: 48.0 instead of 40.3 us at 1500 entries per head, 60.5 instead of 58.5 at 6000; 32 layers,
  // four sequences: 1093 instead of 1074 for two steps)
  constexpr int PB = G >= 4 ? 1 : G == 2 ? 2 : 4;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int last = total - 1;
  const int32_t* mt = a.meta + lbh * 4;
  const int64_t bh = int64_t(b) * a.Hkv + hk;
  const T* Kc = static_cast<const T*>(a.cK) + slot0 * D;
  const T* Vc = static_cast<const T*>(a.cV) + slot0 * D;
  // ---- loads that depend on nothing: the threshold, this step's candidates, the last slot's row
  const double told = a.ctau[lbh];
  int cl[kCand];
#pragma unroll
  for (int i = 0; i < kCand; ++i) cl[i] = a.cand[lbh * kCand + i];
  double e_last[G];
#pragma unroll
  for (int g = 0; g < G; ++g) e_last[g] = ld_agent(&a.elog[elog_index(a, bh, ch0, G, g, last)]);
  // Results that are needed only at the end wait in LDS, not in registers: per wavefront and
  // candidate the best match found so far (`wcm`), and the last slot's row (two elements per thread).
  double* wcm_u = sred + 8 + 8;                            // [4][kCand], behind sred and ired
  int2* wcm_ps = reinterpret_cast<int2*>(wcm_u + 4 * kCand);  // [4][kCand] (position, slot)
  T* park_kv = reinterpret_cast<T*>(wcm_ps + 4 * kCand);
  if (tid < D) {  // (the new token's row, written by another workgroup of this launch)
    park_kv[tid] = ld_agent(Kc + int64_t(last) * D + tid);
    park_kv[256 + tid] = ld_agent(Vc + int64_t(last) * D + tid);
  }
  constexpr int kEmCap = (kStageBytes - 8192) / int(sizeof(double));
  constexpr int kSegSubs = kEmCap / G;  // sub-chunks whose factors fit `em`
  // ---- the first batches of the output and score passes are requested now: they arrive while the
  //      normaliser is formed
  double sc[2][U], e[2][U][G];
  int ps[2][U];
  int seg0 = 0, jend = min(last, kSegSubs * kSub);  // the segment of sub-chunks whose factors `em` holds, and its last slot + 1 (without the new token's)
  auto load_batch = [&](auto set, int j0) {
    constexpr int s = decltype(set)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(j0 + u * 256, max(jend - 1, 0));
      sc[s][u] = a.cscore[slot0 + j];
      ps[s][u] = a.cpos[slot0 + j];
#pragma unroll
      for (int g = 0; g < G; ++g) e[s][u][g] = ld_agent(&a.elog[elog_index(a, bh, ch0, G, g, j)]);
    }
  };
  const std::integral_constant<int, 0> set0;
  const std::integral_constant<int, 1> set1;
  const int c4 = tid % C4, rg = tid / C4;
  const int nchunk = (nsub + 3) / 4;
  constexpr bool kEarlyRows = G <= 4;  // (eight query heads' rows would not fit the registers)
  float4 pr[G][PB];
  auto load_partial = [&](int g, int c0) {
#pragma unroll
    for (int u = 0; u < PB; ++u)
      pr[g][u] = ld_agent4(a.pacc + (chunk_index(a, bh, ch0, min(c0 + u * RG, nchunk - 1)) * G + g) * D + c4 * 4);
  };
  // ---- head maximum and exact normaliser sum_j exp(s_j - max) of each query head (fixed tree),
  //      all query heads in one sweep over the sub-chunk records.  exp(m_sub - max) of every
  //      sub-chunk and query head is kept in LDS (`em`, behind the parked values) for the output
  //      and score passes; for a head with more sub-chunks than fit, the factors overwrite the
  //      maxima in the records and the score pass brings them into LDS segment by segment.
  //      A head of up to 64 sub-chunks, which is the usual one: every wavefront does this for itself, a record per
  //      lane, with a table of its own, so that nothing waits for another wavefront.
  double* em = reinterpret_cast<double*>(park);  // [nsub][G]
  constexpr bool kByWave = G <= 4;               // (four tables of eight query heads do not fit)
  static_assert(!kByWave || 4 * 64 * G <= kEmCap, "four tables");
  const bool em_lds = nsub * G <= kEmCap;
  double Mg[G], Lg[G];
  Best cm[kCand];  // Eq. 9: this step's candidates' matches
  MergeRows<T> mr;
  if (kByWave && nsub <= 64) {
    em += w * 64 * G;
    const int64_t x = sub_index(a, bh, ch0, min(lane, nsub - 1)) * kRec;
    double m[G], l[G], u[kCand];
    int s[kCand], p[kCand];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      m[g] = ld_agent(&a.rec[x + g]);
      l[g] = ld_agent(&a.rec[x + G + g]);
    }
#pragma unroll
    for (int i = 0; i < kCand; ++i) {
      u[i] = ld_agent(&a.rec[x + 2 * G + i]);
      s[i] = int(ld_agent(&a.rec[x + 2 * G + kCand + i]));
      p[i] = int(ld_agent(&a.rec[x + 2 * G + 2 * kCand + i]));
    }
    uint64_t row[16];  // the partial rows of query head w: two columns per lane of every chunk
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      row[c] = 0;
      if (c < nchunk && w < G && lane * 2 < D)
        row[c] = ld_agent(reinterpret_cast<const uint64_t*>(a.pacc + (chunk_index(a, bh, ch0, c) * G + w) * D + lane * 2));
    }
    load_batch(set0, tid);
    const bool has = lane < nsub;
#pragma unroll
    for (int i = 0; i < kCand; ++i) cm[i] = fast_wave_best_match(u[i], p[i], has ? s[i] : -1);
    mr = load_merge_rows<T, D>(a, slot0, cl[0], cm[0].slot);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      Mg[g] = fast_wave_max(has ? m[g] : -INFINITY);
      const double t = has ? exp(m[g] - Mg[g]) : 0.0;
      Lg[g] = fast_wave_sum(has ? l[g] * t : 0.0);
      const double f = t / Lg[g];
      if (has) em[lane * G + g] = f;
      // ---- the output row of query head w (G <= 4): the order of additions is that of the groups of threads below,
      //      chunks r and r + RG first, then r = 0, 1, ...
      if (g == w) {
        double fc = has ? f : 0.0;  // exp(chunk maximum - max): the largest of its sub-chunks' factors
        fc = max_f64(fc, dpp_f64<kDppXor1>(fc));
        fc = max_f64(fc, dpp_f64<kDppXor2>(fc));
        const float cf = float(fc);
        float t0 = 0.f, t1 = 0.f;
#pragma unroll
        for (int r = 0; r < RG && r < 16; ++r) {
          float n0 = 0.f, n1 = 0.f;
#pragma unroll
          for (int c = r; c < 16; c += RG) {
            const float fr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cf), 4 * c));  // (0 past the last chunk)
            n0 = fmaf(__uint_as_float(uint32_t(row[c])), fr, n0);
            n1 = fmaf(__uint_as_float(uint32_t(row[c] >> 32)), fr, n1);
          }
          t0 = r ? t0 + n0 : n0;
          t1 = r ? t1 + n1 : n1;
        }
        if (lane * 2 < D) {
          OT* dst = out + li * ov.sn + b * ov.sb + (hk * G + g) * ov.sh + lane * 2;
          dst[0] = Elem<OT>::from_f32(t0);
          dst[1] = Elem<OT>::from_f32(t1);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    // The record of sub-chunk `tid` (the only one of this thread unless the head has more than 256
    // sub-chunks) is read once, whole, and kept: the sweeps below then cost one memory round trip
    // instead of three.
    double own_m[G], own_l[G], own_u[kCand];
    int own_s[kCand], own_p[kCand];
    {
#pragma unroll
      for (int g = 0; g < G; ++g) Mg[g] = -INFINITY;
      for (int c = tid; c < nsub; c += 256) {
        const int64_t x = sub_index(a, bh, ch0, c) * kRec;
        if (c == tid) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            own_m[g] = ld_agent(&a.rec[x + g]);
            own_l[g] = ld_agent(&a.rec[x + G + g]);
          }
#pragma unroll
          for (int i = 0; i < kCand; ++i) {
            own_u[i] = ld_agent(&a.rec[x + 2 * G + i]);
            own_s[i] = int(ld_agent(&a.rec[x + 2 * G + kCand + i]));
            own_p[i] = int(ld_agent(&a.rec[x + 2 * G + 2 * kCand + i]));
          }
#pragma unroll
          for (int g = 0; g < G; ++g) Mg[g] = fmax(Mg[g], own_m[g]);
        } else {
#pragma unroll
          for (int g = 0; g < G; ++g) Mg[g] = fmax(Mg[g], ld_agent(&a.rec[x + g]));
        }
      }
      if constexpr (kEarlyRows) {
#pragma unroll
        for (int g = 0; g < G; ++g) load_partial(g, rg);
      }
      load_batch(set0, tid);
#pragma unroll
      for (int g = 0; g < G; ++g) Mg[g] = fast_wave_max(Mg[g]);
      lds_barrier();
      if (lane == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) dred[w * G + g] = Mg[g];
      }
      lds_barrier();
#pragma unroll
      for (int g = 0; g < G; ++g) Mg[g] = fmax(fmax(dred[g], dred[G + g]), fmax(dred[2 * G + g], dred[3 * G + g]));
      double part[G];
#pragma unroll
      for (int g = 0; g < G; ++g) part[g] = 0.0;
      for (int c = tid; c < nsub; c += 256) {
        const int64_t x = sub_index(a, bh, ch0, c) * kRec;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const double t = exp((c == tid ? own_m[g] : ld_agent(&a.rec[x + g])) - Mg[g]);
          part[g] += (c == tid ? own_l[g] : ld_agent(&a.rec[x + G + g])) * t;
          if (em_lds)
            em[c * G + g] = t;
          else
            st_agent(&a.rec[x + g], t);  // the factor replaces the maximum (nobody needs it again)
        }
      }
      // (the tree of head_normaliser, all query heads in one exchange)
#pragma unroll
      for (int g = 0; g < G; ++g) part[g] = fast_wave_sum(part[g]);
      if (lane == 0) {
#pragma unroll
        for (int g = 0; g < G; ++g) dred[(4 + w) * G + g] = part[g];
      }
      if (em_lds)
        lds_barrier();
      else
        __syncthreads();  // the factors are in memory: the stores have been acknowledged
#pragma unroll
      for (int g = 0; g < G; ++g) Lg[g] = ((dred[4 * G + g] + dred[5 * G + g]) + dred[6 * G + g]) + dred[7 * G + g];
      // the table holds the factors already divided by the normaliser: a probability is then
      // one product, exp(s_j - m_sub) * em
      if (em_lds) {
        for (int c = tid; c < nsub; c += 256) {
#pragma unroll
          for (int g = 0; g < G; ++g) em[c * G + g] /= Lg[g];
        }
        lds_barrier();
      }
    }
    // ---- Eq. 9 arg-max over the sub-chunks' results, for every candidate of this step (which of
    //      them is evicted is not known yet; ties: earlier position)
#pragma unroll
    for (int i = 0; i < kCand; ++i) cm[i] = Best{0.0, 0, -1};
    for (int c = tid; c < nsub; c += 256) {
      const int64_t x = sub_index(a, bh, ch0, c) * kRec;
#pragma unroll
      for (int i = 0; i < kCand; ++i) {
        const int s = c == tid ? own_s[i] : int(ld_agent(&a.rec[x + 2 * G + kCand + i]));
        if (s >= 0) {
          const double u = c == tid ? own_u[i] : ld_agent(&a.rec[x + 2 * G + i]);
          const int p = c == tid ? own_p[i] : int(ld_agent(&a.rec[x + 2 * G + 2 * kCand + i]));
          if (better_match(u, p, s, cm[i])) cm[i] = Best{u, p, s};
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kCand; ++i) {  // (a thread's entries come from different sub-chunks: all positions differ)
      const Best r = fast_wave_best_match(cm[i].u, cm[i].pos, cm[i].slot);
      if (lane == 0) {
        wcm_u[w * kCand + i] = r.u;
        wcm_ps[w * kCand + i] = make_int2(r.pos, r.slot);
      }
    }
    lds_barrier();  // the wavefronts' matches are in LDS
#pragma unroll
    for (int i = 0; i < kCand; ++i) cm[i] = candidate_match(wcm_u, wcm_ps, i);
    mr = load_merge_rows<T, D>(a, slot0, cl[0], cm[0].slot);
    // ---- output rows: thread (rg, c4) adds the chunks rg, rg + RG, ... of four columns, PB of every query
    //      head in flight; the groups' sums are added in ascending order
    float num[G][4];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) num[g][e] = 0.f;
#pragma unroll 1
    for (int c0 = rg; c0 < nchunk; c0 += PB * RG) {
      if (!kEarlyRows || c0 != rg) {
#pragma unroll
        for (int g = 0; g < G; ++g) load_partial(g, c0);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float4(&v)[PB] = pr[g];
        double fc[PB];
#pragma unroll
        for (int u = 0; u < PB; ++u) {
          const int cc = min(c0 + u * RG, nchunk - 1);
          fc[u] = 0.0;  // exp(chunk maximum - max): the largest of its sub-chunks' factors
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (cc * 4 + i < nsub)
              fc[u] = fmax(fc[u], em_lds ? em[(cc * 4 + i) * G + g]
                                         : ld_agent(&a.rec[sub_index(a, bh, ch0, cc * 4 + i) * kRec + g]) / Lg[g]);
        }
#pragma unroll
        for (int u = 0; u < PB; ++u) {
          if (c0 + u * RG >= nchunk) break;
          const float f = float(fc[u]);
          num[g][0] = fmaf(v[u].x, f, num[g][0]);
          num[g][1] = fmaf(v[u].y, f, num[g][1]);
          num[g][2] = fmaf(v[u].z, f, num[g][2]);
          num[g][3] = fmaf(v[u].w, f, num[g][3]);
        }
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      lds_barrier();
#pragma unroll
      for (int e = 0; e < 4; ++e) fred[e * 256 + tid] = num[g][e];
      lds_barrier();
      if (tid < D) {  // column tid: element tid % 4 of the threads (rg, tid / 4)
        const float* fr = fred + (tid % 4) * 256 + tid / 4;
        float t = fr[0];
#pragma unroll
        for (int i = 1; i < RG; ++i) t += fr[i * C4];
        out[li * ov.sn + b * ov.sb + (hk * G + g) * ov.sh + tid] = Elem<OT>::from_f32(t);
      }
      __builtin_amdgcn_sched_barrier(0);  // one query head after the other (registers)
    }
  }
  const bool evict = total > mt[1];
  // Eq. 6 for the batch's slots, and the lowest scores of the tokens evictable at this step (Eq. 7-8 on count + 1
  // entries), in eviction order: the first is evicted, the others are the next step's candidates, together
  // with the token at position `next_out` + 1, which leaves the recent window then (`out`).
  const int next_out = a.new_pos - mt[2];  // the last evictable position
  Best low[kCand + 1];
#pragma unroll
  for (int i = 0; i <= kCand; ++i) low[i] = Best{0.0, 0, -1};
  double* out_s = sred + 5;  // the score and slot of `out` (-1 on entry)
  int* out_j = ired + 9;
  auto consider = [&](double x, int p, int j) {
    if (p >= a.n_sink && p <= next_out + 1) {
      if (p == next_out + 1) {
        *out_s = x;
        *out_j = j;
      } else {
        insert_entry(low, Best{x, p, j});
      }
    }
  };
  auto apply_batch = [&](auto set, int j0) {
    constexpr int s = decltype(set)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * 256;
      if (j < jend) {
        double s2 = sc[s][u];
#pragma unroll
        for (int g = 0; g < G; ++g) s2 = fma(e[s][u][g], em[(j / kSub - seg0) * G + g], s2);
        a.cscore[slot0 + j] = s2;
        consider(s2, ps[s][u], j);
      }
    }
  };
  // ---- score pass: batches of U slots per thread, the next one's loads in flight while one is worked on
#pragma unroll 1
  for (seg0 = 0; seg0 < nsub; seg0 += kSegSubs) {
    const int nseg = min(kSegSubs, nsub - seg0);
    jend = min(last, (seg0 + nseg) * kSub);
    if (!em_lds) {  // a head of several segments: (re)fill the table for this one
      lds_barrier();
#pragma unroll 1
      for (int i = tid; i < nseg * G; i += 256) {
        double lg = Lg[0];
#pragma unroll
        for (int g = 1; g < G; ++g) lg = (i % G == g) ? Lg[g] : lg;
        em[i] = ld_agent(&a.rec[sub_index(a, bh, ch0, seg0 + i / G) * kRec + i % G]) / lg;
      }
      lds_barrier();
    }
    const int j_lo = seg0 * kSub;
    if (seg0 > 0) load_batch(set0, j_lo + tid);
#pragma unroll 1
    for (int jb = j_lo; jb < jend; jb += 2 * U * 256) {
      if (jb + U * 256 < jend) load_batch(set1, jb + U * 256 + tid);
      apply_batch(set0, jb + tid);
      if (jb + U * 256 >= jend) break;
      if (jb + 2 * U * 256 < jend) load_batch(set0, jb + 2 * U * 256 + tid);
      apply_batch(set1, jb + U * 256 + tid);
    }
    if (tid == 0 && seg0 + nseg == nsub) {  // the new token: its score starts from its own probability
      double s2 = 0.0;
#pragma unroll
      for (int g = 0; g < G; ++g) s2 = fma(e_last[g], em[(last / kSub - seg0) * G + g], s2);
      a.cscore[slot0 + last] = s2;
      sred[4] = s2;  // kept for the move into the freed slot
      ired[8] = a.new_pos;
      consider(s2, a.new_pos, last);
    }
  }
  // ---- the wavefronts' lowest entries, joined by every thread: the first one is evicted, and the next step's
  //      candidates are the others and `out`
  constexpr int NE = kCand + 1;
  Best* ex = reinterpret_cast<Best*>(dred);  // [4][NE]
  static_assert(kCand == 1, "lists of two");
  Best nx[2];
  wave_first_entries(low, nx);
  if (lane == 0) {
    ex[w * NE] = nx[0];
    ex[w * NE + 1] = nx[1];
  }
  lds_barrier();
  {
    Best l1[2] = {ex[2], ex[3]}, l2[2] = {ex[4], ex[5]}, l3[2] = {ex[6], ex[7]};
    nx[0] = ex[0];
    nx[1] = ex[1];
    join_entries(nx, l1);
    join_entries(l2, l3);
    join_entries(nx, l2);
  }
  const Best ev = nx[0];
  if (*out_j >= 0) {
    if (evict) nx[0] = nx[1], nx[1].slot = -1;  // (the evicted entry is no candidate)
    insert_entry(nx, Best{*out_s, next_out + 1, *out_j});
  }
  close_head<T, D>(a, lbh, slot0, total, evict, ev, nx, cl, cm, told, sred, ired, dred, park_kv, mr);
}

// T: the cache's element type (uint8_t: fp8 codes).  (second launch bound: wavefronts per SIMD)
template <typename T, typename OT, int D, int G>
__global__ __launch_bounds__(256, G <= 4 && !(sizeof(T) == 4 && D == 128) ? 4 : 3) void decode_attend(
    DecodeArgs a, const typename TensorType<T>::type* __restrict__ q, View qv, const typename TensorType<T>::type* __restrict__ kn,
    View kv, const typename TensorType<T>::type* __restrict__ vn, View vv, OT* __restrict__ out, View ov) {
  typedef typename TensorType<T>::type IT;  // of q, k_new, v_new
  typedef LaneShare<IT, D> Share;
  typedef LaneShare<T, D> RowShare;
  constexpr int E = Share::E;
  constexpr int VB = sizeof(T) == 1 ? 8 : 16;   // V pass: bytes per lane and load (fp8: 8, which keeps the
                                                // partial sums at eight per lane and query head)
  constexpr int kVec = VB / sizeof(T);          // elements per load
  typedef typename RawBits<VB>::type VRaw;
  constexpr int RB = D * sizeof(T);             // bytes of a cache row
  constexpr int NP = RB / kPiece;               // row pieces staged through LDS
  constexpr int EL = 16 / sizeof(T);            // elements of a lane's 16 bytes of a piece
  constexpr int TPR = RB / VB;                  // V pass: lanes per row
  constexpr int RPI = 64 / TPR;                 // V pass: rows per load instruction
  constexpr int NVL = kSub / RPI;               // V pass: loads per lane
  constexpr bool kMmaV = sizeof(T) <= 2;        // V pass on the matrix core
  constexpr int NV = G + kCand;
  constexpr int CG = (NV + 1) / 4, NR = NV > 4 * CG ? NV - 4 * CG : 0;  // K pass: groups of four operand vectors, and vectors left over
  constexpr int kRec = rec_doubles(G);
  __shared__ __attribute__((aligned(16))) unsigned char stage[kStageBytes];
  // the operand vectors: a copy per wavefront where four fit (the wavefronts then stay independent
  // until they combine their results), else one for the workgroup, behind a barrier
  constexpr bool kOwnOpnd = G <= 2;
  __shared__ __attribute__((aligned(16))) double opnd[kOwnOpnd ? 4 : 1][NV * D];
  __shared__ double wmax[4][G];  // per wavefront: softmax maximum of its sub-chunk (-inf: no rows)
  __shared__ int sh_last;

  // Grid: x = head (fastest), y = flat chunk group over the layers.  Workgroups go round-robin to
  // the XCDs in index order, so with a head count that is a multiple of the XCD count every chunk
  // of a head, and the workgroup that closes it, run on one XCD.
  // (a call of one layer needs no search)
  const LayerEntry entry = a.nl == 1 ? LayerEntry{0, 0, int(gridDim.y)} : find_entry(a, blockIdx.y);
  const int li = entry.layer, grp = blockIdx.y - entry.first;
  const int l = a.layer0 + li, b = blockIdx.x / a.Hkv, hk = blockIdx.x % a.Hkv;
  const int64_t lbh = (int64_t(l) * a.B + b) * a.Hkv + hk;
  // Everything the workgroup needs to know about its head comes through the scalar cache in one
  // round trip (the loads are independent of each other): the fill level, the layer's slot and
  // sub-chunk offsets, the candidates.  The fill level changes when the head is closed, after every
  // workgroup of the head, the idle ones beyond its last row too, has drawn its ticket.
  typedef const int32_t __attribute__((address_space(4))) * ciptr;
  const ciptr mt = (ciptr)a.meta + lbh * 4;
  int count = ((ciptr)a.ccount)[lbh];
  const int mt0 = mt[0], mt3 = mt[3];
  int cs[kCand];
#pragma unroll
  for (int c = 0; c < kCand; ++c) cs[c] = ((ciptr)a.cand)[lbh * kCand + c];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the query heads whose operands this wavefront lays out: all of them, or every fourth
  constexpr int NQ = kOwnOpnd ? G : (G + 3) / 4;
  auto head_of = [&](int i) { return kOwnOpnd ? i : i * 4 + w; };
  const IT* const qh = q + li * qv.sn + b * qv.sb + int64_t(hk) * G * qv.sh;
  typename Share::Bits qraw[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) qraw[i] = Share::load(qh + min(head_of(i), G - 1) * qv.sh, lane);
  asm volatile("" : "+s"(count) : "s"(mt0), "s"(mt3));  // all of them are on their way before the first wait; count is read once
  const int total = count + 1;  // with the new token
  if (grp * kChunk < total) {
    const int64_t bh = int64_t(b) * a.Hkv + hk;
    const int64_t slot0 = bh * a.slots + mt0;
    const unsigned char* Kh = static_cast<const unsigned char*>(a.cK) + slot0 * RB;
    const unsigned char* Vh = static_cast<const unsigned char*>(a.cV) + slot0 * RB;
    // A workgroup owns a chunk of 256 slots; each wavefront works alone on 64 rows ("sub-chunk") of it:
    // while it computes on its keys, its V rows are in flight.
    unsigned char* mine = stage + w * kWaveStage;
    double* mine_opnd = opnd[kOwnOpnd ? w : 0];
    const int ln = lane;
    // K loads of a sub-chunk.  The K pass takes a row's bytes in pieces of 64 (one LDS staging round
    // each); the loads fetch two pieces at a time as whole 128-byte lines: 8 lanes per row, 8 rows
    // per load, 8 loads.  They are non-temporal like the V loads below: every K and V byte is
    // needed once per step, and a stream that does not settle in the caches leaves them to the
    // step's small read-write arrays (measured on a streaming probe with this access pattern:
    // 6.25 -> 6.7 TB/s; in 64-byte half lines the hint costs bandwidth instead, the second half
    // of a line then comes from memory again).  The next pair is requested as soon as this one
    // sits in LDS.
    static_assert(NP % 2 == 0, "pieces are loaded in pairs");
    // Both streams go through buffer descriptors that end with the wavefront's last row: rows past it
    // read as zero, and a load costs at most one address instruction (64-bit addresses of clamped rows
    // cost six, 190 of a bf16 chunk's 2300 vector instructions per wavefront).
    const int sub = __builtin_amdgcn_readfirstlane(grp * (kChunk / kSub) + w);
    const int rows = min(kSub, total - sub * kSub);  // <= 0: nothing for this wavefront
    // The new token's row: its wavefront (at most one of the head) writes it to the cache, puts its K among the staged
    // rows and takes its term of P V from registers; the streams end before it.
    const int jnew = count - sub * kSub;
    const bool owner = jnew >= 0 && jnew < kSub;
    const uint32_t cached = uint32_t(max(min(kSub, jnew), 0) * RB);
    const __amdgpu_buffer_rsrc_t Kb = buffer_of(Kh + int64_t(sub) * kSub * RB, cached);
    const __amdgpu_buffer_rsrc_t Vb = buffer_of(Vh + int64_t(sub) * kSub * RB, cached);
    u32x4 kreg[8];
    const uint32_t koff = (ln >> 3) * RB + (ln & 7) * 16;
    auto load_pair = [&](int p0) {
#pragma unroll
      for (int i = 0; i < 8; ++i) kreg[i] = stream16(Kb, koff + p0 * kPiece + i * 8 * RB);
    };
    // (the candidate's row is needed first, and loads arrive in order)
    typename RowShare::Bits craw[kCand];
    int cexp[kCand];
#pragma unroll
    for (int c = 0; c < kCand; ++c) {
      craw[c] = RowShare::load(static_cast<const T*>(a.cK) + (slot0 + max(cs[c], 0)) * D, lane);
      cexp[c] = sizeof(T) == 1 ? int(a.cKe[slot0 + max(cs[c], 0)]) : 0;
    }
    typename Share::Bits kraw = 0, vraw = 0;
    if (owner) {
      kraw = Share::load(kn + li * kv.sn + b * kv.sb + hk * kv.sh, lane);
      vraw = Share::load(vn + li * vv.sn + b * vv.sb + hk * vv.sh, lane);
    }
    if (rows > 0) load_pair(0);
    // ---- operands to LDS: queries, and the keys of the eviction candidates with their norms
    auto lay_out = [&](int v, const double (&x)[E]) {
      if constexpr (E == 2)
        *reinterpret_cast<double2*>(mine_opnd + operand_index<T, NV>(v, 2 * lane)) = make_double2(x[0], x[1]);
      else
        mine_opnd[operand_index<T, NV>(v, lane)] = x[0];
    };
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      double x[E];
      Share::widen(qraw[i], x);
      if (head_of(i) < G) lay_out(head_of(i), x);
    }
    double cn[kCand];
#pragma unroll
    for (int c = 0; c < kCand; ++c) {
      double x[E];
      RowShare::widen(craw[c], x);
#pragma unroll
      for (int e = 0; e < E; ++e) x[e] = cs[c] < 0 ? 0.0 : sizeof(T) == 1 ? x[e] * pow2_f64(cexp[c]) : x[e];
      if (kOwnOpnd || w == c % 4) lay_out(G + c, x);
      cn[c] = sqrt(square_sum<sizeof(T) == 4, E>(x));
    }
    if (!kOwnOpnd) lds_barrier();  // the operands are in LDS; the K rows may still be on their way
    // the new row's K and V as they enter the cache: K as stored, with an fp8 row's power of two, and V's values
    typename RowShare::Bits knew = 0;
    int kexp = 0;
    float vnew[E];
    if (owner) {
      double y[E];
      Share::widen(vraw, y);
      T* Kc = static_cast<T*>(a.cK) + (slot0 + count) * D;
      T* Vc = static_cast<T*>(a.cV) + (slot0 + count) * D;
      typename RowShare::Bits vst;
      if constexpr (sizeof(T) == 1) {
        // fp8 cache: encoded; the row's largest magnitude decides its power of two
        static_assert(E == 2, "two elements per lane");
        double x[E];
        Share::widen(kraw, x);
        const int ek = fp8_row_exponent(fast_wave_max(fmax(fabs(x[0]), fabs(x[1]))));
        const int ev = fp8_row_exponent(fast_wave_max(fmax(fabs(y[0]), fabs(y[1]))));
        kexp = ek;
        vst = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const uint8_t ck = fp8_encode(ldexp(x[e], -ek)), cv = fp8_encode(ldexp(y[e], -ev));
          knew |= typename RowShare::Bits(ck) << (8 * e);
          vst |= typename RowShare::Bits(cv) << (8 * e);
          vnew[e] = Elem<T>::to_f32(cv) * pow2_f32(ev);
        }
        if (lane == 0) {
          st_agent(a.cKe + slot0 + count, int8_t(ek));
          st_agent(a.cVe + slot0 + count, int8_t(ev));
        }
      } else {
        knew = kraw;
        vst = vraw;
#pragma unroll
        for (int e = 0; e < E; ++e) vnew[e] = float(y[e]);
      }
      // (write-through: the head's closing workgroup may read the row in this launch, and stores the score again)
      st_agent(reinterpret_cast<typename RowShare::Bits*>(Kc) + lane, knew);
      st_agent(reinterpret_cast<typename RowShare::Bits*>(Vc) + lane, vst);
      if (lane == 0) {
        st_agent(a.cscore + slot0 + count, 0.0);
        st_agent(a.cpos + slot0 + count, a.new_pos);
      }
    }
    if (rows <= 0) {  // this wavefront only takes part in the combination
      if (ln < G) wmax[w][ln] = -INFINITY;
    } else {
      const int tr = ln / TPR, tc = ln % TPR;
      // ---- K pass in the layout of v_mfma_f64_4x4x4_4b: D[i][j] += A[i][k] B[k][j] in four blocks b,
      // where lane i + 4 b + 16 k holds A, lane j + 4 b + 16 k holds B and lane j + 4 b + 16 i holds D.
      // i is one of four cache rows, j one of four operand vectors (queries, candidate keys), and k one
      // of the four 16-byte parts of a row piece: a lane takes its part's elements one after the other,
      // for four rows (set s of the staged rows holds rows s + 4 b + 16 i), so that an operand read
      // from LDS serves four products.  Four vectors go through the matrix instruction, which adds the parts
      // up; it does 16 products per cycle, like the vector ALU, so one or two
      // vectors, which would leave its columns empty, are multiplied there (with the squared norm) and
      // only added up by it, as products with ones.
      // Either way the lane's own row (its lane number) is one transposition inside a quad of lanes away.
      // With one row per lane and the operands as scalar loads, fetched a step ahead, a wavefront of a
      // small launch spent 12900 cycles here, most of them waiting for one cache line of operands after
      // the other (2 KB per head at G = 1); it now spends 5300.  Where the stream of K and V is the bound
      // both forms take the same time; issued one layer per call, 32 layers take 4.8 % less.
      double acc[4][CG > 0 ? CG : 1], part[4][NR + 1];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int c = 0; c < CG; ++c) acc[s][c] = 0.0;
#pragma unroll
        for (int c = 0; c <= NR; ++c) part[s][c] = 0.0;
      }
      const unsigned char* arow = mine + (((ln >> 2) & 3) * 4 + (ln & 3)) * kPitch + (ln >> 4) * 16;
      const double* bcol = mine_opnd + (min(ln & 3, NV - 1) * 4 + (ln >> 4)) * 2;  // vector ln % 4 of a group (three: the last one twice)
      const double* ball = mine_opnd + (CG * 16 + (ln >> 4)) * 2;       // first of the left-over vectors
      // the staging lanes' rows: i * 8 + t
      const int t = ln >> 3;
      unsigned char* srow = mine + (t & 3) * kSetBytes + (t >> 2) * 4 * kPitch + (ln & 3) * 16;
      // V rows (load i: rows i * RPI + tr): a bf16 or fp8 sub-chunk is requested whole, as far as the
      // registers allow during the last piece of the K pass (fp8 all of it, bf16 half) and the rest right after;
      // fp32 rows travel in quarters through two register sets.
      constexpr int VE = kMmaV ? (sizeof(T) == 1 ? NVL : NVL / 2) : NVL / 2;  // loads requested during the K pass
      constexpr int VQ = NVL / 4;
      VRaw vbuf[kMmaV ? NVL : NVL / 2];
      const uint32_t voff = tr * RB + tc * VB;
      auto load_v = [&](int i, int slot) { vbuf[slot] = stream_raw<VB>(Vb, voff + i * RPI * RB); };
      // this lane's score-side loads ride along
      const bool valid = ln < rows;
      const int j = sub * kSub + ln;
      const bool fresh = ln == jnew;  // (only in the new row's wavefront)
      const int pos = fresh ? a.new_pos : valid ? a.cpos[slot0 + j] : 0;
      // fp8 cache: the powers of two of this lane's K and V row
      int rek = 0, rev = 0;
      if constexpr (sizeof(T) == 1) {
        rek = fresh ? kexp : valid ? a.cKe[slot0 + j] : 0;
        rev = valid && !fresh ? a.cVe[slot0 + j] : -120;
      }
      constexpr int kShareLanes = kPiece / int(sizeof(knew));  // lanes that hold a piece of the new row
      auto stage_piece = [&](int p) {
        // The staging area is private to the wavefront and LDS serves a wavefront's requests in
        // order, so the piece hand-over needs compiler ordering only.
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (((ln >> 2) & 1) == (p & 1)) {  // the lanes that hold this piece's half of the lines
#pragma unroll
          for (int i = 0; i < 8; ++i)
            *reinterpret_cast<u32x4*>(srow + (((2 * i) & 3) * 4 + (i >> 1)) * kPitch) = kreg[i];
        }
        // The new row, over the zeros that were loaded in its place: its sums then have the order of every other
        // row's, so that twin keys tie (fp32 rows: an order of its own made the newer of two twins the
        // better match in a third of all cases).
        if (owner) {
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          if (ln / kShareLanes == p)
            *reinterpret_cast<typename RowShare::Bits*>(mine + (jnew & 3) * kSetBytes + (((jnew >> 2) & 3) * 4 + (jnew >> 4)) * kPitch +
                                                        ln % kShareLanes * int(sizeof(knew))) = knew;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      };
      auto multiply_piece = [&](int p) {
        u32x4 ar[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) ar[s] = *reinterpret_cast<const u32x4*>(arow + s * kSetBytes);
#pragma unroll
        for (int e = 0; e < EL / 2; ++e) {
          double2 bg[CG > 0 ? CG : 1], br[NR > 0 ? NR : 1];
#pragma unroll
          for (int c = 0; c < CG; ++c) bg[c] = *reinterpret_cast<const double2*>(bcol + (p * (EL / 2) + e) * NV * 8 + c * 32);
#pragma unroll
          for (int c = 0; c < NR; ++c) br[c] = *reinterpret_cast<const double2*>(ball + (p * (EL / 2) + e) * NV * 8 + c * 8);
#pragma unroll
          for (int s0 = 0; s0 < 4; s0 += 2) {  // two sets at a time: independent products, few registers
            double x0[2], x1[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              pair_f64<T>(ar[s0 + i], e, x0[i], x1[i]);
#pragma unroll
              for (int c = 0; c < CG; ++c)
                acc[s0 + i][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(x0[i], bg[c].x, acc[s0 + i][c], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              double(&ps)[NR + 1] = part[s0 + i];
#pragma unroll
              for (int c = 0; c < CG; ++c)
                acc[s0 + i][c] = __builtin_amdgcn_mfma_f64_4x4x4f64(x1[i], bg[c].y, acc[s0 + i][c], 0, 0, 0);
#pragma unroll
              for (int c = 0; c < NR; ++c) ps[c] = fma(x1[i], br[c].y, fma(x0[i], br[c].x, ps[c]));
              ps[NR] = fma(x1[i], x1[i], fma(x0[i], x0[i], ps[NR]));
            }
            __builtin_amdgcn_sched_barrier(0);  // interleaving more of them costs registers
          }
        }
      };
#pragma unroll 1
      for (int p = 0; p < NP - 1; ++p) {
        stage_piece(p);
        if (p & 1) load_pair(p + 1);
        multiply_piece(p);
      }
      stage_piece(NP - 1);
#pragma unroll
      for (int i = 0; i < VE; ++i) load_v(i, i);
      multiply_piece(NP - 1);
      if constexpr (kMmaV) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = VE; i < NVL; ++i) load_v(i, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      // every lane takes its own row's products
      auto own = [&](double v0, double v1, double v2, double v3) {
        const double lo = (ln & 1) ? v1 : v0, hi = (ln & 1) ? v3 : v2;
        return (ln & 2) ? hi : lo;
      };
      double dot[NV], nr;
#pragma unroll
      for (int c = 0; c <= NR; ++c) {
        double t4[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) t4[s] = __builtin_amdgcn_mfma_f64_4x4x4f64(part[s][c], 1.0, 0.0, 0, 0, 0);
        (c == NR ? nr : dot[CG * 4 + c]) = own(t4[0], t4[1], t4[2], t4[3]);
      }
#pragma unroll
      for (int c = 0; c < CG; ++c) {
        auto column = [&](auto jc) {  // operand vector 4 c + jc: lane jc of every quad holds its results
          constexpr int j = decltype(jc)::value, bcast = j * 0x55;
          if (4 * c + j < NV) dot[4 * c + j] = own(dpp_f64<bcast>(acc[0][c]), dpp_f64<bcast>(acc[1][c]),
                                                   dpp_f64<bcast>(acc[2][c]), dpp_f64<bcast>(acc[3][c]));
        };
        column(std::integral_constant<int, 0>{});
        column(std::integral_constant<int, 1>{});
        column(std::integral_constant<int, 2>{});
        column(std::integral_constant<int, 3>{});
      }
      if constexpr (sizeof(T) == 1) {
        // the K pass worked on the codes: the row's power of two scales its dot products and its
        // squared norm (exactly: the sums are exact, see the precision notes of the file header)
        const double sk = pow2_f64(rek);
#pragma unroll
        for (int v = 0; v < NV; ++v) dot[v] *= sk;
        nr *= sk * sk;
      }
      // ---- softmax statistics of the sub-chunk; the lane owns cache row sub*kSub + lane
      const int64_t pidx = sub_index(a, bh, mt3, sub) * G;
      double recv = 0.0;  // this lane's element of the sub-chunk record
      // The probabilities go to the staging area (the K pass is done with it) for the V pass: as fp32, or, for
      // its matrix products, each as three bf16 terms that add up to it exactly (an fp32 value has three times
      // eight significant bits) but for a power of two, in the order of their A operand: term t of query head g is row 3 g + t of
      // kTermPitch bytes, cache row r its element 16 (r % 4) + r / 4.
      constexpr int kTermPitch = 128 + 16;
      static_assert(!kMmaV || (RPI == 4 && 3 * G * kTermPitch <= kWaveStage), "the terms fit the staging area");
      float* psf = reinterpret_cast<float*>(mine);  // [G][kSub]
      unsigned char* const term = mine + ((ln & 3) * 16 + (ln >> 2)) * 2;
      // bf16 ends at 2^-133, an fp32 probability at 2^-149: the terms are those of the probability times 2^kTermScale, which
      // the sums are rid of again (unscaled, a probability of 2e-38 lost 9 of its bits, which a V element of 1e38 shows).
      // fp8 cache: the V pass works on the codes, so a row's power of two rides on its probability, taken
      // relative to the largest of the sub-chunk (which multiplies the sums: the terms keep their range).  These powers lie
      // up to 240 apart, and codes end at 448, 64 of which times 2^112 are finite.
      constexpr int kTermScale = sizeof(T) == 1 ? 112 : 24;
      const int rev_max = sizeof(T) == 1 ? -fast_wave_min(-rev) : 0;  // (-120, the smallest there is, in lanes without a cached row)
      float pnew[G];  // the new row's probabilities
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const double sg = div_root<D>(dot[g]);
        const double mx = fast_wave_max(valid ? sg : -INFINITY);
        const double e = valid ? exp(sg - mx) : 0.0;
        if constexpr (kMmaV) {
          const float p1 = sizeof(T) == 1 ? ldexpf(float(e), rev - rev_max + kTermScale) : float(e) * pow2_f32(kTermScale);
          const float p2 = p1 - __uint_as_float(__float_as_uint(p1) & 0xFFFF0000u);
          const float p3 = p2 - __uint_as_float(__float_as_uint(p2) & 0xFFFF0000u);
          *reinterpret_cast<uint16_t*>(term + (3 * g) * kTermPitch) = uint16_t(__float_as_uint(p1) >> 16);
          *reinterpret_cast<uint16_t*>(term + (3 * g + 1) * kTermPitch) = uint16_t(__float_as_uint(p2) >> 16);
          *reinterpret_cast<uint16_t*>(term + (3 * g + 2) * kTermPitch) = uint16_t(__float_as_uint(p3) >> 16);
        } else {
          psf[g * kSub + ln] = float(e);
        }
        if (owner) pnew[g] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(float(e)), jnew));
        if (valid) st_agent(&a.elog[elog_index(a, bh, mt3, G, g, j)], e);
        const double sm = fast_wave_sum(e);
        if (ln == g) {
          recv = mx;
          wmax[w][g] = mx;
        }
        if (ln == G + g) recv = sm;
      }
      // candidates: cosine of this row against each candidate key (Eq. 9), sub-chunk arg-max
      const double nrow = sqrt(nr);
#pragma unroll
      for (int c = 0; c < kCand; ++c) {
        const double den = cn[c] * nrow;
        const double u = den > 0.0 ? dot[G + c] / den : 0.0;
        const Best m = fast_wave_best_match(u, pos, (valid && cs[c] >= 0 && j != cs[c]) ? j : -1);
        if (ln == 2 * G + c) recv = m.u;
        if (ln == 2 * G + kCand + c) recv = double(m.slot);
        if (ln == 2 * G + 2 * kCand + c) recv = double(m.pos);
      }
      if (ln < kRec) st_agent(&a.rec[(pidx / G) * kRec + ln], recv);  // the record in one store
      // ---- partial P V.  The wavefront's partial rows (one per query head) go to its staging area for the
      // combination over the workgroup.
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      float* xch = reinterpret_cast<float*>(mine);
      if constexpr (kMmaV) {
        // On the matrix core, in fp32: v_mfma_f32_16x16x32_bf16 (lane l: A[l % 16][8 (l / 16) ..], B[8 (l / 16) ..][l % 16],
        // D[4 (l / 16) + r][l % 16]) multiplies the probabilities' terms, query head g's as its rows
        // 4 g .. 4 g + 2, with 32 V rows.  A lane holds eight columns of every fourth row, so instruction
        // j takes column j of every lane, and two rows' elements are one permutation away from a word
        // of its B operand.  The products are exact, the sums over the rows need no exchange between lanes.
        // (One multiply-add per element, query head and lane, and the sums over the row groups through
        // LDS: 780 vector instructions per wavefront with four query heads, 328 with an fp8 cache; now 100 and 120.)
        constexpr int GB = (G + 3) / 4;  // blocks of four query heads
        bf16x8 pa[GB][2];
#pragma unroll
        for (int gb = 0; gb < GB; ++gb)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            // (rows without a term repeat another; their sums are not used)
            const int g = min(gb * 4 + (tc >> 2), G - 1), t = min(tc & 3, 2);
            pa[gb][hf] = *reinterpret_cast<const bf16x8*>(mine + (3 * g + t) * kTermPitch + tr * 32 + hf * 16);
          }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        f32x4 o[GB][8];
#pragma unroll
        for (int j2 = 0; j2 < 4; ++j2) {  // columns 2 j2 and 2 j2 + 1 of the lane's eight
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            u32x4 b0, b1;
#pragma unroll
            for (int x = 0; x < 4; ++x) {  // rows 2 x and 2 x + 1 of the lane's eight
              const VRaw &r0 = vbuf[hf * 8 + 2 * x], &r1 = vbuf[hf * 8 + 2 * x + 1];
              uint32_t lo, hi;  // the two rows' columns, as bf16 pairs
              if constexpr (sizeof(T) == 1) {
                // (codes have four significant bits: exact in bf16)
                const uint32_t pair = __builtin_amdgcn_perm(r1[j2 / 2], r0[j2 / 2], j2 & 1 ? 0x07030602u : 0x05010400u);
                lo = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(pair, 1.0f, false));
                hi = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(pair, 1.0f, true));
              } else {
                lo = __builtin_amdgcn_perm(r1[j2], r0[j2], 0x05040100u);
                hi = __builtin_amdgcn_perm(r1[j2], r0[j2], 0x07060302u);
              }
              b0[x] = lo;
              b1[x] = hi;
            }
#pragma unroll
            for (int gb = 0; gb < GB; ++gb) {
              const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
              o[gb][2 * j2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[gb][hf], __builtin_bit_cast(bf16x8, b0),
                                                                      hf ? o[gb][2 * j2] : zero, 0, 0, 0);
              o[gb][2 * j2 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[gb][hf], __builtin_bit_cast(bf16x8, b1),
                                                                          hf ? o[gb][2 * j2 + 1] : zero, 0, 0, 0);
            }
          }
        }
        auto back = [&](float x) { return sizeof(T) == 1 ? ldexpf(x, rev_max - kTermScale) : x * pow2_f32(-kTermScale); };
        float all = 0.f;  // not finite if a sum is not
#pragma unroll
        for (int gb = 0; gb < GB; ++gb)
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const f32x4 d = o[gb][j];
            o[gb][j][0] = (d[2] + d[1]) + d[0];
            all += o[gb][j][0];
          }
        if (sizeof(T) == 2 && __ballot(!(fabsf(all) < INFINITY))) {
          // An infinite element of V meets terms that are zero, which makes NaN of what is infinite, and scaled sums may
          // overflow (from 2^104 on): the rows once more, two columns per lane, with each probability in one piece.
          float pv[G][2];
#pragma unroll
          for (int g = 0; g < G; ++g) pv[g][0] = pv[g][1] = 0.f;
#pragma unroll 1
          for (int r = 0; r < int(cached / RB); ++r) {
            const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(Vb, r * RB + ln * 4, 0, 0);
            const uint16_t* tp = reinterpret_cast<const uint16_t*>(mine) + (r & 3) * 16 + (r >> 2);
#pragma unroll
            for (int g = 0; g < G; ++g) {
              float p = 0.f;
#pragma unroll
              for (int t = 2; t >= 0; --t) p += __uint_as_float(uint32_t(tp[(3 * g + t) * (kTermPitch / 2)]) << 16);
              p = back(p);
              pv[g][0] = fmaf(p, __uint_as_float(x << 16), pv[g][0]);
              pv[g][1] = fmaf(p, __uint_as_float(x & 0xFFFF0000u), pv[g][1]);
            }
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
#pragma unroll
          for (int g = 0; g < G; ++g) *reinterpret_cast<float2*>(xch + g * D + ln * 2) = make_float2(pv[g][0], pv[g][1]);
        } else {
#pragma unroll
          for (int gb = 0; gb < GB; ++gb) {
            const int g = gb * 4 + tr;
            if (g < G) {
#pragma unroll
              for (int j = 0; j < 8; ++j) xch[g * D + tc * 8 + j] = back(o[gb][j][0]);
            }
          }
        }
      } else {
        // fp32 rows: TPR lanes per row, RPI rows per load, then a sum over the row groups
        float pv[G][kVec];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < kVec; ++e) pv[g][e] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
          for (int i = 0; i < VQ; ++i) {
            const int r = (q * VQ + i) * RPI + tr;
            const VRaw& x = vbuf[(q & 1) * VQ + i];
#pragma unroll
            for (int g = 0; g < G; ++g) {
              const float p = psf[g * kSub + r];  // 0 for rows beyond the end
#pragma unroll
              for (int e = 0; e < kVec; ++e) pv[g][e] = fmaf(p, __uint_as_float(x[e]), pv[g][e]);
            }
          }
          if (q + 2 < 4) {
#pragma unroll
            for (int i = 0; i < VQ; ++i) load_v((q + 2) * VQ + i, (q & 1) * VQ + i);
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int g = 0; g < G; ++g) {
#pragma unroll
          for (int e = 0; e < kVec; ++e) {
            float t = pv[g][e];
#pragma unroll
            for (int o = TPR; o < 64; o <<= 1) t += __shfl_xor(t, o, 64);
            pv[g][e] = t;
          }
          if (tr == 0) {
#pragma unroll
            for (int e = 0; e < kVec; ++e) xch[g * D + tc * kVec + e] = pv[g][e];
          }
        }
      }
      if (owner) {  // the new row's term
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < E; ++e) xch[g * D + E * lane + e] = fmaf(pnew[g], vnew[e], xch[g * D + E * lane + e]);
      }
    }
    // ---- one partial output row per chunk and query head: the four wavefronts' rows, each
    //      rescaled from its sub-chunk's maximum to the chunk's (fp32, like the rows themselves).
    //      A quarter of the partial-output bytes of a row per sub-chunk: on this chip a written
    //      byte costs the stream of K and V rows several read bytes.
    lds_barrier();
    for (int g = w; g < G; g += 4) {
      double mc = wmax[0][g];
#pragma unroll
      for (int i = 1; i < 4; ++i) mc = fmax(mc, wmax[i][g]);
      if (lane * 2 < D) {
        float o0 = 0.f, o1 = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const double mw = wmax[i][g];
          if (mw != -INFINITY) {
            const float f = expf(float(mw - mc));
            const float* xr = reinterpret_cast<const float*>(stage + i * kWaveStage) + g * D + lane * 2;
            o0 = fmaf(f, xr[0], o0);
            o1 = fmaf(f, xr[1], o1);
          }
        }
        const uint64_t two = uint64_t(__float_as_uint(o0)) | (uint64_t(__float_as_uint(o1)) << 32);
        st_agent(reinterpret_cast<uint64_t*>(a.pacc + (chunk_index(a, bh, mt3, grp) * G + g) * D + lane * 2), two);
      }
    }
  }  // (the workgroup has rows)
  // ---- ticket: the last workgroup of the head to arrive closes the head.  Every store above
  //      that it will read is a write-through store; they have completed once the memory
  //      counters are zero, before the barrier that precedes the ticket.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  // the staging area is free: it holds the closing code's exchange buffers
  float* fred = reinterpret_cast<float*>(stage);
  double* dred = reinterpret_cast<double*>(stage + 4 * 256 * sizeof(float));
  double* sred = dred + D;
  int* ired = reinterpret_cast<int*>(sred + 8);  // 16 words
  if (tid == 0) {
    sh_last = (__hip_atomic_fetch_add(&a.ticket[lbh], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
               unsigned(entry.chunks - 1)) ? 1 : 0;
    ired[9] = -1;  // (head_tail's `out`)
  }
  __syncthreads();
  if (!sh_last) return;
  // Consumer side of the hand-over.  The other workgroups' results (rec, elog, pacc) are read
  // below through ld_agent only, which goes around this XCD's L2 whatever the compiler does
  // with plain loads; this fence keeps the compiler from moving any load of the closing code
  // above the ticket.  Plain loads in the closing code are limited to data that no other
  // workgroup of this launch writes: ctau, cand, meta of this head, and cscore and cpos of its older slots.
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  if (tid == 0) a.ctotal[lbh] = total > a.big_rows ? total : 0;
  if (total > a.big_rows) {
    // A very large head: two more launches close it (decode_close_part / _final).  All its
    // sub-chunk records are there now, so this workgroup leaves them the head's softmax
    // maxima and exact normalisers (the sweep and summation tree of the single-workgroup form),
    // while other heads' chunks still stream.
    head_normaliser<G>(a, int64_t(b) * a.Hkv + hk, mt3, (total + kSub - 1) / kSub, a.hnorm + lbh * 16, dred, sred);
    return;
  }
  head_tail<T, OT, D, G>(a, out, ov, li, b, hk, lbh, (int64_t(b) * a.Hkv + hk) * a.slots + mt0, mt3, total,
                         (total + kSub - 1) / kSub, sred, ired, fred, dred, stage + 8192);
}

struct StepViews {
  View q, k, v, out;
};

template <typename T, typename OT, int D, int G>
hipError_t run_attend(d2o_ctx* c, const DecodeArgs& a, int flat_chunks, const StepViews& t, hipStream_t s) {
  typedef typename TensorType<T>::type IT;
  KernelTimer kt(c, D2O_K_DECODE_ATTEND, s);
  decode_attend<T, OT, D, G><<<dim3(a.B * a.Hkv, flat_chunks), 256, 0, s>>>(a, (const IT*)t.q.ptr, t.q, (const IT*)t.k.ptr, t.k,
                                                                           (const IT*)t.v.ptr, t.v, (OT*)t.out.ptr, t.out);
  return hipGetLastError();
}

template <typename T, int D, int G>
hipError_t run_decode(d2o_ctx* c, const DecodeArgs& a, int fc, const StepViews& t, hipStream_t s) {
  if (a.out_f32) return run_attend<T, float, D, G>(c, a, fc, t, s);
  return run_attend<T, typename TensorType<T>::type, D, G>(c, a, fc, t, s);
}

template <typename T, int D>
hipError_t run_decode_g(d2o_ctx* c, const DecodeArgs& a, int fc, const StepViews& t, hipStream_t s) {
  switch (a.G) {
    case 1: return run_decode<T, D, 1>(c, a, fc, t, s);
    case 2: return run_decode<T, D, 2>(c, a, fc, t, s);
    case 4: return run_decode<T, D, 4>(c, a, fc, t, s);
    case 8: return run_decode<T, D, 8>(c, a, fc, t, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int decode_candidates() { return kCand; }

// Sizes (in bytes, each rounded up to 256) of the four scratch arrays of a decode step, in the
// order elog, rec, pacc, part.
static void decode_scratch_sizes(const d2o_ctx* c, size_t (&sz)[4]) {
  const d2o_config& cf = c->cfg;
  const size_t B = cf.batch, L = cf.n_layers, Hq = cf.n_q_heads, Hkv = cf.n_kv_heads, d = cf.head_dim;
  const size_t G = Hq / Hkv, bh = B * Hkv, nch = c->nchunk_cap, nsub = nch * 4;
  sz[0] = nch * B * Hq * kChunk * sizeof(double);
  sz[1] = bh * nsub * rec_doubles(int(G)) * sizeof(double);  // one record per 64 slots
  sz[2] = bh * nch * G * d * sizeof(float);                  // one partial output row per chunk and query head
  sz[3] = (bh * nch * kPartRecDoubles + L * bh * 16) * sizeof(double);  // part records, then 16 doubles per head
  for (size_t& x : sz) x = (x + 255) & ~size_t(255);
}

size_t decode_static_scratch_need(const d2o_ctx* c) {
  size_t sz[4];
  decode_scratch_sizes(c, sz);
  return sz[0] + sz[1] + sz[2] + sz[3];
}
size_t decode_static_scratch_capacity() { return kStaticScratchBytes; }

hipError_t launch_decode(d2o_ctx* c, int layer0, int nl_all, View q, View k, View v, View out, int new_pos,
                         hipStream_t s, unsigned char* static_scratch) {
  const d2o_config& cf = c->cfg;
  DecodeArgs a;
  a.ccount = c->ccount;
  a.ctotal = c->ctotal;
  a.ctau = c->ctau;
  a.meta = c->meta;
  a.cK = c->cacheK;
  a.cV = c->cacheV;
  a.cKe = c->cKe;
  a.cVe = c->cVe;
  a.cscore = c->cscore;
  a.cpos = c->cpos;
  a.cand = c->ccand;
  a.ticket = c->cticket;
  a.cmiss = c->cmiss;
  a.elog = c->d_logit;
  a.rec = c->d_rec;
  a.pacc = c->d_pacc;
  a.part = c->d_part;
  if (static_scratch) {  // the same four arrays, carved from the library's static device array
    size_t sz[4];
    decode_scratch_sizes(c, sz);
    unsigned char* p = static_scratch;
    a.elog = reinterpret_cast<double*>(p);
    a.rec = reinterpret_cast<double*>(p += sz[0]);
    a.pacc = reinterpret_cast<float*>(p += sz[1]);
    a.part = reinterpret_cast<double*>(p += sz[2]);
  }
  a.ev_evicted = c->ev_evicted;
  a.ev_target = c->ev_target;
  a.ev_ustar = c->ev_ustar;
  a.slots = cf.slots_per_seq;
  a.B = cf.batch;
  a.Hkv = cf.n_kv_heads;
  a.G = cf.n_q_heads / cf.n_kv_heads;
  a.new_pos = new_pos;
  a.n_sink = cf.n_sink;
  a.out_f32 = cf.out_f32;
  a.merge_average = cf.merge_average;
  a.part_chunks = cf.split_rows > 0 ? std::min(8, std::max(1, cf.split_rows / (4 * kChunk))) : 8;
  a.beta = cf.beta;
  a.tau_force = cf.tau_force;
  // the per-layer tensors of one call are [layer][...]: groups of at most kMaxLayersPerCall
  for (int g0 = 0; g0 < nl_all; g0 += kMaxLayersPerCall) {
    const int nl = std::min(kMaxLayersPerCall, nl_all - g0);
    a.layer0 = layer0 + g0;
    a.nl = nl;
    int mc[kMaxLayersPerCall], chunk_id[kMaxLayersPerCall];
    const int nc = nl;
    int64_t rows = 0;  // cache rows this launch streams
    for (int i = 0; i < nl; ++i) {
      chunk_id[i] = i;
      mc[i] = 1;
      for (const auto& mt : c->layers[a.layer0 + i].meta) {
        mc[i] = std::max(mc[i], (mt.budget + 1 + kChunk - 1) / kChunk);
        rows += mt.budget + 1;
      }
    }
    // Which heads are too large for one closing workgroup.  A head's last workgroup closes it
    // while the other heads' chunks still stream, which costs nothing as long as the head is a
    // small part of the launch; a head that holds more than about half a percent of the
    // launch's rows (a few giant layers after Eq. 5, or a launch of one layer) would leave the
    // chip waiting for its closing workgroup, and is finished by the split kernels instead.
    a.hnorm = a.part + size_t(cf.batch) * cf.n_kv_heads * c->nchunk_cap * kPartRecDoubles;
    a.big_rows = cf.split_rows > 0 ? cf.split_rows
                                   : int(std::min<int64_t>(kMaxAutoSplitRows, std::max<int64_t>(kMinAutoSplitRows, rows / 200)));
    auto shift = [&](View x, int elem_bytes) {  // first layer of this group
      x.ptr = static_cast<char*>(x.ptr) + size_t(g0) * x.sn * elem_bytes;
      return x;
    };
    const int es = c->esize, os = cf.out_f32 ? 4 : c->esize;
    const StepViews tg{shift(q, es), shift(k, es), shift(v, es), shift(out, os)};
    hipError_t e;
    // ---- attention over the caches, one workgroup per 256 slots; the layers with most chunks first
    {
      std::stable_sort(chunk_id, chunk_id + nc, [&](int x, int y) { return mc[x] > mc[y]; });
      int flat = 0;
      for (int i = 0; i < nc; ++i) {
        a.lay_id[i] = chunk_id[i];
        a.lay_off[i] = flat;
        flat += mc[chunk_id[i]];
      }
      for (int i = nc; i <= kMaxLayersPerCall; ++i) a.lay_off[i] = i == nc ? flat : 0x7FFFFFFF;
      if (cf.cache_fp8)
        e = run_decode_g<uint8_t, 128>(c, a, flat, tg, s);
      else if (cf.dtype == D2O_BF16)
        e = run_decode_g<uint16_t, 128>(c, a, flat, tg, s);
      else if (cf.head_dim == 64)
        e = run_decode_g<float, 64>(c, a, flat, tg, s);
      else
        e = run_decode_g<float, 128>(c, a, flat, tg, s);
      if (e != hipSuccess) return e;
      // ---- heads too large for one closing workgroup (their entry count can reach budget + rows
      //      appended since): the same grid finishes them in parts
      bool big = false;
      for (int i = 0; i < nl; ++i) big = big || int64_t(mc[i]) * kChunk > a.big_rows;
      if (big) {
        e = launch_decode_split(c, a, mc, nl, tg.out, s);
        if (e != hipSuccess) return e;
      }
    }
  }
  return hipSuccess;
}

}  // namespace d2o
