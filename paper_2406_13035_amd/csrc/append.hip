// Multi-token append (a block of m new tokens on one layer's compressed caches).  Two stages:
// the block's attention (block_* kernels, further down: rows appended, every token's softmax row
// added to the scores, nothing evicted), then Eq. 7-12 once on every cache.  The second stage is
// the prompt-phase kernels of tokens.hip, which work on rows in ascending token position; a
// cache's slots are physically unordered, so this file lays every cache of the layer out in
// position order first:
//
//   rank_by_bits, rank_by_position   per (sequence, KV head): rank of every slot's position among the head's
//                      positions (positions are distinct), the ordered positions and fp64 scores,
//                      and the number of entries;
//   permute_rows       K and V rows of every slot to their rank in the ordered copy.
#include <type_traits>

#include "d2o_internal.h"
#include "device_utils.h"

namespace d2o {
namespace {

constexpr int kRankTile = 4096;  // positions held in LDS at a time

template <int U>  // slots per thread: 4 amortises the LDS reads on large caches, 1 gives small ones more workgroups
__global__ __launch_bounds__(256) void rank_by_position(const int32_t* __restrict__ ccount,   // the layer's [B][Hkv]
                                                        const int32_t* __restrict__ meta,     // the layer's [B][Hkv][4]
                                                        const double* __restrict__ cscore,
                                                        const int32_t* __restrict__ cpos, int32_t* __restrict__ rank,
                                                        int32_t* __restrict__ opos, double* __restrict__ oscore,
                                                        int32_t* __restrict__ on, int npad, int64_t slots) {
  __shared__ __attribute__((aligned(16))) int32_t tile[kRankTile];
  const int hk = blockIdx.x, b = blockIdx.y, Hkv = gridDim.x, tid = threadIdx.x;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int n = ccount[bh];
  const int64_t slot0 = bh * slots + meta[bh * 4 + 0];
  if (tid == 0 && blockIdx.z == 0) on[bh] = n;
  // A workgroup owns 256 U slots at a time (a thread U of them; the workgroups of a head stride
  // over its slots); all positions of the head pass through LDS tile by tile, and each owned
  // slot counts the smaller ones (all threads read the same LDS words, eight at a time).
  for (int j0 = blockIdx.z * 256 * U; j0 < n; j0 += gridDim.z * 256 * U) {
    int mine[U], cnt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * 256 + tid;
      mine[u] = j < n ? cpos[slot0 + j] : 0x7FFFFFFF;
      cnt[u] = 0;
    }
    for (int t0 = 0; t0 < n; t0 += kRankTile) {
      __syncthreads();
      const int lim = min(kRankTile, (n - t0 + 7) & ~7);  // the padding compares as "not smaller"
      for (int i = tid; i < lim; i += 256) tile[i] = t0 + i < n ? cpos[slot0 + t0 + i] : 0x7FFFFFFF;
      __syncthreads();
#pragma unroll 4
      for (int i = 0; i < lim; i += 8) {  // (unrolled: several LDS reads in flight)
        const int4 pa = *reinterpret_cast<const int4*>(&tile[i]), pb = *reinterpret_cast<const int4*>(&tile[i + 4]);
#pragma unroll
        for (int u = 0; u < U; ++u)
          cnt[u] += (pa.x < mine[u]) + (pa.y < mine[u]) + (pa.z < mine[u]) + (pa.w < mine[u]) + (pb.x < mine[u]) +
                    (pb.y < mine[u]) + (pb.z < mine[u]) + (pb.w < mine[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * 256 + tid;
      if (j < n) {
        rank[bh * npad + j] = cnt[u];
        opos[bh * npad + cnt[u]] = mine[u];
        oscore[bh * npad + cnt[u]] = cscore[slot0 + j];
      }
    }
  }
}

// The same for caches whose positions are all below 32 kBitWords: a set of the positions as bits in LDS, and the
// number of bits below a position is its rank.  One workgroup per head; comparing every slot with every other took 25 us
// for 32 heads of 2304 entries, this takes 6.
constexpr int kBitWords = 16384;  // 64 KB: positions up to 524287
__global__ __launch_bounds__(1024) void rank_by_bits(const int32_t* __restrict__ ccount, const int32_t* __restrict__ meta,
                                                     const double* __restrict__ cscore, const int32_t* __restrict__ cpos,
                                                     int32_t* __restrict__ rank, int32_t* __restrict__ opos,
                                                     double* __restrict__ oscore, int32_t* __restrict__ on, int npad,
                                                     int64_t slots, int nwords) {
  extern __shared__ uint32_t bits[];          // [nwords], a multiple of 1024
  int* below = reinterpret_cast<int*>(bits + nwords);  // [1024] bits in the words before thread t's
  __shared__ int wsum[16];
  const int hk = blockIdx.x, b = blockIdx.y, Hkv = gridDim.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int n = ccount[bh];
  const int64_t slot0 = bh * slots + meta[bh * 4 + 0];
  if (tid == 0) on[bh] = n;
  constexpr int U = 4;  // slots in flight per thread
  int outside = 0;
  for (int i = tid; i < nwords; i += 1024) bits[i] = 0;
  __syncthreads();
  for (int j0 = tid; j0 < n; j0 += U * 1024) {
    int p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) p[u] = cpos[slot0 + min(j0 + u * 1024, n - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = uint32_t(p[u]) < uint32_t(nwords) * 32u;
      if (!in) outside = 1;
      if (in && j0 + u * 1024 < n) atomicOr(&bits[p[u] >> 5], 1u << (p[u] & 31));
    }
  }
  // A position that the host does not know of (a captured call, replayed on a cache that was imported since): every slot
  // against every other.
  if (__syncthreads_or(outside)) {
    for (int j = tid; j < n; j += 1024) {
      const int p = cpos[slot0 + j];
      int r = 0;
      for (int i = 0; i < n; ++i) r += cpos[slot0 + i] < p;
      rank[bh * npad + j] = r;
      opos[bh * npad + r] = p;
      oscore[bh * npad + r] = cscore[slot0 + j];
    }
    return;
  }
  // thread t counts the words [t per, t per + per); a scan over the threads counts those before
  const int per = nwords / 1024;
  int mine = 0;
  for (int i = 0; i < per; ++i) mine += __popc(bits[tid * per + i]);
  int inc = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int off = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) off += i < w ? wsum[i] : 0;
  below[tid] = off + inc - mine;
  __syncthreads();
  for (int j0 = tid; j0 < n; j0 += U * 1024) {
    int p[U];
    double sc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      p[u] = cpos[slot0 + min(j0 + u * 1024, n - 1)];
      sc[u] = cscore[slot0 + min(j0 + u * 1024, n - 1)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * 1024;
      if (j >= n) continue;
      const int word = p[u] >> 5, t = word / per;
      int r = below[t] + __popc(bits[word] & ((1u << (p[u] & 31)) - 1u));
      for (int i = t * per; i < word; ++i) r += __popc(bits[i]);
      rank[bh * npad + j] = r;
      opos[bh * npad + r] = p[u];
      oscore[bh * npad + r] = sc[u];
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void permute_rows(const int32_t* __restrict__ on, const int32_t* __restrict__ meta,
                                                    const int32_t* __restrict__ rank, const T* __restrict__ cK,
                                                    const T* __restrict__ cV, T* __restrict__ oK, T* __restrict__ oV,
                                                    int npad, int d, int64_t slots) {
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int64_t bh = int64_t(b) * Hkv + hk;
  constexpr int kVec = 16 / sizeof(T);
  const int tpr = d / kVec, rows_per_blk = 256 / tpr;
  const int j = blockIdx.x * rows_per_blk + threadIdx.x / tpr;
  if (j >= on[bh]) return;
  const int c = (threadIdx.x % tpr) * kVec;
  const int64_t src = (bh * slots + meta[bh * 4 + 0] + j) * d + c;
  const int64_t dst = (bh * npad + rank[bh * npad + j]) * d + c;
  *reinterpret_cast<u32x4*>(oK + dst) = *reinterpret_cast<const u32x4*>(cK + src);
  *reinterpret_cast<u32x4*>(oV + dst) = *reinterpret_cast<const u32x4*>(cV + src);
}


// ---------------------------------------------------------------------------------------------
// Attention of a block of m new tokens over the cache (Sec. 3 Eq. 2-3, Eq. 6 for every token of
// the block, nothing evicted): the block's rows are appended first; query i*G + g (token i, query
// head g of the group) then attends to the cache's N - m old entries and to the block's tokens
// 0..i.  Logits, softmax and score accumulation in fp64 as in the generation step; P V in fp32.
// Both products are dense contractions (rows x queries x d, queries x d x rows) and run on the
// matrix cores: the fp64 16x16x4 instruction for the logits (its sums of products of bf16 or
// fp8 values are exact, so they do not depend on the order of the contraction), the bf16 16x16x32
// or, fp32 caches, fp32 16x16x4 instruction for P V.
//
//   block_begin   per head: appends the block's K, V rows (score 0, positions first_pos + i),
//                 lays the queries out as fp64 vectors, sets the entry count to N.
//   block_stats   per (head, 256 rows, slice of the queries): the rows are staged in LDS once; a
//                 wavefront takes tiles of 16 queries and forms their logits against the 256
//                 rows, 64 rows at a time; exp(logit - maximum of the 64 rows) of every one goes to
//                 memory; per query the maximum and exp-sum over the chunk's visible rows.
//   block_norm    per head and query: maximum and exact normaliser over the chunks.
//   block_apply   the same tiling: p = the stored exponential times exp(maximum of the 64 rows - maximum)
//                 / normaliser; per row the sum
//                 of the p of every query that sees it; the wavefront's 16 x d partial output
//                 tile over the 256 rows, accumulated in fp32 by the matrix instruction whose A
//                 operand is the probability tile as the logits' instruction left it.
//   block_scores  per row: score += the sums (Eq. 6).
//   block_finish  per head and query: the chunks' partial output rows added in ascending order.
// A head's queries are cut into up to kMaxQuerySlices slices that run as workgroups of their own
// (a block on a cache of a few thousand rows is too little work per head to fill the chip
// otherwise); a row's score then grows by the slices' sums in slice order.  The exponentials are kept, in fp64, because
// the logits and they are what bounds the block (the fp64 units): with both formed again in block_apply, 256 tokens on
// 2048-entry caches (32 heads) took 123 + 182 us in the two kernels, with 151 MB written and read 131 + 74 (46 since).  They
// have a place of kBlockTermBytes, or of four tiles, which the position-ordered copy takes afterwards: the query tiles go through the
// three kernels in as many passes as it takes.
//
// Register layouts of the two instructions (lane l, c = l % 16, kq = l / 16):
//   operands   A[i = c][k = kq], B[k = kq][j = c]
//   fp64 result register r: D[i = 4 r + kq][j = c]
//   fp32 result register r: D[i = 4 kq + r][j = c]
// so with rows as i and queries as j, lane l holds the logits of query c against the rows
// 16 t + 4 r + kq of a 64-row group (t = 0..3), and for fixed (t, r) these values, taken as the A
// operand of the fp32 instruction (i = query c, k = kq), meet the four consecutive rows
// 16 t + 4 r + kq of V as B.
constexpr int kQT = 16;  // queries per tile

template <typename T, typename IT, int D>
__global__ __launch_bounds__(256) void block_begin(const int32_t* __restrict__ ccount, int32_t* __restrict__ ctotal,
                                                   const int32_t* __restrict__ meta, T* __restrict__ cK,
                                                   T* __restrict__ cV, double* __restrict__ cscore,
                                                   int32_t* __restrict__ cpos, const IT* __restrict__ q, View qv,
                                                   const IT* __restrict__ kn, View kv, const IT* __restrict__ vn, View vv,
                                                   double* __restrict__ aq, int m, int G, int maxq, int first_pos,
                                                   int64_t slots) {
  const int hk = blockIdx.x, b = blockIdx.y, Hkv = gridDim.x;
  const int tid = blockIdx.z * 256 + threadIdx.x, nt = gridDim.z * 256;  // the head's work is strided over its workgroups
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int count = ccount[bh];  // the entry count moves to N in block_norm, when no workgroup of this launch reads it any more
  const int64_t slot0 = bh * slots + meta[bh * 4 + 0];
  if constexpr (sizeof(T) == sizeof(IT)) {  // (an fp8 cache gets its rows from block_rows_fp8)
    for (int x = tid; x < m * D; x += nt) {
      const int i = x / D, c = x % D;
      cK[(slot0 + count + i) * D + c] = kn[b * kv.sb + hk * kv.sh + int64_t(i) * kv.sn + c];
      cV[(slot0 + count + i) * D + c] = vn[b * vv.sb + hk * vv.sh + int64_t(i) * vv.sn + c];
    }
  }
  for (int i = tid; i < m; i += nt) {
    cscore[slot0 + count + i] = 0.0;
    cpos[slot0 + count + i] = first_pos + i;
  }
  const int nq = m * G, nq_pad = (nq + kQT - 1) / kQT * kQT;  // the queries of a last, partial tile are zero
  for (int x = tid; x < nq_pad * D; x += nt) {
    const int qi = x / D, c = x % D;
    double v = 0.0;
    if (qi < nq) v = Elem<IT>::to_f64(q[b * qv.sb + (hk * G + qi % G) * qv.sh + int64_t(qi / G) * qv.sn + c]);
    aq[(bh * maxq + qi) * D + c] = v;
  }
  if (tid == 0) ctotal[bh] = count + m;
}

template <typename T, int D>
struct BlockRows {
  static constexpr int RB = D * sizeof(T);   // bytes of a cache row
  static constexpr int kPitch = RB + 16;     // LDS pitch of a staged row (conflict-free for the operand reads below)
  static constexpr int kWaveBytes = 64 * kPitch;
  static constexpr int kRowsBytes = 4 * kWaveBytes;                 // the chunk's 256 rows
  static constexpr int kScaleBytes = sizeof(T) == 1 ? 256 * 12 : 0;  // fp8: the rows' powers of two (K as fp64, V as fp32)
  static constexpr int KS = D / 4;           // contraction steps of the logits
  static constexpr int CT = D / 16;          // output column tiles of P V (lane c holds columns CT c .. CT c + CT - 1)
  // The chunk's rows [r0, r0 + 256) of `src` (rows past `last` repeat it) into LDS, each
  // wavefront 64 of them, coalesced; fp8: the rows' powers of two behind them.
  static __device__ __forceinline__ void stage(const T* src, const int8_t* ke, const int8_t* ve, int64_t slot0, int r0,
                                               int last, unsigned char* smem, int tid) {
    const int lane = tid & 63, w = tid >> 6;
    unsigned char* mine = smem + w * kWaveBytes;
#pragma unroll
    for (int i = 0; i < RB / 16; ++i) {
      const int ch = i * 64 + lane, row = ch / (RB / 16), col = ch % (RB / 16);
      *reinterpret_cast<u32x4*>(mine + row * kPitch + col * 16) =
          *reinterpret_cast<const u32x4*>(src + (slot0 + min(r0 + w * 64 + row, last)) * D + col * (16 / sizeof(T)));
    }
    if constexpr (sizeof(T) == 1) {
      reinterpret_cast<double*>(smem + kRowsBytes)[tid] = pow2_f64(ke[slot0 + min(r0 + tid, last)]);
      reinterpret_cast<float*>(smem + kRowsBytes + 256 * 8)[tid] = pow2_f32(ve[slot0 + min(r0 + tid, last)]);
    }
    __syncthreads();
  }
  // element e of 16 bytes of a staged row as fp64 (fp8: the code, without the row's power of two)
  static constexpr int EL = 16 / sizeof(T);
  static __device__ __forceinline__ double elem(const u32x4& raw, int e) {
    if constexpr (sizeof(T) == 1) {
      const int wd = int(raw[e / 4]);
      return double(e % 4 == 0   ? __builtin_amdgcn_cvt_f32_fp8(wd, 0)
                    : e % 4 == 1 ? __builtin_amdgcn_cvt_f32_fp8(wd, 1)
                    : e % 4 == 2 ? __builtin_amdgcn_cvt_f32_fp8(wd, 2)
                                 : __builtin_amdgcn_cvt_f32_fp8(wd, 3));
    } else if constexpr (sizeof(T) == 2) {
      return double(__uint_as_float(e & 1 ? raw[e / 2] & 0xFFFF0000u : raw[e / 2] << 16));
    } else {
      return double(__uint_as_float(raw[e]));
    }
  }
  // The contraction takes a row's quarters side by side: step s multiplies element (D / 4) kq + s in
  // lane group kq, so that a lane reads its quarter of a row 16 bytes at a time.
  // The query tile's B operands: bq[s] = that element of query q0 + c.
  static __device__ __forceinline__ void load_queries(const double* aq_head, int q0, int lane, double (&bq)[KS]) {
    const double* qp = aq_head + int64_t(q0 + (lane & 15)) * D + (lane >> 4) * KS;
#pragma unroll
    for (int s = 0; s < KS; s += 2) {
      const double2 v = *reinterpret_cast<const double2*>(qp + s);
      bq[s] = v.x;
      bq[s + 1] = v.y;
    }
  }
  // Logits of the tile's 16 queries against the rows [64 g, 64 g + 64) of the chunk:
  // S[t][r] = (row 64 g + 16 t + 4 r + kq) . (query c) / sqrt(d) (fp8: times the row's power of two, exactly).
  static __device__ __forceinline__ void logits(const unsigned char* smem, int g, int lane, const double (&bq)[KS],
                                                f64x4 (&S)[4]) {
    const int c = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) S[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < KS; s += EL) {
      u32x4 raw[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        raw[t] = *reinterpret_cast<const u32x4*>(smem + (g * 64 + t * 16 + c) * kPitch + kq * (RB / 4) + s * int(sizeof(T)));
#pragma unroll
      for (int e = 0; e < EL; ++e)
#pragma unroll
        for (int t = 0; t < 4; ++t) S[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(elem(raw[t], e), bq[s + e], S[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double v = S[t][r];
        if constexpr (sizeof(T) == 1) v *= reinterpret_cast<const double*>(smem + kRowsBytes)[g * 64 + t * 16 + 4 * r + kq];
        S[t][r] = div_root<D>(v);
      }
  }
};

// The logits of rows this lane's query does not see (behind the last row, or later block tokens) to minus
// infinity, whose exponential is zero: the exponentials of a tile are then one straight run of
// instructions (each behind a branch of its own, they ran one after the other).  `last`: the last row it
// sees; tile_last: the last row that all queries of the tile see; j0: the row of S[0][0].
__device__ __forceinline__ void mask_logits(f64x4 (&S)[4], int j0, int last, int group_last, int tile_last) {
  if (group_last <= tile_last) return;  // (the same for the wavefront)
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (j0 + t * 16 + 4 * r > last) S[t][r] = -INFINITY;
}

// sum / maximum over the four lanes that hold the same query column (kq = 0..3)
__device__ __forceinline__ double kq_max(double v) {
  v = fmax(v, __shfl_xor(v, 16, 64));
  return fmax(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ double kq_sum(double v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// Sums of sixteen values per lane over the sixteen lanes c of a lane group: every exchange also halves the
// number of values a lane still adds up, and lane c ends with the sum of value
// c / 8 + 2 (c % 2) + 4 (c / 2 % 2) + 8 (c / 4 % 2) (seven instructions per exchange; sixteen butterflies
// through the LDS permutation cost eight LDS instructions each).
__device__ __forceinline__ int row16_sums_owner(int c) { return (c >> 3 & 1) | (c & 1) << 1 | (c >> 1 & 1) << 2 | (c >> 2 & 1) << 3; }
__device__ __forceinline__ double row16_sums(const double (&v)[16], int c) {
  constexpr int kRor8 = 0x128, kShl4 = 0x104, kShr4 = 0x114;  // rotation by 8 lanes, shifts by 4, inside a row of 16
  double a[8], b[4], d[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const double keep = c & 8 ? v[2 * i + 1] : v[2 * i], send = c & 8 ? v[2 * i] : v[2 * i + 1];
    a[i] = keep + dpp_f64<kRor8>(send);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double keep = c & 1 ? a[2 * i + 1] : a[2 * i], send = c & 1 ? a[2 * i] : a[2 * i + 1];
    b[i] = keep + dpp_f64<kDppXor1>(send);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = c & 2 ? b[2 * i + 1] : b[2 * i], send = c & 2 ? b[2 * i] : b[2 * i + 1];
    d[i] = keep + dpp_f64<kDppXor2>(send);
  }
  const double keep = c & 4 ? d[1] : d[0], send = c & 4 ? d[0] : d[1];
  const double up = dpp_f64<kShl4>(send), down = dpp_f64<kShr4>(send);  // from lane c + 4 and from lane c - 4
  return keep + (c & 4 ? down : up);
}

// How the four wavefronts of a workgroup share a slice's query tiles [t_lo, t_hi) and a chunk's 64-row groups: a tile
// each, round by round; a slice of one or two tiles (a short block) gives a tile `share` wavefronts, which
// take its groups in turn and combine their results.  (One wavefront per tile: 214 us for 16 tokens
// on 2048-entry caches, 32 heads; now 190.)
struct WaveWork {
  int share, tile, group;  // wavefronts per tile, this wavefront's (first) tile and first group
};
__device__ __forceinline__ WaveWork wave_work(int w, int t_lo, int t_hi) {
  const int share = t_hi - t_lo == 1 ? 4 : t_hi - t_lo == 2 ? 2 : 1;
  return WaveWork{share, t_lo + w / share, w % share};
}

// Place of the exponentials of row `row` of a chunk (256 rows) and query tile (counted from the pass's first):
// [tile][chunk][head][256 rows][16 queries], so that the sixteen lanes of a row, and the four rows of an
// instruction, are 512 bytes side by side.
__device__ __forceinline__ int64_t term_index(int tile, int nch, int chunk, int heads, int bh, int row) {
  return (((int64_t(tile) * nch + chunk) * heads + bh) * kChunk + row) * kQT;
}

template <typename T, int D>
__global__ __launch_bounds__(256) void block_stats(const int32_t* __restrict__ ctotal, const int32_t* __restrict__ meta,
                                                   const T* __restrict__ cK, const int8_t* __restrict__ cKe,
                                                   const double* __restrict__ aq, double* __restrict__ stat,
                                                   double* __restrict__ gmax, double* __restrict__ term, int m, int G,
                                                   int maxq, int64_t slots, int tile0, int tile1, int tiles_per_slice) {
  typedef BlockRows<T, D> BR;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int bhN = gridDim.x, bh = blockIdx.x, chunk = blockIdx.y;
  const int N = ctotal[bh];
  if (chunk * kChunk >= N) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, kq = lane >> 4;
  const int64_t slot0 = int64_t(bh) * slots + meta[bh * 4 + 0];
  const int nc = N - m, nq = m * G;
  BR::stage(cK, cKe, cKe, slot0, chunk * kChunk, N - 1, smem, tid);
  const int ngroup = min(4, (N - chunk * kChunk + 63) / 64);  // 64-row groups of the chunk that hold rows
  const int t_lo = tile0 + blockIdx.z * tiles_per_slice, t_hi = min(tile1, t_lo + tiles_per_slice);
  const WaveWork ww = wave_work(w, t_lo, t_hi);
  for (int qt = ww.tile; qt < t_hi; qt += 4) {  // this wavefront's query tiles
    const int q0 = qt * kQT, query = q0 + c;
    double bq[BR::KS];
    BR::load_queries(aq + int64_t(bh) * maxq * D, q0, lane, bq);
    const int seen = min(nc + query / G, N - 1);  // the last row this query attends to
    const int tile_last = min(nc + q0 / G, N - 1);
    double M = -INFINITY, L = 0.0;
#pragma unroll 1
    for (int g = ww.group; g < ngroup; g += ww.share) {
      f64x4 S[4];
      BR::logits(smem, g, lane, bq, S);
      const int j0 = chunk * kChunk + g * 64 + kq;
      mask_logits(S, j0, seen, chunk * kChunk + g * 64 + 63, tile_last);
      double mg = -INFINITY;  // (stays so where every logit is NaN: rows with NaN keys leave the others' probabilities alone)
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) mg = max_f64(mg, S[t][r]);
      mg = kq_max(mg);
      // (a query that sees no row of the group: its exponentials are zero relative to any finite value)
      const double ref = mg == -INFINITY ? 0.0 : mg;
      double lt[4] = {0.0, 0.0, 0.0, 0.0};
      double* const to = term + term_index(qt - tile0, gridDim.y, chunk, bhN, bh, g * 64 + kq) + c;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double e = exp(S[t][r] - ref);
          lt[r] += e;
          to[(16 * t + 4 * r) * kQT] = e;
        }
      if (kq == 0) gmax[((int64_t(chunk) * bhN + bh) * maxq + query) * 4 + g] = mg;  // (maxq is a whole number of tiles)
      const double lg = kq_sum((lt[0] + lt[1]) + (lt[2] + lt[3]));
      const double Mn = fmax(M, mg);
      if (Mn == -INFINITY) continue;
      L = (M == -INFINITY ? 0.0 : L * exp(M - Mn)) + (mg == -INFINITY ? 0.0 : lg * exp(mg - Mn));
      M = Mn;
    }
    if (ww.share > 1) {  // (one round, all wavefronts take part)
      double2* ml = reinterpret_cast<double2*>(smem);  // [4][16]: the rows are done with
      __syncthreads();
      if (kq == 0) ml[w * 16 + c] = make_double2(M, L);
      __syncthreads();
      M = -INFINITY;
      L = 0.0;
      for (int i = 0; i < ww.share; ++i) {  // in group order, the same for all sharers
        const double2 o = ml[(w / ww.share * ww.share + i) * 16 + c];
        const double Mn = fmax(M, o.x);
        if (Mn == -INFINITY) continue;
        L = (M == -INFINITY ? 0.0 : L * exp(M - Mn)) + (o.x == -INFINITY ? 0.0 : o.y * exp(o.x - Mn));
        M = Mn;
      }
    }
    if (ww.group == 0 && kq == 0 && query < nq) {
      double* st = stat + ((int64_t(chunk) * bhN + bh) * maxq + query) * 2;
      st[0] = M;
      st[1] = L;
    }
  }
}

__global__ __launch_bounds__(256) void block_norm(const int32_t* __restrict__ ctotal, int32_t* __restrict__ ccount,
                                                  const double* __restrict__ stat, double* __restrict__ norm, int q0, int q1,
                                                  int maxq) {
  const int bhN = gridDim.x, bh = blockIdx.x;
  const int N = ctotal[bh], nch = (N + kChunk - 1) / kChunk;
  if (threadIdx.x == 0) ccount[bh] = N;
  for (int q = q0 + threadIdx.x; q < q1; q += 256) {
    double M = -INFINITY;
#pragma unroll 4
    for (int c = 0; c < nch; ++c) M = fmax(M, stat[((int64_t(c) * bhN + bh) * maxq + q) * 2]);
    double L = 0.0;
    for (int c = 0; c < nch; ++c) {
      const double* st = stat + ((int64_t(c) * bhN + bh) * maxq + q) * 2;
      if (st[0] != -INFINITY) L += st[1] * exp(st[0] - M);
    }
    norm[(int64_t(bh) * maxq + q) * 2] = M;
    norm[(int64_t(bh) * maxq + q) * 2 + 1] = L;
  }
}

// P V: what bounded this kernel was the fp32 matrix instruction (half the time of the logits' products).  The
// elements of a bf16 or 8-bit V are bf16 numbers and an fp32 probability is the sum of three (three times eight
// significant bits), so with these types it is three products of the bf16 instruction, exact, with fp32 sums: 74 -> 46 us
// for 256 tokens on 2048-entry caches, 32 heads, and two thirds of the former error against 64 bits.  A probability is
// scaled by 2^kTermScale, which keeps its last term above 2^-126, and the sums are rid of it again.  (bf16: three of the 168
// registers that three wavefronts per SIMD leave are spilled.)
constexpr int kTermScale = 24;
constexpr uint32_t kHighHalves = 0x07060302u, kLowHalves = 0x05040100u;  // v_perm_b32: two words' upper, lower halves
template <typename T, int D>
__global__ __launch_bounds__(256, sizeof(T) == 4 && D == 128 ? 2 : 3) void block_apply(const int32_t* __restrict__ ctotal, const int32_t* __restrict__ meta,
                                                   const T* __restrict__ cV, const int8_t* __restrict__ cVe,
                                                   double* __restrict__ spart, const double* __restrict__ norm,
                                                   const double* __restrict__ gmax, const double* __restrict__ term,
                                                   float* __restrict__ pout, int m, int G, int maxq, int64_t slots,
                                                   int rows_cap, int tile0, int tile1, int tiles_per_slice) {
  constexpr int CT = D / 16;  // output column tiles (lane c holds columns CT c .. CT c + CT - 1)
  constexpr int RB = D * int(sizeof(T));  // bytes of a cache row
  constexpr int VW = CT * int(sizeof(T)) / 4;
  static_assert(VW % 4 == 0 || VW == 2, "16- or 8-byte loads");
  struct VRow {  // this lane's columns of a V row, as stored
    uint32_t w[VW];
  };
  __shared__ double rs[4 * 256];                  // per wavefront and row, the sum of its queries' probabilities
  __shared__ float vscale[sizeof(T) == 1 ? 256 : 1];  // fp8: the rows' powers of two
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  f32x4* ot = reinterpret_cast<f32x4*>(smem);     // [4][CT][64]: output tiles of wavefronts that share a query tile
  const int bhN = gridDim.x, bh = blockIdx.x, chunk = blockIdx.y;
  const int N = ctotal[bh];
  if (chunk * kChunk >= N) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, kq = lane >> 4;
  const int64_t slot0 = int64_t(bh) * slots + meta[bh * 4 + 0];
  const int nc = N - m, nq = m * G;
#pragma unroll
  for (int i = 0; i < 4; ++i) rs[i * 256 + tid] = 0.0;
  if constexpr (sizeof(T) == 1) vscale[tid] = pow2_f32(cVe[slot0 + min(chunk * kChunk + tid, N - 1)]);
  __syncthreads();
  const int ngroup = min(4, (N - chunk * kChunk + 63) / 64);
  const int t_lo = tile0 + blockIdx.z * tiles_per_slice, t_hi = min(tile1, t_lo + tiles_per_slice);
  const WaveWork ww = wave_work(w, t_lo, t_hi);
  const __amdgpu_buffer_rsrc_t rows = buffer_of(cV + (slot0 + chunk * kChunk) * D, uint32_t(min(kChunk, N - chunk * kChunk) * RB));
  for (int qt = ww.tile; qt < t_hi; qt += 4) {
    const int q0 = qt * kQT, query = q0 + c;
    const int seen = query < nq ? min(nc + query / G, N - 1) : -1;  // a padding query sees nothing
    const int tile_last = q0 + kQT <= nq ? min(nc + q0 / G, N - 1) : -1;
    const double M = query < nq ? norm[(int64_t(bh) * maxq + query) * 2] : 0.0;
    const double Linv = query < nq ? 1.0 / norm[(int64_t(bh) * maxq + query) * 2 + 1] : 0.0;
    const __amdgpu_buffer_rsrc_t terms = buffer_of(term + term_index(qt - tile0, gridDim.y, chunk, bhN, bh, 0), kChunk * kQT * 8);
    // the probabilities of a group's rows 16 t + 4 r + kq, value 4 t + r
    auto load_probs = [&](int g, float (&pf)[16], bool add) {
      double pr[16];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        pr[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                               terms, ((g * 64 + kq) * kQT + c) * 8 + i * (4 * kQT * 8), 0, 0));
      // (the division by the normaliser is a multiplication by its reciprocal here: the
      // probabilities are compared within the float tolerance, never bit for bit)
      const double f = exp(gmax[((int64_t(chunk) * bhN + bh) * maxq + query) * 4 + g] - M) * Linv;
#pragma unroll
      for (int i = 0; i < 16; ++i) pr[i] *= f;
      const int j0 = chunk * kChunk + g * 64 + kq;
      if (chunk * kChunk + g * 64 + 63 > tile_last) {  // (a normaliser that is not finite stays with the rows the query sees)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (j0 + 4 * i > seen) pr[i] = 0.0;
      }
      if (add) {  // Eq. 6: the rows' sums over the tile's queries, one row per lane, then over the wavefront's tiles
        const double ps = row16_sums(pr, c);
        const int own = row16_sums_owner(c);
        rs[w * 256 + g * 64 + (own >> 2) * 16 + 4 * (own & 3) + kq] += ps;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) pf[i] = float(pr[i]);
    };
    auto v_row = [&](int g, int i) {  // of probability i (zero past the last row)
      const int off = (g * 64 + kq) * RB + c * (CT * int(sizeof(T))) + i * 4 * RB;
      VRow v;
      if constexpr (VW >= 4) {
#pragma unroll
        for (int x = 0; x < VW; x += 4) {
          const u32x4 q = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, off + x * 4, 0, 0));
#pragma unroll
          for (int y = 0; y < 4; ++y) v.w[x + y] = q[y];
        }
      } else {
        const u32x2 q = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rows, off, 0, 0));
        v.w[0] = q[0];
        v.w[1] = q[1];
      }
      return v;
    };
    f32x4 O[CT];
    auto clear = [&]() {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) O[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // P V on the fp32 matrix instruction, a contraction step per probability (rows 4 i + kq), for V rows that came four at a time
    auto multiply_f32 = [&](int g, const float (&pf)[16], const VRow (&vr)[4], int i0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float pa = pf[i0 + r];
        if constexpr (sizeof(T) == 1) pa *= vscale[g * 64 + 4 * (i0 + r) + kq];
        float vb[CT];
#pragma unroll
        for (int wd = 0; wd < VW; ++wd) {
          const uint32_t raw = vr[r].w[wd];
          if constexpr (sizeof(T) == 1) {
            vb[4 * wd] = __builtin_amdgcn_cvt_f32_fp8(int(raw), 0);
            vb[4 * wd + 1] = __builtin_amdgcn_cvt_f32_fp8(int(raw), 1);
            vb[4 * wd + 2] = __builtin_amdgcn_cvt_f32_fp8(int(raw), 2);
            vb[4 * wd + 3] = __builtin_amdgcn_cvt_f32_fp8(int(raw), 3);
          } else if constexpr (sizeof(T) == 2) {
            vb[2 * wd] = __uint_as_float(raw << 16);
            vb[2 * wd + 1] = __uint_as_float(raw & 0xFFFF0000u);
          } else {
            vb[wd] = __uint_as_float(raw);
          }
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) O[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa, vb[ct], O[ct], 0, 0, 0);
      }
    };
    clear();
#pragma unroll 1
    for (int g = ww.group; g < ngroup; g += ww.share) {
      float pf[16];
      if constexpr (sizeof(T) == 4) {
        // V rows come from memory four steps at a time, requested before the arithmetic that precedes them
        // (read where they are multiplied, the compiler waited for each row in turn)
        VRow vr[2][4];
        auto load_v = [&](int t) {
#pragma unroll
          for (int r = 0; r < 4; ++r) vr[t & 1][r] = v_row(g, 4 * t + r);
        };
        load_v(0);
        load_probs(g, pf, true);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          __builtin_amdgcn_sched_barrier(0);
          if (t < 3) load_v(t + 1);
          __builtin_amdgcn_sched_barrier(0);
          multiply_f32(g, pf, vr[t & 1], 4 * t);
        }
      } else {
        VRow vr[8];
        auto load_v = [&](int h) {
#pragma unroll
          for (int j = 0; j < 8; ++j) vr[j] = v_row(g, 8 * h + j);
        };
        load_v(0);
        load_probs(g, pf, true);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (h == 1) load_v(1);
          __builtin_amdgcn_sched_barrier(0);
          // v_mfma_f32_16x16x32_bf16: lane l holds A[l % 16][8 (l / 16) ..] and B[8 (l / 16) ..][l % 16]; contraction index
          // 8 kq + j is row 4 (8 h + j) + kq.
          bf16x8 a[3];
          {
            u32x4 t1, t2, t3;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              uint32_t b1[2], b2[2], b3[2];
#pragma unroll
              for (int y = 0; y < 2; ++y) {
                const int i = 8 * h + 2 * x + y;
                float p1 = pf[i] * pow2_f32(kTermScale);
                if constexpr (sizeof(T) == 1) p1 *= vscale[g * 64 + 4 * i + kq];
                const float p2 = p1 - __uint_as_float(__float_as_uint(p1) & 0xFFFF0000u);
                const float p3 = p2 - __uint_as_float(__float_as_uint(p2) & 0xFFFF0000u);
                b1[y] = __float_as_uint(p1);
                b2[y] = __float_as_uint(p2);
                b3[y] = __float_as_uint(p3);
              }
              t1[x] = __builtin_amdgcn_perm(b1[1], b1[0], kHighHalves);
              t2[x] = __builtin_amdgcn_perm(b2[1], b2[0], kHighHalves);
              t3[x] = __builtin_amdgcn_perm(b3[1], b3[0], kHighHalves);
            }
            a[0] = __builtin_bit_cast(bf16x8, t1);
            a[1] = __builtin_bit_cast(bf16x8, t2);
            a[2] = __builtin_bit_cast(bf16x8, t3);
          }
#pragma unroll
          for (int c2 = 0; c2 < CT / 2; ++c2) {  // columns 2 c2 and 2 c2 + 1 of the lane's
            uint32_t two[8];  // of each row, as bf16
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              if constexpr (sizeof(T) == 1) {  // (a code has four significant bits)
                const int wd = int(vr[j].w[c2 / 2]);
                const auto v = c2 & 1 ? __builtin_amdgcn_cvt_pk_f32_fp8(wd, true) : __builtin_amdgcn_cvt_pk_f32_fp8(wd, false);
                two[j] = __builtin_amdgcn_perm(__float_as_uint(v[1]), __float_as_uint(v[0]), kHighHalves);
              } else {
                two[j] = vr[j].w[c2];
              }
            }
            u32x4 lo, hi;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              lo[x] = __builtin_amdgcn_perm(two[2 * x + 1], two[2 * x], kLowHalves);
              hi[x] = __builtin_amdgcn_perm(two[2 * x + 1], two[2 * x], kHighHalves);
            }
            const bf16x8 b0 = __builtin_bit_cast(bf16x8, lo), b1 = __builtin_bit_cast(bf16x8, hi);
#pragma unroll
            for (int t = 0; t < 3; ++t) {
              O[2 * c2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b0, O[2 * c2], 0, 0, 0);
              O[2 * c2 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b1, O[2 * c2 + 1], 0, 0, 0);
            }
          }
        }
      }
    }
    if constexpr (sizeof(T) <= 2) {
      bool finite = true;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          finite = finite && fabsf(O[ct][r]) < INFINITY;
          O[ct][r] *= pow2_f32(-kTermScale);
        }
      if (!__all(finite)) {  // a term 0 beside an infinite value, or a scaled sum out of range: whole probabilities
        clear();
#pragma unroll 1
        for (int g = ww.group; g < ngroup; g += ww.share) {
          float pf[16];
          load_probs(g, pf, false);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const VRow vr[4] = {v_row(g, 4 * t), v_row(g, 4 * t + 1), v_row(g, 4 * t + 2), v_row(g, 4 * t + 3)};
            multiply_f32(g, pf, vr, 4 * t);
          }
        }
      }
    }
    if (ww.share > 1) {  // the sharers' output tiles, added in group order
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) ot[(w * CT + ct) * 64 + lane] = O[ct];
      __syncthreads();
      if (ww.group == 0)
        for (int i = 1; i < ww.share; ++i)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const f32x4 o = ot[((w + i) * CT + ct) * 64 + lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) O[ct][r] += o[r];
          }
    }
    // O[ct][r]: query q0 + 4 kq + r, column CT c + ct
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int qo = q0 + 4 * kq + r;
      if (ww.group == 0 && qo < nq) {
        float* dst = pout + ((int64_t(chunk) * bhN + bh) * maxq + qo) * D + c * CT;
#pragma unroll
        for (int x = 0; x < CT; x += 4) *reinterpret_cast<f32x4*>(dst + x) = f32x4{O[x][r], O[x + 1][r], O[x + 2][r], O[x + 3][r]};
      }
    }
  }
  __syncthreads();
  const int j = chunk * kChunk + tid;
  if (j < N) spart[(int64_t(blockIdx.z) * bhN + bh) * rows_cap + j] = (rs[tid] + rs[256 + tid]) + (rs[512 + tid] + rs[768 + tid]);
}

// Eq. 6 for the block: a row's score grows by the slices' sums, added in slice order (slices hold
// ascending ranges of (token, query head)).
__global__ __launch_bounds__(256) void block_scores(const int32_t* __restrict__ ctotal, const int32_t* __restrict__ meta,
                                                    double* __restrict__ cscore, const double* __restrict__ spart,
                                                    int nslice, int64_t slots, int rows_cap) {
  const int bhN = gridDim.x, bh = blockIdx.x, j = blockIdx.y * 256 + threadIdx.x;
  if (j >= ctotal[bh]) return;
  const int64_t slot0 = int64_t(bh) * slots + meta[bh * 4 + 0];
  double sc = cscore[slot0 + j];
  for (int z = 0; z < nslice; ++z) sc += spart[(int64_t(z) * bhN + bh) * rows_cap + j];
  cscore[slot0 + j] = sc;
}

template <typename OT, int D>
__global__ __launch_bounds__(D) void block_finish(const int32_t* __restrict__ ctotal, const float* __restrict__ pout,
                                                  OT* __restrict__ out, View ov, int G, int maxq, int Hkv) {
  const int bhN = gridDim.x, bh = blockIdx.x, q = blockIdx.y, c = threadIdx.x;
  const int N = ctotal[bh], nch = (N + kChunk - 1) / kChunk;
  float t = 0.f;
#pragma unroll 8
  for (int ch = 0; ch < nch; ++ch) t += pout[((int64_t(ch) * bhN + bh) * maxq + q) * D + c];
  const int b = bh / Hkv, hk = bh % Hkv;
  out[b * ov.sb + (hk * G + q % G) * ov.sh + int64_t(q / G) * ov.sn + c] = Elem<OT>::from_f32(t);
}

// fp8 cache: the same permutation, decoding every row into the bf16 copy on the way (a code times
// a power of two has four significant bits: exact in bf16).  One wavefront per row, D = 128.
__global__ __launch_bounds__(256) void permute_decode_rows(const int32_t* __restrict__ on, const int32_t* __restrict__ meta,
                                                           const int32_t* __restrict__ rank, const uint8_t* __restrict__ cK,
                                                           const uint8_t* __restrict__ cV, const int8_t* __restrict__ cKe,
                                                           const int8_t* __restrict__ cVe, uint16_t* __restrict__ oK,
                                                           uint16_t* __restrict__ oV, int npad, int64_t slots) {
  constexpr int D = 128;
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y, lane = threadIdx.x & 63;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (j >= on[bh]) return;
  const int64_t src = bh * slots + meta[bh * 4 + 0] + j;
  const int64_t dst = (bh * npad + rank[bh * npad + j]) * D;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const uint16_t codes = reinterpret_cast<const uint16_t*>((which ? cV : cK) + src * D)[lane];
    const float sc = pow2_f32((which ? cVe : cKe)[src]);
    const float v0 = Elem<uint8_t>::to_f32(uint8_t(codes & 0xFF)) * sc, v1 = Elem<uint8_t>::to_f32(uint8_t(codes >> 8)) * sc;
    reinterpret_cast<uint32_t*>((which ? oV : oK) + dst)[lane] = (__float_as_uint(v0) >> 16) | (__float_as_uint(v1) & 0xFFFF0000u);
  }
}

// fp8 cache: the block's K and V rows encoded into the cache (one wavefront per new row).
__global__ __launch_bounds__(256) void block_rows_fp8(const int32_t* __restrict__ ccount, const int32_t* __restrict__ meta,
                                                      uint8_t* __restrict__ cK, uint8_t* __restrict__ cV,
                                                      int8_t* __restrict__ cKe, int8_t* __restrict__ cVe,
                                                      const uint16_t* __restrict__ kn, View kv,
                                                      const uint16_t* __restrict__ vn, View vv, int m, int64_t slots) {
  constexpr int D = 128;
  const int hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y, lane = threadIdx.x & 63;
  const int64_t bh = int64_t(b) * Hkv + hk;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= m) return;
  const int64_t dst = bh * slots + meta[bh * 4 + 0] + ccount[bh] + i;  // (the entry count moves later, in block_norm)
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const uint16_t* src = which ? vn + b * vv.sb + hk * vv.sh + int64_t(i) * vv.sn : kn + b * kv.sb + hk * kv.sh + int64_t(i) * kv.sn;
    const uint32_t two = reinterpret_cast<const uint32_t*>(src)[lane];
    const double x0 = double(__uint_as_float(two << 16)), x1 = double(__uint_as_float(two & 0xFFFF0000u));
    const int e = fp8_row_exponent(wave_max(fmax(fabs(x0), fabs(x1))));
    reinterpret_cast<uint16_t*>((which ? cV : cK) + dst * D)[lane] =
        uint16_t(fp8_encode(ldexp(x0, -e))) | uint16_t(uint16_t(fp8_encode(ldexp(x1, -e))) << 8);
    if (lane == 0) (which ? cVe : cKe)[dst] = int8_t(e);
  }
}

template <typename T, int D>
hipError_t run_block_attend(d2o_ctx* c, int layer, View q, View k, View v, View out, int m, int first_pos, hipStream_t s) {
  typedef typename std::conditional<sizeof(T) == 1, uint16_t, T>::type IT;  // the tensors' type (an fp8 cache takes bf16 tensors)
  const d2o_config& cf = c->cfg;
  const int G = cf.n_q_heads / cf.n_kv_heads, bh = cf.batch * cf.n_kv_heads, maxq = c->ap_maxq;
  const size_t lo = size_t(layer) * bh;
  int32_t* ccount = c->ccount + lo;
  int32_t* ctotal = c->ctotal + lo;
  const int32_t* meta = c->meta + lo * 4;
  int max_rows = 0;
  for (const auto& mt : c->layers[layer].meta) max_rows = std::max(max_rows, mt.budget + m);
  const int nch = (max_rows + kChunk - 1) / kChunk;
  if (nch > c->ap_nch || m * G > maxq) return hipErrorInvalidValue;
  block_begin<T, IT, D><<<dim3(cf.n_kv_heads, cf.batch, 32), 256, 0, s>>>(ccount, ctotal, meta, (T*)c->cacheK, (T*)c->cacheV, c->cscore,
                                                                         c->cpos, (const IT*)q.ptr, q, (const IT*)k.ptr, k,
                                                                         (const IT*)v.ptr, v, c->ap_q, m, G, maxq, first_pos,
                                                                         cf.slots_per_seq);
  if constexpr (sizeof(T) == 1)
    block_rows_fp8<<<dim3((m + 3) / 4, cf.n_kv_heads, cf.batch), 256, 0, s>>>(ccount, meta, (uint8_t*)c->cacheK, (uint8_t*)c->cacheV,
                                                                               c->cKe, c->cVe, (const uint16_t*)k.ptr, k,
                                                                               (const uint16_t*)v.ptr, v, m, cf.slots_per_seq);
  typedef BlockRows<T, D> BR;
  constexpr int kStatsLds = BR::kRowsBytes + BR::kScaleBytes;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(block_stats<T, D>), hipFuncAttributeMaxDynamicSharedMemorySize, kStatsLds);
  if (e != hipSuccess) return e;
  const int rows_cap = c->ap_nch * kChunk;
  // few heads and chunks give few workgroups: the query tiles of a head are cut into slices that
  // run as workgroups of their own (whole rounds of the four wavefronts), enough of them to fill
  // the chip a few times over
  const int want = std::max(1, std::min(kMaxQuerySlices, 2048 / std::max(1, bh * nch)));
  const int ntile = (m * G + kQT - 1) / kQT;
  const int per_pass = int(std::min<int64_t>(ntile, int64_t(c->ap_tiles) * c->ap_nch / nch));  // query tiles whose exponentials fit
  for (int t0 = 0; t0 < ntile; t0 += per_pass) {
    const int t1 = std::min(ntile, t0 + per_pass);
    const int tiles_per_slice = 4 * ((t1 - t0 + 4 * want - 1) / (4 * want));
    const int nslice = (t1 - t0 + tiles_per_slice - 1) / tiles_per_slice;
    const dim3 grid(bh, nch, nslice);
    block_stats<T, D><<<grid, 256, kStatsLds, s>>>(ctotal, meta, (const T*)c->cacheK, c->cKe, c->ap_q, c->ap_stat, c->ap_gmax,
                                                   c->ap_term, m, G, maxq, cf.slots_per_seq, t0, t1, tiles_per_slice);
    block_norm<<<dim3(bh), 256, 0, s>>>(ctotal, ccount, c->ap_stat, c->ap_norm, t0 * kQT, std::min(m * G, t1 * kQT), maxq);
    // (the place for shared tiles only where a slice has one or two: it would cost the others a workgroup per CU)
    const int rest = (t1 - t0) % tiles_per_slice;
    const int shared_tiles = rest == 1 || rest == 2 ? 4 * (D / 16) * 64 * int(sizeof(f32x4)) : 0;
    block_apply<T, D><<<grid, 256, shared_tiles, s>>>(ctotal, meta, (const T*)c->cacheV, c->cVe, c->ap_spart, c->ap_norm, c->ap_gmax,
                                           c->ap_term, c->ap_out, m, G, maxq, cf.slots_per_seq, rows_cap, t0, t1, tiles_per_slice);
    block_scores<<<dim3(bh, nch), 256, 0, s>>>(ctotal, meta, c->cscore, c->ap_spart, nslice, cf.slots_per_seq, rows_cap);
  }
  if (cf.out_f32)
    block_finish<float, D><<<dim3(bh, m * G), D, 0, s>>>(ctotal, c->ap_out, (float*)out.ptr, out, G, maxq, cf.n_kv_heads);
  else
    block_finish<IT, D><<<dim3(bh, m * G), D, 0, s>>>(ctotal, c->ap_out, (IT*)out.ptr, out, G, maxq, cf.n_kv_heads);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_cache_sort(d2o_ctx* c, int layer, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const int32_t* meta = c->meta + size_t(layer) * cf.batch * cf.n_kv_heads * 4;
  const int32_t* ccount = c->ccount + size_t(layer) * cf.batch * cf.n_kv_heads;
  int max_rows = 0;
  for (const auto& mt : c->layers[layer].meta) max_rows = std::max(max_rows, mt.budget + c->grow);
  // Every position is below the next one, unless an import brought larger ones.  (A block of 4 tokens on 20000 entries of
  // one head: positions in the set 0.12 ms, beyond the largest set, by rank_by_position, 0.47; with positions that the
  // set, sized by the next position alone, did not hold, compared by its one workgroup, 16.8.)
  const LayerState& st = c->layers[layer];
  const int64_t words = (std::max<int64_t>(st.next_pos, st.pos_end) + 32 * 1024 - 1) / (32 * 1024) * 1024;
  if (words <= kBitWords) {
    const int lds = int(words + 1024) * int(sizeof(uint32_t));
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(rank_by_bits), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (kBitWords + 1024) * int(sizeof(uint32_t)));
    if (e != hipSuccess) return e;
    rank_by_bits<<<dim3(cf.n_kv_heads, cf.batch), 1024, lds, s>>>(ccount, meta, c->cscore, c->cpos, c->app_rank, c->app_pos,
                                                                  c->app_score, c->app_n, c->npad, cf.slots_per_seq, int(words));
  } else if (max_rows <= 8192)
    rank_by_position<1><<<dim3(cf.n_kv_heads, cf.batch, (max_rows + 255) / 256), 256, 0, s>>>(
        ccount, meta, c->cscore, c->cpos, c->app_rank, c->app_pos, c->app_score, c->app_n, c->npad, cf.slots_per_seq);
  else
    rank_by_position<4><<<dim3(cf.n_kv_heads, cf.batch, (max_rows + 1023) / 1024), 256, 0, s>>>(
        ccount, meta, c->cscore, c->cpos, c->app_rank, c->app_pos, c->app_score, c->app_n, c->npad, cf.slots_per_seq);
  if (cf.cache_fp8) {
    permute_decode_rows<<<dim3((max_rows + 3) / 4, cf.n_kv_heads, cf.batch), 256, 0, s>>>(
        c->app_n, meta, c->app_rank, (const uint8_t*)c->cacheK, (const uint8_t*)c->cacheV, c->cKe, c->cVe,
        (uint16_t*)c->app_K, (uint16_t*)c->app_V, c->npad, cf.slots_per_seq);
  } else if (cf.dtype == D2O_BF16) {
    const int rows = 256 / (cf.head_dim / 8);
    permute_rows<uint16_t><<<dim3((max_rows + rows - 1) / rows, cf.n_kv_heads, cf.batch), 256, 0, s>>>(
        c->app_n, meta, c->app_rank, (const uint16_t*)c->cacheK, (const uint16_t*)c->cacheV, (uint16_t*)c->app_K,
        (uint16_t*)c->app_V, c->npad, cf.head_dim, cf.slots_per_seq);
  } else {
    const int rows = 256 / (cf.head_dim / 4);
    permute_rows<float><<<dim3((max_rows + rows - 1) / rows, cf.n_kv_heads, cf.batch), 256, 0, s>>>(
        c->app_n, meta, c->app_rank, (const float*)c->cacheK, (const float*)c->cacheV, (float*)c->app_K,
        (float*)c->app_V, c->npad, cf.head_dim, cf.slots_per_seq);
  }
  return hipGetLastError();
}

hipError_t launch_block_attend(d2o_ctx* c, int layer, View q, View k, View v, View out, int m, int first_pos,
                               hipStream_t s) {
  const d2o_config& cf = c->cfg;
  if (cf.cache_fp8) return run_block_attend<uint8_t, 128>(c, layer, q, k, v, out, m, first_pos, s);
  if (cf.dtype == D2O_BF16) return run_block_attend<uint16_t, 128>(c, layer, q, k, v, out, m, first_pos, s);
  if (cf.head_dim == 64) return run_block_attend<float, 64>(c, layer, q, k, v, out, m, first_pos, s);
  return run_block_attend<float, 128>(c, layer, q, k, v, out, m, first_pos, s);
}

}  // namespace d2o
