// Prompt-phase attention for fp32 tensors (the small configuration) and the density
// reduction shared by both dtypes.  fp32 inputs are never down-converted: both products run on
// v_mfma_f32_16x16x4_f32, whose products and sums are fp32 FMAs (twice the rate of the unpacked
// vector ALU).  The bf16 path is in prefill_bf16.hip.
//
// Pass 1 (Sec. 4.1 Eq. 4, Sec. 3 Eq. 3): O = softmax(Q K^T / sqrt(d)) V, causal, and the row
//   log-sum-exp.  Pass 2 (column sums of the attention matrix, Sec. 4.1; Eq. 6 prompt case):
//   score[j] = sum_g sum_{i >= j} exp(s_ij - lse_i), plus per-query-head partial sums of the
//   column sums and their squares for the variance of Eq. 4.
//
// Operand layout of the instruction (lane l, m = l % 16, q = l / 16): A[m][q], B[q][m],
// D[4q + r][m] for r = 0..3.  Both passes form S^T = K Q^T: a lane holds one query's logits
// against keys 4q .. 4q+3.  The contraction runs over d in an order of its own (part q of a row
// is its q-th quarter, taken element by element), so that every lane reads contiguous memory,
// and operands come straight from memory: the matrices of these sizes live in L2.
#include <algorithm>

#include "d2o_internal.h"
#include "device_utils.h"

namespace d2o {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

constexpr int kWaves = 8;      // pass 1: wavefronts that share a row block's keys
constexpr int kColWaves = 16;  // pass 2: kF32BN / 16 key blocks x query shares
constexpr int kColShares = kColWaves / (kF32BN / 16);

// A quarter of a row (the one of this lane), as the operand elements of D / 4 steps.
template <int D>
__device__ __forceinline__ void load_quarter(const float* row, int q, f32x4 (&v)[D / 16]) {
#pragma unroll
  for (int c = 0; c < D / 16; ++c) v[c] = *reinterpret_cast<const f32x4*>(row + q * (D / 4) + 4 * c);
}
template <int D>
__device__ __forceinline__ f32x4 logits_t(const f32x4 (&k)[D / 16], const f32x4 (&qy)[D / 16]) {
  // four chains, added pairwise: shorter sums round less (and wait less for each other)
  f32x4 s[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < D / 16; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[c][e], qy[c][e], s[e], 0, 0, 0);
  return (s[0] + s[1]) + (s[2] + s[3]);
}

// 16 query rows per workgroup; its wavefronts take 32 keys at a time in turn, with an online softmax
// state of their own, and are combined through LDS.  Bound by latency at the sizes it is for: a
// row block of 512 tokens is two rounds of 32 keys per wavefront, and four heads of them are
// 128 workgroups, so splitting the keys (not the rows) over wavefronts is what fills the chip.
// The probabilities of register r, which belong to keys 4q + r, are the B operand of a step of
// V^T P^T over those four keys as they are.  512 tokens, 4 heads, d = 64: 74 us (one wavefront
// per row on the vector ALU) -> 12 us.
template <int D>
__global__ __launch_bounds__(64 * kWaves) void attn_rows_f32(const float* __restrict__ Q, View qv, const float* __restrict__ K,
                                                     View kv, const float* __restrict__ V, View vv, float* __restrict__ O,
                                                     View ov, float* __restrict__ lse2, int n, int npad, int G) {
  constexpr int DT = D / 16;  // output columns per lane and register
  __shared__ float po[kWaves][16][D + 4];
  __shared__ float pm[kWaves][16], pl[kWaves][16];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  const int row0 = (gridDim.x - 1 - blockIdx.x) * 16;  // the longest row blocks start first
  const int hq = blockIdx.y, b = blockIdx.z, hk = hq / G;
  const float scale2 = kLog2e / sqrtf(float(D));
  const float* kb = K + b * kv.sb + hk * kv.sh;
  const float* vb = V + b * vv.sb + hk * vv.sh;
  const int row = row0 + m;
  f32x4 qy[D / 16];
  load_quarter<D>(Q + b * qv.sb + hq * qv.sh + int64_t(min(row, n - 1)) * qv.sn, q, qy);
  f32x4 acc[DT];  // acc[c][r]: column (4q + r) * DT + c of the row
#pragma unroll
  for (int c = 0; c < DT; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mx = -INFINITY, l = 0.f, p[2][4];
  bool special = false;  // the last tile holds infinite or NaN values
  const int nkt = min(row0 + 15, n - 1) / 32 + 1;  // 32-key tiles that any row of the block sees
  f32x4 k0[D / 16], k1[D / 16];
  auto load_keys = [&](int t) {
    load_quarter<D>(kb + int64_t(min(t * 32 + m, n - 1)) * kv.sn, q, k0);
    load_quarter<D>(kb + int64_t(min(t * 32 + 16 + m, n - 1)) * kv.sn, q, k1);
  };
  if (w < nkt) load_keys(w);
  for (int t = w; t < nkt; t += kWaves) {
    f32x4 s[2] = {logits_t<D>(k0, qy), logits_t<D>(k1, qy)};
    // V rows of keys 4q + r, columns m * DT .. + DT - 1
    f32x4 v[2][4][DT / 4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < DT / 4; ++c)
          v[u][r][c] = *reinterpret_cast<const f32x4*>(vb + int64_t(min(t * 32 + u * 16 + 4 * q + r, n - 1)) * vv.sn +
                                                       m * DT + 4 * c);
    if (t + kWaves < nkt) load_keys(t + kWaves);
    float tm = -INFINITY;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = t * 32 + u * 16 + 4 * q + r;
        s[u][r] = key <= row ? s[u][r] : -INFINITY;
        tm = fmaxf(tm, s[u][r]);
      }
    tm = fmaxf(tm, __shfl_xor(tm, 16, 64));
    tm = fmaxf(tm, __shfl_xor(tm, 32, 64));  // a row of the block that sees no key of the tile: -inf
    const float mn = fmaxf(mx, tm * scale2), ref = mn == -INFINITY ? 0.f : mn;
    const float a = exp2f(mx - ref);
    float ps = 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[u][r] = exp2f(fmaf(s[u][r], scale2, -ref));
        ps += p[u][r];
      }
    l = l * a + ps;
    mx = mn;
    // Keys that a row does not see enter the products with probability 0, and 0 times an infinite or NaN value is
    // NaN.  All of them are in the row block's last tile (the rows behind the end too): there such values are set
    // to 0 in the operands and added afterwards, one by one, to the rows that see them.
    if (t == nkt - 1) {
      uint32_t top = 0;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < DT; ++c) top = max(top, __float_as_uint(v[u][r][c / 4][c % 4]) << 1);
      special = __any(top >= 0xFF000000u);
      if (special) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < DT; ++c)
              if (!isfinite(v[u][r][c / 4][c % 4])) v[u][r][c / 4][c % 4] = 0.f;
      }
    }
#pragma unroll
    for (int c = 0; c < DT; ++c) {
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[c][r] *= a;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[u][r][c / 4][c % 4], p[u][r], acc[c], 0, 0, 0);
    }
  }
  if (special) {
    const int t = nkt - 1;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll 1
        for (int kq = 0; kq < 4; ++kq) {
          const int key = t * 32 + u * 16 + 4 * kq + r;
          const float pk = __shfl(p[u][r], 16 * kq + m, 64);
          if (key >= n) continue;  // (the same for all lanes)
          const float* x = vb + int64_t(key) * vv.sn + 4 * q * DT;
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int c = 0; c < DT; ++c)
              if (key <= row && !isfinite(x[e * DT + c])) acc[c][e] = fmaf(pk, x[e * DT + c], acc[c][e]);
        }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (q == 0) {
    pm[w][m] = mx;
    pl[w][m] = l;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < DT; ++c) po[w][m][(4 * q + r) * DT + c] = acc[c][r];
  __syncthreads();
  for (int i = threadIdx.x; i < 16 * D; i += 64 * kWaves) {
    const int r = i / D, c = i % D, gr = row0 + r;
    float M = pm[0][r];
#pragma unroll
    for (int u = 1; u < kWaves; ++u) M = fmaxf(M, pm[u][r]);  // finite: every row sees key 0
    float lt = 0.f, o = 0.f;
#pragma unroll
    for (int u = 0; u < kWaves; ++u) {
      const float f = exp2f(pm[u][r] - M);
      lt += pl[u][r] * f;
      o += po[u][r][c] * f;
    }
    if (gr < n) {
      if (O) O[b * ov.sb + hq * ov.sh + int64_t(gr) * ov.sn + c] = o / lt;
      if (c == 0) lse2[(int64_t(b) * gridDim.y + hq) * npad + gr] = M + log2f(lt);
    }
  }
}

// kF32BN keys of a KV head per workgroup, the stationary operand (16 per wavefront); the wavefronts
// of the same keys share the query tiles i >= j, 16 at a time in turn.  Adds the G query heads of
// the group in ascending order.  512 tokens, 4 heads, d = 64: 422 us (one wavefront per key, one
// after the other, on the vector ALU) -> 12 us.
template <int D>
__global__ __launch_bounds__(64 * kColWaves) void colsum_f32(const float* __restrict__ Q, View qv, const float* __restrict__ K,
                                                  View kv, const float* __restrict__ lse2, float* __restrict__ score,
                                                  double* __restrict__ varpart, int n, int npad, int G, int Hq) {
  __shared__ float cs[kColShares][kF32BN];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, m = lane & 15, q = lane >> 4;
  const int tile = blockIdx.x, hk = blockIdx.y, b = blockIdx.z, Hkv = gridDim.y;
  const int kblk = w % (kF32BN / 16), share = w / (kF32BN / 16);
  const int key0 = tile * kF32BN + kblk * 16;
  const float scale2 = kLog2e / sqrtf(float(D));
  f32x4 k[D / 16];
  load_quarter<D>(K + b * kv.sb + hk * kv.sh + int64_t(min(key0 + m, n - 1)) * kv.sn, q, k);
  float total = 0.f;  // thread t < kF32BN owns key tile * kF32BN + t
  for (int g = 0; g < G; ++g) {
    const int hq = hk * G + g;
    const float* qb = Q + b * qv.sb + hq * qv.sh;
    const float* lrow = lse2 + (int64_t(b) * Hq + hq) * npad;
    float sum[4] = {0.f, 0.f, 0.f, 0.f};  // keys key0 + 4q + r
    const int nqt = (n + 15) / 16;
    f32x4 qy[D / 16];
    float ls = 0.f;
    auto load_queries = [&](int t) {
      const int i = min(t * 16 + m, n - 1);
      load_quarter<D>(qb + int64_t(i) * qv.sn, q, qy);
      ls = lrow[i];
    };
    int t = key0 / 16 + share;
    if (t < nqt) load_queries(t);
    for (; t < nqt; t += kColShares) {
      const f32x4 s = logits_t<D>(k, qy);
      const float lq = ls;
      const int query = t * 16 + m;
      if (t + kColShares < nqt) load_queries(t + kColShares);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float p = exp2f(fmaf(s[r], scale2, -lq));
        sum[r] += query >= key0 + 4 * q + r && query < n ? p : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) sum[r] += __shfl_xor(sum[r], o, 64);
    }
    __syncthreads();  // the previous head's sums have been read
    if (m == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) cs[share][kblk * 16 + 4 * q + r] = sum[r];
    }
    __syncthreads();
    if (w == 0) {  // kF32BN <= 64: one wavefront
      double s1 = 0.0, s2 = 0.0;
      if (lane < kF32BN && tile * kF32BN + lane < n) {
        float c = cs[0][lane];
#pragma unroll
        for (int u = 1; u < kColShares; ++u) c += cs[u][lane];
        total += c;
        s1 = double(c);
        s2 = double(c) * double(c);
      }
      s1 = wave_sum(s1);
      s2 = wave_sum(s2);
      if (lane == 0) {
        double* vp = varpart + ((int64_t(b) * Hq + hq) * (npad / kF32BN) + tile) * 2;
        vp[0] = s1;
        vp[1] = s2;
      }
    }
  }
  if (threadIdx.x < kF32BN && tile * kF32BN + int(threadIdx.x) < n)
    score[(int64_t(b) * Hkv + hk) * npad + tile * kF32BN + threadIdx.x] = total;
}

// Per sequence: variance of every query head's column sums (population, Eq. 4) from the
// partial sums of its blocks of bn keys, and their mean over heads.  One wavefront per head, the
// blocks over its lanes: as one thread per head adding them up one by one this took 5 to 130 us
// (4096 to 131072 tokens) of nothing but memory latency.
// The workgroups behind the first one of a sequence (y > 0; bf16 with G > 1 query heads per KV head) add the query
// heads' column sums up to the KV heads' scores, in ascending head order.
__global__ __launch_bounds__(1024) void density_kernel(const double* __restrict__ varpart, double* __restrict__ head_var,
                               double* __restrict__ layer_F, const float* __restrict__ colpart, float* __restrict__ score,
                               int n, int npad, int Hq, int G, int bn) {
  __shared__ double hv[256];
  const int b = blockIdx.x, lane = threadIdx.x & 63;
  if (blockIdx.y > 0) {
    const int Hkv = Hq / G;
    const int64_t nv = int64_t(Hkv) * (npad / 4), step = int64_t(gridDim.y - 1) * 1024;  // npad is a multiple of 128
    for (int64_t x = int64_t(blockIdx.y - 1) * 1024 + threadIdx.x; x < nv; x += step) {
      const int hk = int(x / (npad / 4)), k = int(x % (npad / 4)) * 4;
      if (k >= n) continue;
      const float* cp = colpart + (int64_t(b) * Hq + hk * G) * npad + k;
      f32x4 t = {0.f, 0.f, 0.f, 0.f};
      for (int g = 0; g < G; ++g) t += *reinterpret_cast<const f32x4*>(cp + int64_t(g) * npad);
      float* out = score + (int64_t(b) * Hkv + hk) * npad + k;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (k + i < n) out[i] = t[i];
    }
    return;
  }
  const int nblk = (n + bn - 1) / bn;
  for (int hq = threadIdx.x >> 6; hq < Hq; hq += 16) {
    const double* vp = varpart + (int64_t(b) * Hq + hq) * (npad / bn) * 2;
    double s1 = 0.0, s2 = 0.0;
    for (int t = lane; t < nblk; t += 64) {
      s1 += vp[2 * t];
      s2 += vp[2 * t + 1];
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    const double mu = s1 / double(n);
    const double var = s2 / double(n) - mu * mu;
    if (lane == 0) {
      head_var[int64_t(b) * Hq + hq] = var;
      hv[hq] = var;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int hq = 0; hq < Hq; ++hq) t += hv[hq];
    layer_F[b] = t / double(Hq);
  }
}

}  // namespace

hipError_t launch_prefill_f32(d2o_ctx* c, int layer, View Q, View K, View V, View O, int n, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const int G = cf.n_q_heads / cf.n_kv_heads;
  float* score = c->score_pre + size_t(layer) * cf.batch * cf.n_kv_heads * c->npad;
  dim3 g1((n + 15) / 16, cf.n_q_heads, cf.batch), g2((n + kF32BN - 1) / kF32BN, cf.n_kv_heads, cf.batch);
  if (cf.head_dim == 64) {
    { KernelTimer kt(c, D2O_K_ATTN_FWD, s);
    attn_rows_f32<64><<<g1, 64 * kWaves, 0, s>>>((const float*)Q.ptr, Q, (const float*)K.ptr, K, (const float*)V.ptr, V,
                                         (float*)O.ptr, O, c->lse, n, c->npad, G); }
    KernelTimer kt(c, D2O_K_COLSUM, s);
    colsum_f32<64><<<g2, 64 * kColWaves, 0, s>>>((const float*)Q.ptr, Q, (const float*)K.ptr, K, c->lse, score, c->varpart, n,
                                      c->npad, G, cf.n_q_heads);
  } else {
    { KernelTimer kt(c, D2O_K_ATTN_FWD, s);
    attn_rows_f32<128><<<g1, 64 * kWaves, 0, s>>>((const float*)Q.ptr, Q, (const float*)K.ptr, K, (const float*)V.ptr, V,
                                          (float*)O.ptr, O, c->lse, n, c->npad, G); }
    KernelTimer kt(c, D2O_K_COLSUM, s);
    colsum_f32<128><<<g2, 64 * kColWaves, 0, s>>>((const float*)Q.ptr, Q, (const float*)K.ptr, K, c->lse, score, c->varpart, n,
                                       c->npad, G, cf.n_q_heads);
  }
  return hipGetLastError();
}

hipError_t launch_density(d2o_ctx* c, int layer, int n, hipStream_t s) {
  const d2o_config& cf = c->cfg;
  const int G = cf.n_q_heads / cf.n_kv_heads;
  const bool add = cf.dtype == D2O_BF16 && G > 1;
  const int adders = add ? int(std::min<int64_t>(64, (int64_t(cf.n_kv_heads) * (c->npad / 4) + 1023) / 1024)) : 0;
  density_kernel<<<dim3(cf.batch, 1 + adders), 1024, 0, s>>>(
      c->varpart, c->head_var + size_t(layer) * cf.batch * cf.n_q_heads, c->layer_F + size_t(layer) * cf.batch, c->colpart,
      c->score_pre + size_t(layer) * cf.batch * cf.n_kv_heads * c->npad, n, c->npad, cf.n_q_heads, G,
      cf.dtype == D2O_F32 ? kF32BN : 128);
  return hipGetLastError();
}

}  // namespace d2o
