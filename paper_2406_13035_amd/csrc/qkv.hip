// Upstream step of the hot path (Sec. 3 Eq. 1): Q = X W_Q, K = X W_K, V = X W_V for one layer as
// ONE matrix product on the CDNA4 matrix cores, with the rotary position embedding of queries
// and keys applied to the fp32 accumulators before they are stored, and the three results
// written directly in the [sequence][head][token][d] layout that the prompt attention reads.
//
// bf16 operands, fp32 accumulation, head_dim 128.  X [B * n][hidden] and the stacked weights
// W [(Hq + 2 Hkv) * 128][hidden] are both contiguous along `hidden`, which is the layout both
// operands of v_mfma_f32_32x32x16_bf16 want (lane l: row l % 32, eight consecutive k from
// 8 * (l / 32)).
//
// A workgroup (4 wavefronts) computes 256 tokens x 256 features = two heads; a wavefront owns 128
// tokens x one head's 128 features (4 x 4 accumulator blocks: eight LDS operand reads feed sixteen
// matrix instructions).  The feature pair (c, c + 64) that the rotary embedding mixes lives in the
// same lane and register of accumulator blocks j and j + 2, so the rotation needs no exchange.  The
// rotated tile goes through LDS once so that every lane stores 16 contiguous bytes of a token's
// head vector.
#include <algorithm>
#include <type_traits>

#include "d2o_internal.h"
#include "device_utils.h"
#include "qkv_tile.h"

namespace d2o {
namespace {

using namespace qkv;

constexpr int kTokenStages = 3, kWeightStages = 2;  // k-tiles of the two operands in LDS
constexpr int kStageElems = kBM * kLd;       // (kBM = kHeadsPerWg * kBN)
constexpr int kSmemBytes = (kTokenStages + kWeightStages) * kStageElems * 2;  // all 160 KB of a CU
constexpr int kCus = 256;                    // workgroups that run at a time, one per CU

enum Loads { kNothing, kTokens, kWeights };
template <Loads W>
using LoadsOf = std::integral_constant<Loads, W>;

struct QkvArgs {
  const uint16_t* X;
  const uint16_t* W;
  View q, k, v;        // [b][head][token][d]
  int M, n, hidden, Hq, Hkv, pos0;
  double log2_base;
};

// What bounds it: the matrix core, which on operands that toggle like these runs at the clock the
// power limit leaves (a bare loop of these instructions on random data reaches 1.7 PFLOP/s).  One
// wavefront per SIMD with 256 accumulator registers reads 8 KB of operands per 16 instructions
// (half of what LDS delivers in their time); with two wavefronts of 64 x 128 it was 12 KB per 16.
// k-tiles go from memory to LDS without passing through registers (the swizzle applied to the
// addresses the lanes read from) and hold whole 128-byte lines of a row: with k-tiles of 32
// every line was fetched twice.  The operand reads of the next quarter tile and the loads are placed between the
// matrix instructions of the current one, so the matrix core only waits at the barrier, once
// per tile.  The workgroups are persistent (one per CU): the first k-tiles of the next output
// tile arrive during the epilogue, and the workgroups of an XCD stay close enough to each other
// that a line one of them fetched is still in the XCD's L2 when the others ask for it.
// 32768 tokens x 4096 -> 96 heads: 2.49-2.67 ms = 1.24-1.32 PFLOP/s (8 wavefronts, k-tiles of 32
// through registers, one output tile per workgroup: 3.3-3.4 ms).  A k-tile takes 2250 cycles of
// which 2048 are matrix instructions; an output tile's epilogue (6 us of a 100 us tile) is not
// overlapped.
// Wide: rows of more than kMaxBufferHidden columns, whose offsets inside a tile pass 31 bits; loaded by 64-bit
// address with the rows clamped (more address arithmetic per load, so not for the others).
template <bool Wide>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void qkv_rope_bf16(QkvArgs a, int nft, int ntiles, int nwg) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, m = lane & 31, h = lane >> 5;
  const int nheads = a.Hq + 2 * a.Hkv;
  const int wm = w & 1, wn = w >> 1;      // the wavefront's 128 tokens, and which head of the pair
  const uint32_t row_bytes = uint32_t(a.hidden) * 2;
  const bool half = a.hidden % kBK != 0;  // the last k-tile has 32 columns
  const int nfull = a.hidden / kBK, nkt = nfull + (half ? 1 : 0);
  // Workgroups go to the eight XCDs round-robin in launch order.  Each XCD takes one eighth of
  // the heads (its slice of W stays close to it) and walks the token tiles with its heads as
  // the fast index, so the workgroups that run together share a few token tiles and that slice.
  auto tile_of = [&](int lin, int& ftile, int& rt) {  // ftile: a pair of heads out of [Q heads | K heads | V heads]
    if (nft % 8 == 0) {
      const int xcd = lin & 7, s_ = lin >> 3, fpx = nft / 8;
      ftile = xcd * fpx + s_ % fpx;
      rt = s_ / fpx;
    } else {
      ftile = lin % nft;
      rt = lin / nft;
    }
  };
  // ---- loads.  One instruction fills 8 rows of a k-tile (64 lanes x 16 bytes, consecutive in LDS); a
  // wavefront issues eight for the tokens and eight for the weights.  The buffers end with the
  // output tile's last row: what lies behind it (rows of a last tile, and columns of the last k-tile
  // in the last row) is not read, arrives as zero and is never used.  k-tiles form one sequence over all output
  // tiles of the workgroup; `next` is the place two of them ahead of the one being multiplied.
  // The tokens of a k-tile are requested seven quarters of a tile before they are needed, its
  // weights four (LDS holds five half k-tiles): two and two left the matrix core waiting for a
  // fifth of the time.
  struct Cursor {
    __amdgpu_buffer_rsrc_t x, w;
    const uint16_t *xp, *wp;  // Wide: instead of the buffers
    int xrows, wrows;
    int lin, kt;
  } next;
  auto open = [&](int lin) {
    int ftile, rt;
    tile_of(min(lin, ntiles - 1), ftile, rt);
    next.xp = a.X + int64_t(rt) * kBM * a.hidden;
    next.wp = a.W + int64_t(ftile) * kHeadsPerWg * kBN * a.hidden;
    next.xrows = min(kBM, a.M - rt * kBM);
    next.wrows = min(kHeadsPerWg, nheads - ftile * kHeadsPerWg) * kBN;
    if constexpr (!Wide) {  // past the last output tile: empty buffers
      next.x = buffer_of(next.xp, lin < ntiles ? buffer_bytes(next.xrows, row_bytes) : 0u);
      next.w = buffer_of(next.wp, lin < ntiles ? buffer_bytes(next.wrows, row_bytes) : 0u);
    }
    next.lin = lin;
    next.kt = 0;
  };
  auto advance = [&]() {
    if (++next.kt == nkt) open(next.lin + nwg);
  };
  const uint32_t off_even = lane_offset(w, lane, false, row_bytes), off_odd = lane_offset(w, lane, true, row_bytes);
  auto tokens = [&](int sa) { return smem + sa * kStageElems; };
  auto weights = [&](int sb) { return smem + (kTokenStages + sb) * kStageElems; };
  auto load = [&](int i, bool tok, uint16_t* stage) {  // load i (0..7) of the k-tile `next`
    uint16_t* dst = stage + lds_start(w, i);
    if constexpr (Wide)
      load_lds16((tok ? next.xp : next.wp) + wide_offset(w, lane, i, next.kt, tok ? next.xrows : next.wrows, int64_t(a.hidden) * 2) / 2, dst);
    else
      load_lds16(tok ? next.x : next.w, ((i & 1) ? off_odd : off_even) + load_step(i, next.kt, row_bytes), dst);
  };
  // operand i (0..3: token blocks, 4..7: feature blocks) of quarter ks of the k-tile in these stages
  const int swz = (m >> 1) & 7;
  auto operand = [&](int i, int ks, int sa, int sb) -> bf16x8 {
    const uint16_t* row = i < 4 ? tokens(sa) + (wm * 128 + i * 32 + m) * kLd : weights(sb) + (wn * kBN + (i - 4) * 32 + m) * kLd;
    return *reinterpret_cast<const bf16x8*>(row + (((ks * 2 + h) ^ swz) << 3));
  };
  f32x16 acc[4][4];
  bf16x8 S0[8], S1[8];
  auto mma2 = [&](const bf16x8 (&S)[8], int q) {  // two of the sixteen matrix instructions of a quarter tile
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 2 * q; u < 2 * q + 2; ++u)
      acc[u >> 2][u & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(S[u >> 2], S[4 + (u & 3)], acc[u >> 2][u & 3], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // the operands in the order in which the matrix instructions need them
  constexpr int kOrder[8] = {0, 4, 5, 6, 7, 1, 2, 3};
  // One quarter: multiplies Sa while the operands of quarter ks of stages (sa, sb) arrive in Sb, spread
  // out so that the four wavefronts do not queue at the LDS; the loads of the tokens or weights of `next` into `dst`
  // go out in between.
  auto quarter = [&](const bf16x8 (&Sa)[8], bf16x8 (&Sb)[8], int ks, int sa, int sb, auto what, uint16_t* dst) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      mma2(Sa, q);
      if (ks != 3) {
        Sb[kOrder[q]] = operand(kOrder[q], ks, sa, sb);
      } else if (q < 4) {  // the barrier that follows waits for them
        Sb[kOrder[2 * q]] = operand(kOrder[2 * q], ks, sa, sb);
        Sb[kOrder[2 * q + 1]] = operand(kOrder[2 * q + 1], ks, sa, sb);
      }
      if constexpr (decltype(what)::value != kNothing) load(q, decltype(what)::value == kTokens, dst);
    }
  };
  // Behind this barrier every wavefront has its last operands of the current k-tile in registers
  // and its loads of the following one in LDS (the tokens of the one after that may be on their
  // way): the current stages are free and the following k-tile complete.
  auto turn = [&]() {
    wait_lgkm0();
    wait_vm<8>();
    __builtin_amdgcn_s_barrier();
  };
  open(blockIdx.x);
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
    for (int i = 0; i < 8; ++i) load(i, true, tokens(kt));
#pragma unroll
    for (int i = 0; i < 8; ++i) load(i, false, weights(kt));
    advance();
  }
  wait_vm<16>();
  __builtin_amdgcn_s_barrier();
  int sa = 0, sb = 0;  // stages of the current k-tile
#pragma unroll 1
  for (int lin = blockIdx.x; lin < ntiles; lin += nwg) {
    int ftile, rt;
    tile_of(lin, ftile, rt);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) S0[i] = operand(i, 0, sa, sb);
#pragma unroll 1
    for (int t = 0; t < nfull; ++t) {
      const int sa1 = sa == 2 ? 0 : sa + 1, sa2 = sa == 0 ? 2 : sa - 1;
      quarter(S0, S1, 1, sa, sb, LoadsOf<kTokens>{}, tokens(sa2));
      quarter(S1, S0, 2, sa, sb, LoadsOf<kNothing>{}, nullptr);
      quarter(S0, S1, 3, sa, sb, LoadsOf<kNothing>{}, nullptr);
      turn();
      quarter(S1, S0, 0, sa1, sb ^ 1, LoadsOf<kWeights>{}, weights(sb));
      advance();
      sa = sa1;
      sb ^= 1;
    }
    if (half) {  // 32 more columns
      const int sa1 = sa == 2 ? 0 : sa + 1, sa2 = sa == 0 ? 2 : sa - 1;
      quarter(S0, S1, 1, sa, sb, LoadsOf<kTokens>{}, tokens(sa2));
#pragma unroll
      for (int q = 0; q < 8; ++q) mma2(S1, q);
      turn();
#pragma unroll
      for (int i = 0; i < 8; ++i) load(i, false, weights(sb));
      advance();
      sa = sa1;
      sb ^= 1;
    }
    // ---- rotary embedding on queries and keys.  Accumulator layout: acc[i][j][r] is token
    //      wm*128 + i*32 + (r/4)*8 + 4h + r%4 of the tile, feature j*32 + m of the wavefront's head.
    //      Features c < 64 pair with c + 64: blocks (0, 2) and (1, 3) of the same lane and register.
    int eln = lane;  // (opaque: address arithmetic hoisted out of the tile loop would not fit the registers)
    asm volatile("" : "+v"(eln));
    const int em = eln & 31, eh = eln >> 5;
    const int ft = ftile * kHeadsPerWg + wn;  // this wavefront's head (an odd head count leaves the last tile's second half idle)
    const int row0 = rt * kBM;                // first token (flattened over sequences) of the tile
    // Token of the flattened row row0 + r (0 <= r < kBM) and its sequence: the tile starts inside
    // sequence seq0 at token tok0; a sequence shorter than a tile can end several times in it.
    const int seq0 = row0 / a.n, tok0 = row0 - seq0 * a.n, first = a.n - tok0;
    const float inv_n = 1.0f / float(a.n);
    auto place = [&](int r, int& seq, int& tok) {
      // sequences that end before the row (exact: r - first < 256, n >= 1; -1 stands for all rows before the first end)
      const int q = int(floorf((float(max(r - first, -1)) + 0.5f) * inv_n)) + 1;
      seq = seq0 + q;
      tok = tok0 + r - q * a.n;
    };
    const bool rotate = ft < a.Hq + a.Hkv, whole = first >= kBM;  // whole: the tile's tokens are of one sequence
    double turns_per_pos[2];  // turns (angle / 2 pi) per position step of this lane's two feature pairs
#pragma unroll
    for (int j = 0; j < 2; ++j)
      turns_per_pos[j] = exp2(-(2.0 * double(j * 32 + em) / double(kBN)) * a.log2_base) * 0.15915494309189535;
    // ---- rotated and through LDS, 32 tokens of the wavefront at a time: [token][feature] in bf16, then
    //      16 contiguous bytes per lane.  The token stage that is free until the next k-tile's loads has room
    //      for it, every wavefront in the part that its own loads fill.
    View dst = a.q;
    int head = ft;
    if (ft >= a.Hq + a.Hkv) {
      dst = a.v;
      head = ft - a.Hq - a.Hkv;
    } else if (ft >= a.Hq) {
      dst = a.k;
      head = ft - a.Hq;
    }
    uint16_t* out = static_cast<uint16_t*>(dst.ptr) + head * dst.sh;
    uint16_t* Cs = tokens(sa == 0 ? 2 : sa - 1) + w * 64 * kLd;
    // the block's values of register r, and their place in the staged rows (rows 4 h apart are
    // written together: the half row's offset puts them on different banks)
    auto put = [&](int r, int j, float v) {
      Cs[((r >> 2) * 8 + eh * 4 + (r & 3)) * kBN + ((j * 32 + em) ^ (eh << 5))] = Elem<uint16_t>::from_f32(v);
    };
    auto put_rotated = [&](int i, int r, int j, float frac) {
      // the hardware sine and cosine take their argument in turns
      const float sn = __builtin_amdgcn_sinf(frac), cs = __builtin_amdgcn_cosf(frac);
      const float x0 = acc[i][j][r], x1 = acc[i][j + 2][r];
      put(r, j, x0 * cs - x1 * sn);
      put(r, j + 2, x1 * cs + x0 * sn);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // the angle in fp64, reduced to a fraction of a turn before the fp32 sine and cosine
      // (positions reach 10^5: an fp32 product would be off by a hundredth of a radian)
      if (!rotate) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) put(r, j, acc[i][j][r]);
      } else if (whole) {  // four consecutive tokens: one product; each angle is reduced before it is rounded
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const double turns = double(a.pos0 + tok0 + wm * 128 + i * 32 + g * 8 + eh * 4) * turns_per_pos[j];
            const double frac = turns - rint(turns);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double t = fma(double(e), turns_per_pos[j], frac);
              put_rotated(i, 4 * g + e, j, float(t - rint(t)));
            }
            __builtin_amdgcn_sched_barrier(0);  // one group after the other: interleaving them costs registers
          }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          int seq, tok;
          place(wm * 128 + i * 32 + (r >> 2) * 8 + eh * 4 + (r & 3), seq, tok);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const double turns = double(a.pos0 + tok) * turns_per_pos[j];
            put_rotated(i, r, j, float(turns - rint(turns)));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int row = c * 4 + (eln >> 4), col = (eln & 15) * 8;
        const int tile_row = wm * 128 + i * 32 + row;
        if (row0 + tile_row < a.M && ft < nheads) {
          int b, tok;
          place(tile_row, b, tok);
          *reinterpret_cast<u32x4*>(out + b * dst.sb + int64_t(tok) * dst.sn + col) =
              *reinterpret_cast<const u32x4*>(Cs + row * kBN + (col ^ (((row >> 2) & 1) << 5)));
        }
      }
    }
  }
}

}  // namespace
}  // namespace d2o

using namespace d2o;

extern "C" int d2o_qkv_project(int32_t batch, int32_t n, int32_t hidden, int32_t n_q_heads, int32_t n_kv_heads,
                               int32_t head_dim, int32_t dtype, const void* X, const void* W, d2o_view Q,
                               d2o_view K, d2o_view V, int32_t pos0, double rope_base, void* stream) {
  if (batch < 1 || n < 1 || hidden < 1 || n_q_heads < 1 || n_kv_heads < 1 || !X || !W || pos0 < 0 ||
      !(rope_base > 1.0))
    return D2O_ERR_INVALID_ARG;
  if (dtype != D2O_BF16 || head_dim != kBN) return D2O_ERR_UNSUPPORTED;
  if (hidden % (kBK / 2)) return D2O_ERR_UNSUPPORTED;
  if (int64_t(batch) * n > 0x7FFFFFFF) return D2O_ERR_INVALID_ARG;
  for (const d2o_view* v : {&Q, &K, &V}) {
    if (!v->ptr || (reinterpret_cast<uintptr_t>(v->ptr) & 15) || v->stride_b % 8 || v->stride_h % 8 ||
        v->stride_n % 8 || v->stride_n < head_dim)
      return D2O_ERR_INVALID_ARG;
  }
  if ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(W)) & 15) return D2O_ERR_INVALID_ARG;
  QkvArgs a;
  a.X = static_cast<const uint16_t*>(X);
  a.W = static_cast<const uint16_t*>(W);
  a.q = to_view(Q);
  a.k = to_view(K);
  a.v = to_view(V);
  a.M = batch * n;
  a.n = n;
  a.hidden = hidden;
  a.Hq = n_q_heads;
  a.Hkv = n_kv_heads;
  a.pos0 = pos0;
  a.log2_base = std::log2(rope_base);
  const int nft = (n_q_heads + 2 * n_kv_heads + kHeadsPerWg - 1) / kHeadsPerWg, ntiles = nft * ((a.M + kBM - 1) / kBM);
  const auto kernel = hidden > kMaxBufferHidden ? qkv_rope_bf16<true> : qkv_rope_bf16<false>;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kSmemBytes) != hipSuccess)
    return D2O_ERR_HIP;
  const int nwg = std::min(ntiles, kCus);
  kernel<<<nwg, kThreads, kSmemBytes, static_cast<hipStream_t>(stream)>>>(a, nft, ntiles, nwg);
  return hipGetLastError() == hipSuccess ? D2O_OK : D2O_ERR_HIP;
}
