// Selection steps of two score-based evictors, built only to price the
// selection signal that Random Attention does without (not used by the
// method).  Section 2 ("Baselines as choices of s") defines the scores:
//   R-KV: s_i = lambda * SnapKV_i - (1 - lambda) * softmax_i(cbar), cbar_i
//         the mean cosine similarity of key i to the other cached keys, its
//         most recent near-duplicates not counted;
//   VaSE: keep the n_large rows of largest value range, fill the rest of the
//         budget by sampling without replacement in proportion to SnapKV.
// Both read the raw observation-window scores that window_score.hip wrote
// for the same state (SnapKV_i = their max over rows i-3 .. i+3), select the
// m rows to drop among the candidates (every cached row outside the r most
// recent: the prompt competes), and write the ascending drop list that the
// compaction of evict.hip consumes.  One workgroup per (sequence, layer, KV
// head); candidates live in registers, KPT consecutive rows per thread.
#include <math.h>

#include <type_traits>

#include "philox.h"
#include "ra_internal.h"
#include "select.h"

namespace ra {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kNT = 512;
constexpr int kPoolHalf = 3;

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) {
  bf16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) {
  return __uint_as_float(h << 16);
}

// Order-preserving maps of floating-point values onto unsigned integers.
__device__ __forceinline__ uint64_t order_key_f64(double x) {
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(x));
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ uint64_t order_key_f32(float x) {
  const uint32_t b = __float_as_uint(x);
  return (b >> 31) ? static_cast<uint64_t>(~b) : static_cast<uint64_t>(b | 0x80000000u);
}

// SnapKV score of candidate c: the raw window score max-pooled over 7 rows.
__device__ __forceinline__ float pooled_score(const float* raw, int c, int len) {
  float mx = 0.f;
  for (int j = max(0, c - kPoolHalf); j <= min(len - 1, c + kPoolHalf); ++j)
    mx = fmaxf(mx, raw[j]);
  return mx;
}

struct Head {
  int slot, lg, layer, g, len, lp, m, n_cand, budget;
  int64_t region;
  bool active;
};

__device__ __forceinline__ Head locate_head(const SeqMeta* meta, int L, int Hkv, int r,
                                            int slot_lo) {
  Head h;
  const int per_seq = L * Hkv;
  h.slot = slot_lo + static_cast<int>(blockIdx.x) / per_seq;
  h.lg = static_cast<int>(blockIdx.x) % per_seq;
  h.layer = h.lg / Hkv;
  h.g = h.lg % Hkv;
  const SeqMeta& M = meta[h.slot];
  h.len = M.len;
  h.lp = M.prompt_len;
  h.budget = M.prompt_len + M.k_keep;
  h.n_cand = M.len - r;
  h.m = h.n_cand - h.budget;
  h.region = M.base + static_cast<int64_t>(h.lg) * M.cap;
  h.active = M.active && h.m > 0;
  return h;
}

// ---------------------------------------------------------------------------
// VaSE
// ---------------------------------------------------------------------------

template <int KPT>
__global__ __launch_bounds__(kNT) void vase_kernel(
    const SeqMeta* __restrict__ meta, const uint16_t* __restrict__ vpool,
    const int32_t* __restrict__ pos, const float* __restrict__ raw_scores, int score_stride,
    int32_t* __restrict__ drops, int every, int L, int Hkv, int r, int slot_lo,
    int n_large_cfg, uint64_t seed) {
  extern __shared__ uint32_t vmm[];             // per row: bf16 max (hi) | bf16 min (lo)
  __shared__ SelectShared sel_sh;
  __shared__ int f[kMaxEvery];
  const Head h = locate_head(meta, L, Hkv, r, slot_lo);
  if (!h.active) return;
  const SeqMeta& M = meta[h.slot];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int32_t* P = pos + h.region;
  const float* raw = raw_scores + static_cast<int64_t>(blockIdx.x) * score_stride;

  // 1. value range of every candidate row: a wavefront takes an 8-row value
  // tile (128 channels x 8 rows, transposed); lane l reads channels 2l and
  // 2l + 1 (16 bytes each) and the wavefront reduces max and min per row
  const int n_tiles = (h.n_cand + 7) / 8;
  for (int tile = wave; tile < n_tiles; tile += kNT / 64) {
    const uint16_t* base = vpool + (h.region + 8 * tile) * kHeadDim;
    float mx[8], mn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mx[e] = -__builtin_huge_valf();
      mn[e] = __builtin_huge_valf();
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(base + (2 * lane + c) * 8);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = bf16_bits_to_f32((w[e >> 1] >> (16 * (e & 1))) & 0xFFFF);
        mx[e] = fmaxf(mx[e], x);
        mn[e] = fminf(mn[e], x);
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        mx[e] = fmaxf(mx[e], __shfl_xor(mx[e], o, 64));
        mn[e] = fminf(mn[e], __shfl_xor(mn[e], o, 64));
      }
    }
    if (lane < 8) {
      float a = mx[0], b = mn[0];
#pragma unroll
      for (int e = 1; e < 8; ++e)
        if (lane == e) {
          a = mx[e];
          b = mn[e];
        }
      const int row = 8 * tile + lane;
      // bf16 values: the upper 16 bits of their float are exact
      if (row < h.n_cand) vmm[row] = (__float_as_uint(a) & 0xFFFF0000u) | (__float_as_uint(b) >> 16);
    }
  }
  __syncthreads();

  // 2. the large set: the n_large largest (range, position); the other
  // candidates are the n_cand - n_large smallest
  const int n_large = n_large_cfg < 0 ? h.budget / 2 : min(n_large_cfg, h.budget);
  uint64_t key[KPT];
  uint32_t tie[KPT];
  uint32_t valid = 0;
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const int c = t * KPT + i;
    key[i] = 0;
    tie[i] = 0;
    if (c < h.n_cand) {
      const uint32_t mm = vmm[c];
      const double rg = static_cast<double>(bf16_bits_to_f32(mm >> 16)) -
                        static_cast<double>(bf16_bits_to_f32(mm & 0xFFFF));
      key[i] = static_cast<uint64_t>(__double_as_longlong(rg));   // >= 0: bits are ordered
      tie[i] = static_cast<uint32_t>(P[c]);
      valid |= 1u << i;
    }
  }
  const uint32_t small = n_large > 0
      ? select_smallest<kNT, KPT, 64>(key, tie, valid, h.n_cand - n_large, sel_sh)
      : valid;
  __syncthreads();

  // 3. proportional fill among the others: Efraimidis-Spirakis keys
  // log(u) / w (the largest kept), u in (0, 1] from the Philox word of the
  // position, w the SnapKV score; the m smallest are dropped
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    if ((small >> i) & 1) {
      const int c = t * KPT + i;
      const int p = P[c];
      const uint64_t x = philox_score(static_cast<uint64_t>(p), static_cast<uint64_t>(M.event),
                                      static_cast<uint64_t>(h.layer), static_cast<uint64_t>(h.g),
                                      seed, M.rid);
      const double u = static_cast<double>((x >> 11) + 1) * 0x1.0p-53;
      const float w = pooled_score(raw, c, h.len);
      const double e = w > 0.f ? log(u) / static_cast<double>(w) : -__builtin_huge_val();
      key[i] = order_key_f64(e);
    }
  }
  const uint32_t drop = select_smallest<kNT, KPT, 64>(key, tie, small, h.m, sel_sh);
  drop_list<kNT, KPT>(drop, 0, f, sel_sh);
  int32_t* out = drops + static_cast<int64_t>(blockIdx.x) * every;
  for (int k = t; k < h.m; k += kNT) out[k] = f[k] + k;
}

// ---------------------------------------------------------------------------
// R-KV
// ---------------------------------------------------------------------------

constexpr int kRowTiles = 4;                          // 16-row tiles per wavefront
constexpr int kChunkRows = (kNT / 64) * kRowTiles * 16;   // rows per workgroup: 512
constexpr int kColBlk = 128;      // columns (cached keys) per LDS block
constexpr int kColTiles = kColBlk / 16;
constexpr int kColStride = 136;   // bf16 elements per LDS row (256 B + 16 B pad)
constexpr int kXcds = 8;          // workgroups go to the dies round robin

// Sum of squares of 8 bf16 elements.
__device__ __forceinline__ float sumsq8(u32x4 u) {
  const bf16x8 v = as_bf16x8(u);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float x = static_cast<float>(v[e]);
    s = fmaf(x, x, s);
  }
  return s;
}

__device__ __forceinline__ float inv_norm(float sumsq) {
  return sumsq > 0.f ? 1.f / sqrtf(sumsq) : 0.f;
}

constexpr int kPieces = kColBlk * kHeadDim / 8 / kNT;   // 16-byte pieces per thread and block
static_assert(kPieces == 4, "store_cols deals four keys' norms to the lanes of a row");

// This thread's pieces of the column block that starts at key kb (the 16
// threads of a lane row hold one key; zeros past the last key).
__device__ __forceinline__ void fetch_cols(u32x4 (&u)[kPieces], const uint16_t* Kr, int kb,
                                           int len) {
#pragma unroll
  for (int q = 0; q < kPieces; ++q) {
    const int piece = threadIdx.x + q * kNT, row = kb + (piece >> 4);
    const u32x4 z = {0u, 0u, 0u, 0u};
    u[q] = row < len ? *reinterpret_cast<const u32x4*>(
                           Kr + static_cast<int64_t>(row) * kHeadDim + (piece & 15) * 8)
                     : z;
  }
}

// The sum over the 16 lanes of a row, in every lane of it.
__device__ __forceinline__ float row_sum(float x) {
  const auto ror = [](float v, auto n) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v),
                                                      0x120 + decltype(n)::value, 0xf, 0xf, false));
  };
  x += ror(x, std::integral_constant<int, 8>{});
  x += ror(x, std::integral_constant<int, 4>{});
  x += ror(x, std::integral_constant<int, 2>{});
  x += ror(x, std::integral_constant<int, 1>{});
  return x;
}

// The block into LDS, with 1 / norm of every key: one lane of a row for each of
// its four keys.
__device__ __forceinline__ void store_cols(const u32x4 (&u)[kPieces], uint16_t* lk,
                                           float* linv) {
  float ss[kPieces];
#pragma unroll
  for (int q = 0; q < kPieces; ++q) {
    const int piece = threadIdx.x + q * kNT, row = piece >> 4;
    *reinterpret_cast<u32x4*>(lk + row * kColStride + (piece & 15) * 8) = u[q];
    ss[q] = row_sum(sumsq8(u[q]));
  }
  const int q = threadIdx.x & 3;
  const float mine = q & 2 ? (q & 1 ? ss[3] : ss[2]) : (q & 1 ? ss[1] : ss[0]);
  if ((threadIdx.x & 15) < kPieces) linv[(threadIdx.x + q * kNT) >> 4] = inv_norm(mine);
}

// cbar of the candidate rows [chunk * 512, chunk * 512 + 512) of one head.
// D = K_rows . K_cols^T on v_mfma_f32_16x16x32_bf16: lane l holds rows
// 4*(l/16) + i of a row tile and column l % 16 of a column tile.  Columns are
// swept from the most recent (highest slot = highest position in the
// chronological layout) down, so the first `recent_dups` near-duplicates a
// row meets are the ones not counted; a ballot gives each row its
// near-duplicate columns in a tile.
//
// Bound by the matrix cores and the vector work per similarity together.  The
// workgroup streams 128 columns at a time through LDS (the next block in
// registers meanwhile), so a key is loaded and its norm taken once per 512
// rows instead of once per 64, and a similarity that is not near a duplicate
// costs a multiply, a fused add and half a maximum.  A wavefront's four row
// tiles are four independent chains of products, the next column tile's
// operand on its way from LDS meanwhile.  The chunks of a head run
// on one die, whose L2 then holds its keys.  256 heads of 4,524 rows
// (1.37 TFLOP of products): 2.65 -> 1.27 ms (1.08 PFLOP/s).
__global__ __launch_bounds__(kNT, 2) void rkv_cbar_kernel(
    const SeqMeta* __restrict__ meta, const uint16_t* __restrict__ kpool,
    float* __restrict__ cbar_out, int stride, int n_heads, int n_chunks, int L, int Hkv, int r,
    int slot_lo, float threshold, int recent_dups) {
  __shared__ __align__(16) uint16_t lk[2][kColBlk * kColStride];   // 16-byte pieces
  __shared__ float linv[2][kColBlk];
  const int die = static_cast<int>(blockIdx.x) % kXcds, nth = static_cast<int>(blockIdx.x) / kXcds;
  const int head_idx = nth / n_chunks * kXcds + die;
  const int chunk = nth % n_chunks;
  if (head_idx >= n_heads) return;
  const int per_seq = L * Hkv;
  const int slot = slot_lo + head_idx / per_seq;
  const int lg = head_idx % per_seq;
  const SeqMeta& M = meta[slot];
  const int len = M.len, n_cand = M.len - r;
  if (!M.active || n_cand - (M.prompt_len + M.k_keep) <= 0) return;
  if (chunk * kChunkRows >= n_cand) return;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int qi = lane & 15, grp = lane >> 4;
  const int rt0 = (chunk * kChunkRows) / 16 + wave * kRowTiles;
  const bool busy = rt0 * 16 < n_cand;   // past the candidates: a wavefront only loads
  const uint16_t* Kr = kpool + (M.base + static_cast<int64_t>(lg) * M.cap) * kHeadDim;

  bf16x8 a[kRowTiles][4];
  float sum[kRowTiles][4], invr[kRowTiles][4];
  int found[kRowTiles][4];
#pragma unroll
  for (int q = 0; q < kRowTiles; ++q) {
    const uint16_t* row = Kr + static_cast<int64_t>(min((rt0 + q) * 16 + qi, len - 1)) * kHeadDim;
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x4 u = *reinterpret_cast<const u32x4*>(row + 32 * s + 8 * grp);
      a[q][s] = as_bf16x8(u);
      ss += sumsq8(u);
    }
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    const float inv = inv_norm(ss);                          // row qi of the tile
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sum[q][i] = 0.f;
      found[q][i] = 0;
      invr[q][i] = __shfl(inv, 4 * grp + i, 64);             // D-row 4*grp + i
    }
  }
  const int n_blk = (len + kColBlk - 1) / kColBlk;
  u32x4 next[kPieces];
  fetch_cols(next, Kr, (n_blk - 1) * kColBlk, len);
  store_cols(next, lk[0], linv[0]);
  __syncthreads();
  for (int b = n_blk - 1, cur = 0; b >= 0; --b, cur ^= 1) {
    if (b > 0) fetch_cols(next, Kr, (b - 1) * kColBlk, len);   // next block in flight
    if (busy) {
      const uint16_t* krow = lk[cur] + qi * kColStride + 8 * grp;
      const auto load_cols = [&](bf16x8 (&bop)[4], float& invc, int kt) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
          bop[s] = as_bf16x8(
              *reinterpret_cast<const u32x4*>(krow + kt * 16 * kColStride + 32 * s));
        invc = linv[cur][kt * 16 + qi];
      };
      // the last block's tiles past the last key hold zeros
      bf16x8 bop[2][4];
      float invc[2];
      load_cols(bop[(kColTiles - 1) & 1], invc[(kColTiles - 1) & 1], kColTiles - 1);
#pragma unroll
      for (int kt = kColTiles - 1; kt >= 0; --kt) {
        const int ct = b * kColTiles + kt;
        if (kt > 0) load_cols(bop[(kt - 1) & 1], invc[(kt - 1) & 1], kt - 1);
        f32x4 d[kRowTiles];
#pragma unroll
        for (int q = 0; q < kRowTiles; ++q) d[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int q = 0; q < kRowTiles; ++q)
            d[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[q][s], bop[kt & 1][s], d[q], 0, 0, 0);
        // a row's own column counts as nothing
        if (ct >= rt0 && ct < rt0 + kRowTiles) {
#pragma unroll
          for (int q = 0; q < kRowTiles; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (ct == rt0 + q && 4 * grp + i == qi) d[q][i] = 0.f;
        }
        // every similarity into the sums; the largest x of the lane as an
        // integer, whose order is the order of the positive values (a NaN is
        // the largest)
        const float ic = invc[kt & 1];
        int top = 0;
#pragma unroll
        for (int q = 0; q < kRowTiles; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float x = d[q][i] * invr[q][i];
            sum[q][i] = fmaf(x, ic, sum[q][i]);
            top = max(top, __float_as_int(x));
          }
        // the few tiles with a near-duplicate take the recent ones out again.
        // The factor ic is not negative: the largest similarity is that of `top`.
        if (threshold < 0.f || __ballot(!(__int_as_float(top) * ic <= threshold))) {
          const int col = ct * 16 + qi;
#pragma unroll
          for (int q = 0; q < kRowTiles; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int row = (rt0 + q) * 16 + 4 * grp + i;
              const bool ok = col < len && col != row;
              const float c = d[q][i] * invr[q][i] * ic;
              const uint64_t bal = __ballot(ok && c > threshold);
              const uint32_t bits = static_cast<uint32_t>(bal >> (16 * grp)) & 0xFFFFu;
              const int need = recent_dups - found[q][i];
              // this column is one of the row's `need` most recent duplicates here
              const bool skip = need > 0 && ((bits >> qi) & 1u) && __popc(bits >> (qi + 1)) < need;
              if (skip) sum[q][i] -= c;
              if (need > 0) found[q][i] += min(need, __popc(bits));
            }
        }
      }
    }
    // the other buffer was last read before the previous barrier
    if (b > 0) store_cols(next, lk[cur ^ 1], linv[cur ^ 1]);
    __syncthreads();
  }
  if (!busy) return;
  float* out = cbar_out + static_cast<int64_t>(head_idx) * stride;
#pragma unroll
  for (int q = 0; q < kRowTiles; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v = sum[q][i];
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
      const int row = (rt0 + q) * 16 + 4 * grp + i;
      if (qi == 0 && row < n_cand) out[row] = v / static_cast<float>(len - 1);
    }
}

// softmax of cbar over the candidates, the mix with SnapKV, and the m lowest.
template <int KPT>
__global__ __launch_bounds__(kNT) void rkv_select_kernel(
    const SeqMeta* __restrict__ meta, const int32_t* __restrict__ pos,
    const float* __restrict__ raw_scores, const float* __restrict__ cbar_in, int stride,
    int32_t* __restrict__ drops, int every, int L, int Hkv, int r, int slot_lo,
    float lambda) {
  __shared__ SelectShared sel_sh;
  __shared__ int f[kMaxEvery];
  __shared__ float red[kNT / 64];
  const Head h = locate_head(meta, L, Hkv, r, slot_lo);
  if (!h.active) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int32_t* P = pos + h.region;
  const float* raw = raw_scores + static_cast<int64_t>(blockIdx.x) * stride;
  const float* cbar = cbar_in + static_cast<int64_t>(blockIdx.x) * stride;

  float cb[KPT];
  float mx = -__builtin_huge_valf();
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const int c = t * KPT + i;
    cb[i] = c < h.n_cand ? cbar[c] : -__builtin_huge_valf();
    mx = fmaxf(mx, cb[i]);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  mx = red[0];
#pragma unroll
  for (int w = 1; w < kNT / 64; ++w) mx = fmaxf(mx, red[w]);
  __syncthreads();
  float sm = 0.f;
#pragma unroll
  for (int i = 0; i < KPT; ++i)
    if (t * KPT + i < h.n_cand) sm += expf(cb[i] - mx);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) sm += __shfl_xor(sm, o, 64);
  if (lane == 0) red[wave] = sm;
  __syncthreads();
  sm = 0.f;
#pragma unroll
  for (int w = 0; w < kNT / 64; ++w) sm += red[w];

  uint64_t key[KPT];
  uint32_t tie[KPT];
  uint32_t valid = 0;
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const int c = t * KPT + i;
    key[i] = 0;
    tie[i] = 0;
    if (c < h.n_cand) {
      const float s = lambda * pooled_score(raw, c, h.len) -
                      (1.f - lambda) * (expf(cb[i] - mx) / sm);
      key[i] = order_key_f32(s);
      tie[i] = static_cast<uint32_t>(P[c]);
      valid |= 1u << i;
    }
  }
  const uint32_t drop = select_smallest<kNT, KPT, 32>(key, tie, valid, h.m, sel_sh);
  drop_list<kNT, KPT>(drop, 0, f, sel_sh);
  int32_t* out = drops + static_cast<int64_t>(blockIdx.x) * every;
  for (int k = t; k < h.m; k += kNT) out[k] = f[k] + k;
}

template <int KPT>
hipError_t launch_kpt(int scorer, dim3 grid, size_t lds_rows, hipStream_t s,
                      const SeqMeta* meta, const void* vpool, const int32_t* pos,
                      const float* raw, const float* cbar, int stride, int32_t* drops,
                      int every, int L, int Hkv, int r, int slot_lo, float lambda,
                      int n_large, uint64_t seed) {
  if (scorer == 2) {
    hipLaunchKernelGGL((vase_kernel<KPT>), grid, dim3(kNT), lds_rows * sizeof(uint32_t), s,
                       meta, static_cast<const uint16_t*>(vpool), pos, raw, stride, drops,
                       every, L, Hkv, r, slot_lo, n_large, seed);
  } else {
    hipLaunchKernelGGL((rkv_select_kernel<KPT>), grid, dim3(kNT), 0, s, meta, pos, raw,
                       cbar, stride, drops, every, L, Hkv, r, slot_lo, lambda);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_scored_select(const Shape& sh, int scorer, const SeqMeta* meta,
                                const void* kpool, const void* vpool, const int32_t* pos,
                                const float* raw_scores, float* cbar_scratch,
                                int score_stride, int32_t* drops, int slot_lo, int slot_hi,
                                int max_len, float lambda, float threshold, int recent_dups,
                                int n_large, uint64_t seed, hipStream_t s) {
  if (slot_hi <= slot_lo) return hipSuccess;
  const int heads = (slot_hi - slot_lo) * sh.L * sh.Hkv;
  const dim3 grid(heads);
  const int n_cand = max_len;   // upper bound of len - r
  if (scorer == 1) {
    const int n_chunks = (n_cand + kChunkRows - 1) / kChunkRows;
    const int groups = (heads + kXcds - 1) / kXcds * kXcds * n_chunks;
    hipLaunchKernelGGL(rkv_cbar_kernel, dim3(groups), dim3(kNT), 0, s, meta,
                       static_cast<const uint16_t*>(kpool), cbar_scratch, score_stride,
                       heads, n_chunks, sh.L, sh.Hkv, sh.r, slot_lo, threshold, recent_dups);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const size_t rows = static_cast<size_t>(max_len);
#define RA_SC_LAUNCH(K)                                                                  \
  launch_kpt<K>(scorer, grid, rows, s, meta, vpool, pos, raw_scores, cbar_scratch,       \
                score_stride, drops, sh.every, sh.L, sh.Hkv, sh.r, slot_lo, lambda,      \
                n_large, seed)
  if (n_cand <= kNT * 4) return RA_SC_LAUNCH(4);
  if (n_cand <= kNT * 8) return RA_SC_LAUNCH(8);
  if (n_cand <= kNT * 16) return RA_SC_LAUNCH(16);
  if (n_cand <= kNT * 32) return RA_SC_LAUNCH(32);
#undef RA_SC_LAUNCH
  return hipErrorInvalidValue;
}

}  // namespace ra
