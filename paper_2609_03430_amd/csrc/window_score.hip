// Observation-window scorer: the scoring pass of a score-based evictor,
// built only to measure what Random Attention saves (not used by the method).
//
// Section 2 ("Baselines as choices of s") defines SnapKV's score of a cached
// position as the sum of the attention weights of the last w queries,
// max-pooled over neighbouring positions; Eq. 1 keeps the top-scoring
// candidates (cached rows outside the r most recent).  Per (sequence, layer,
// KV head), one workgroup of 1,024 or 512 threads:
//   pass 1: for every window query (G heads x 64 steps) the softmax reference
//           and sum of q.k/sqrt(d) over the cached rows at or before its
//           position;
//   pass 2: the same logits again, the weights summed over queries into a
//           per-row score held in LDS;
//   then max-pool over 7 rows, and the m lowest candidates (the same m as
//   Random Attention drops at this event) by the shared radix select.
// Both passes run on v_mfma_f32_16x16x32_bf16 with 16 queries x 16 keys per
// tile.
//
// Bound by the vector work per logit (a fused multiply-add, an exponential at
// a quarter of the rate, an addition), which the matrix products of the other
// wavefronts of a SIMD run beside: a head has one workgroup, so it fills all
// four wavefronts of every SIMD (128 registers each, none spilled: two query
// tiles; what the loops do not need is derived again where it is used).
// They divide the query tiles and, where these are few, the keys of a
// block between them, so that a key tile read from LDS serves two query tiles
// (one: the LDS reads take longer than the logits).
// Pass 1 keeps its reference as long as no logit passes it by more than 2^8,
// instead of raising it in every block.  240 heads of 9,376 rows,
// G = 4: 575 -> 449 us (G = 1: 220 -> 133 at 192 heads of 4,890 rows, G = 8: 414 ->
// 354; G = 16, 24 heads, whose operands spilled: 4.1 -> 0.63 ms).
#include <type_traits>

#include "ra_internal.h"
#include "select.h"

namespace ra {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Key rows per LDS block of a workgroup of NT threads.
template <int NT>
constexpr int kBlk = NT / 8;
constexpr int kWin = 64;          // window queries per query head
constexpr int kRowStride = 136;   // bf16 elements per LDS row (256 B + 16 B pad)
constexpr int kTilesPerWave = 2;  // query tiles a wavefront holds in registers
constexpr int kPoolHalf = 3;      // max-pool over 7 rows
constexpr float kNegInf = -__builtin_huge_valf();
// Pass 1 raises a query's reference when a logit exceeds it by more than this
// many powers of two: the sums keep their relative precision, far from overflow.
constexpr float kSlack = 8.f;
constexpr float kNoReference = 3e38f;   // minus the reference of a query without keys

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) {
  bf16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}

// LDS of a workgroup besides the scores: 87 KB for 1,024 threads, beside which
// the scores of the longest cache (16,384 rows) take 64 of the 160 KB; 39 KB for
// 512.  The sums of a block are read while the next block's are written.
template <int NT>
struct Lds {
  static constexpr int kWaves = NT / 64;
  union {
    struct {
      uint16_t k[2][kBlk<NT> * kRowStride];
      int pos[2][kBlk<NT>];
      union {
        float sums[2][kWaves][kBlk<NT>];         // [.][query group][key]
        struct {
          float off[kWaves][16], sum[kWaves][16];   // one tile of every wavefront
        } merge;
      };
    } stream;
    struct {
      SelectShared sel;
      int f[kMaxEvery];
    } pick;
  };
};

// A value that the compiler takes as new: what it derives from it is computed
// where it is used, not kept in registers through the loops.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

constexpr int kPieces = 2;
static_assert(kBlk<1024> * 16 == kPieces * 1024, "a block is two pieces per thread");
struct KBlock {
  u32x4 u[kPieces];    // this thread's 16-byte pieces of a block
  int p;               // position of row t (the first threads)
};

template <int NT>
__device__ __forceinline__ void fetch_block(KBlock& b, const uint16_t* Kr,
                                            const int32_t* P, int kb, int len) {
  const int t = fresh(threadIdx.x);
  const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int q = 0; q < kPieces; ++q) {
    const int piece = t + q * NT;          // 16 pieces of 16 bytes to a row
    const int row = piece >> 4, col = piece & 15;
    b.u[q] = (kb + row < len)
        ? *reinterpret_cast<const u32x4*>(Kr + static_cast<int64_t>(kb + row) * kHeadDim + col * 8)
        : z;
  }
  b.p = (t < kBlk<NT> && kb + t < len) ? P[kb + t] : 0x7fffffff;
}

template <int NT>
__device__ __forceinline__ void store_block(const KBlock& b, uint16_t* lk, int* lpos) {
  const int t = fresh(threadIdx.x);
#pragma unroll
  for (int q = 0; q < kPieces; ++q) {
    const int piece = t + q * NT;
    const int row = piece >> 4, col = piece & 15;
    *reinterpret_cast<u32x4*>(lk + row * kRowStride + col * 8) = b.u[q];
  }
  if (t < kBlk<NT>) lpos[t] = b.p;
}

// Stream the head's cached rows through LDS (the next block prefetched into
// registers while the current one is used) and call body(b, keys, positions)
// once per block, with the whole workgroup.
template <int NT, typename Body>
__device__ __forceinline__ void stream_blocks(const uint16_t* Kr, const int32_t* P, int len,
                                              Lds<NT>& lds, Body body) {
  auto& st = lds.stream;
  const int nblk = (len + kBlk<NT> - 1) / kBlk<NT>;
  KBlock nb;
  fetch_block<NT>(nb, Kr, P, 0, len);
  __syncthreads();                 // the previous user of the buffers is done with them
  store_block<NT>(nb, st.k[0], st.pos[0]);
  __syncthreads();
  for (int b = 0; b < nblk; ++b) {
    const int cur = b & 1;
    if (b + 1 < nblk) fetch_block<NT>(nb, Kr, P, (b + 1) * kBlk<NT>, len);
    body(b, st.k[cur], st.pos[cur]);
    // the other buffer was last read before the previous barrier
    if (b + 1 < nblk) store_block<NT>(nb, st.k[cur ^ 1], st.pos[cur ^ 1]);
    __syncthreads();
  }
}

// Key operand of subtile kt (keys kt*16 .. kt*16+15 of the block): lane
// (qi, grp) holds key kt*16 + qi, channels 32s + 8grp .. + 7 at k-step s.
__device__ __forceinline__ void load_kop(bf16x8 (&kop)[4], const uint16_t* lkb, int kt,
                                         int qi, int grp) {
  const uint16_t* krow = lkb + (kt * 16 + qi) * kRowStride + 8 * grp;
#pragma unroll
  for (int s = 0; s < 4; ++s) kop[s] = as_bf16x8(*reinterpret_cast<const u32x4*>(krow + 32 * s));
}

// S^T tiles of two 16-key tiles: 16 window queries (rows) x 16 keys (columns)
// each; the lane holds rows 4*grp + i of column qi.  All chains of products
// advance together.
template <int N>
__device__ __forceinline__ void score_tiles(f32x4 (&x)[2][N],
                                            const bf16x8 (&qop)[kTilesPerWave][4],
                                            const uint16_t* lkb, int kt, int qi, int grp) {
  bf16x8 kop[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    load_kop(kop[h], lkb, kt + h, qi, grp);
#pragma unroll
    for (int j = 0; j < N; ++j) x[h][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < N; ++j)
        x[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qop[j][s], kop[h][s], x[h][j], 0, 0, 0);
}

template <int NT, int KPT>
__global__ __launch_bounds__(NT, 4) void window_score_kernel(
    const SeqMeta* __restrict__ meta, const uint16_t* __restrict__ kpool,
    const int32_t* __restrict__ pos, const uint16_t* __restrict__ qwin,
    float* __restrict__ scores_out, int32_t* __restrict__ drops_out,
    int scores_stride, int L, int Hq, int Hkv, int G, int r, int every,
    int slot_lo, float scale_log2) {
  constexpr int kWaves = NT / 64;
  extern __shared__ __align__(16) char smem[];
  Lds<NT>& lds = *reinterpret_cast<Lds<NT>*>(smem);
  float* score = reinterpret_cast<float*>(smem + sizeof(Lds<NT>));   // [len]

  const int per_seq = L * Hkv;
  const int slot = slot_lo + static_cast<int>(blockIdx.x) / per_seq;
  const int lg = static_cast<int>(blockIdx.x) % per_seq;
  const int layer = lg / Hkv, g = lg % Hkv;
  const SeqMeta& M = meta[slot];
  if (!M.active) return;
  const int len = M.len, lp = M.prompt_len;
  const int m = len - lp - r - M.k_keep;          // rows Random Attention drops
  const int n_cand = len - r;
  const int64_t region = M.base + static_cast<int64_t>(lg) * M.cap;
  const uint16_t* Kr = kpool + region * kHeadDim;
  const int32_t* P = pos + region;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int qi = lane & 15, grp = lane >> 4;
  for (int i = t; i < len; i += NT) score[i] = 0.f;

  const int first_pos = lp + M.step - kWin;     // position of window row 0
  const int n_tiles = G * 4;
  // rounds of as many query tiles as the wavefronts hold (one, up to G = 8)
  for (int tile0 = 0, round = 0; tile0 < n_tiles; tile0 += round) {
    // wavefront = key group * query groups + query group; key group kg takes
    // the 16-key tiles [kg * tiles, (kg + 1) * tiles) of every block.  As many
    // key groups as the round's query tiles leave wavefronts for, but two key
    // tiles at least: G = 1 and 2: 4, G = 3 and 4: 2, more: 1.
    round = min(n_tiles - tile0, kWaves * kTilesPerWave);
    int qgroups = 4;
    while (qgroups * kTilesPerWave < round) qgroups *= 2;
    const int qg = wave % qgroups;
    const int tiles = kBlk<NT> / 16 * qgroups / kWaves, kt0 = wave / qgroups * tiles;
    // this wavefront's query tiles: qt = tile0 + j * qgroups + qg for j < ntile
    // (round robin, so that they spread evenly over the SIMDs; one or two, as
    // a round has at least qgroups tiles); tile qt covers head qt / 4, window
    // rows 16 * (qt % 4) .. + 15
    const int ntile = (round - qg + qgroups - 1) / qgroups;
    const auto by_tiles = [&](auto&& work) {
      if (ntile == kTilesPerWave) work(std::integral_constant<int, kTilesPerWave>{});
      else work(std::integral_constant<int, kTilesPerWave - 1>{});
    };
    bf16x8 qop[kTilesPerWave][4];
#pragma unroll
    for (int j = 0; j < kTilesPerWave; ++j) {
      const int qt = j < ntile ? tile0 + j * qgroups + qg : 0;
      const uint16_t* qrow =
          qwin + ((static_cast<int64_t>(slot) * L + layer) * Hq + g * G + qt / 4) * kWin * kHeadDim +
          static_cast<int64_t>(16 * (qt % 4) + qi) * kHeadDim + 8 * grp;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        qop[j][s] = as_bf16x8(*reinterpret_cast<const u32x4*>(qrow + 32 * s));
    }
    // position of the lane's D-row i of tile j (its window query)
    auto qpos = [&](int j, int i) {
      return first_pos + 16 * ((tile0 + j * qgroups + qg) % 4) + 4 * grp + i;
    };

    // pass 1: per (tile, D-row) minus the reference (in log2 units) and the sum
    // of 2^(x * scale - reference) over this lane's key columns; every window
    // query sees every key of a block unless the block reaches past the first
    // window position (rows beyond len carry an infinite position): only then
    // is the causal mask applied
    float off[kTilesPerWave][4], sum[kTilesPerWave][4];
#pragma unroll
    for (int j = 0; j < kTilesPerWave; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        off[j][i] = kNoReference;
        sum[j][i] = 0.f;
      }
    auto pass1_block = [&](const uint16_t* lkb, const int* lpb, auto count) {
      constexpr int kTiles = decltype(count)::value;
      const bool masked = lpb[kBlk<NT> - 1] > first_pos;
      for (int kt = kt0; kt < kt0 + tiles; kt += 2) {
        f32x4 x[2][kTiles];
        score_tiles(x, qop, lkb, kt, qi, grp);
        if (masked) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int kpos = lpb[(kt + h) * 16 + qi];
#pragma unroll
            for (int j = 0; j < kTiles; ++j)
#pragma unroll
              for (int i = 0; i < 4; ++i)
                if (kpos > qpos(j, i)) x[h][j][i] = kNegInf;
          }
        }
        // the largest exponent as an integer, whose order is the order of the
        // positive values
        float y[2][kTiles][4];
        int top = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int j = 0; j < kTiles; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              y[h][j][i] = fmaf(x[h][j][i], scale_log2, off[j][i]);
              top = max(top, __float_as_int(y[h][j][i]));
            }
        if (__ballot(top > __float_as_int(kSlack))) {
#pragma unroll
          for (int j = 0; j < kTiles; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float o = fminf(off[j][i], -fmaxf(x[0][j][i], x[1][j][i]) * scale_log2);
              sum[j][i] *= __builtin_amdgcn_exp2f(o - off[j][i]);
              off[j][i] = o;
#pragma unroll
              for (int h = 0; h < 2; ++h) y[h][j][i] = fmaf(x[h][j][i], scale_log2, o);
            }
        }
#pragma unroll
        for (int j = 0; j < kTiles; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            sum[j][i] += __builtin_amdgcn_exp2f(y[0][j][i]) + __builtin_amdgcn_exp2f(y[1][j][i]);
      }
    };
    stream_blocks(Kr, P, len, lds, [&](int, const uint16_t* lkb, const int* lpb) {
      by_tiles([&](auto count) { pass1_block(lkb, lpb, count); });
    });
    // merge the 16 lanes holding the same queries, then the key groups; sum
    // becomes the weights' factor 1 / sum (the stream ended with a barrier)
    auto& mg = lds.stream.merge;
#pragma unroll
    for (int j = 0; j < kTilesPerWave; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float o = off[j][i], s = sum[j][i];
#pragma unroll
        for (int w = 1; w < 16; w <<= 1) {
          const float o2 = __shfl_xor(o, w, 64), s2 = __shfl_xor(s, w, 64);
          const float on = fminf(o, o2);
          s = s * __builtin_amdgcn_exp2f(on - o) + s2 * __builtin_amdgcn_exp2f(on - o2);
          o = on;
        }
        if (qi == 0) {
          mg.off[wave][4 * grp + i] = o;
          mg.sum[wave][4 * grp + i] = s;
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float o = kNoReference, s = 0.f;
        for (int w = qg; w < kWaves; w += qgroups) o = fminf(o, mg.off[w][4 * grp + i]);
        for (int w = qg; w < kWaves; w += qgroups)
          s += mg.sum[w][4 * grp + i] * __builtin_amdgcn_exp2f(o - mg.off[w][4 * grp + i]);
        off[j][i] = o;
        sum[j][i] = s == 0.f ? 0.f : 1.f / s;
      }
      __syncthreads();
    }

    // pass 2: the same logits again; the weights of the wavefront's window
    // queries summed per key
    auto pass2_tiles = [&](const uint16_t* lkb, const int* lpb, float* out, auto count,
                           auto masked) {
      constexpr int kTiles = decltype(count)::value;
      for (int kt = kt0; kt < kt0 + tiles; kt += 2) {
        f32x4 d[2][kTiles];
        score_tiles(d, qop, lkb, kt, qi, grp);
        float colsum[2] = {0.f, 0.f};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int kpos = lpb[(kt + h) * 16 + qi];
#pragma unroll
          for (int j = 0; j < kTiles; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float w = __builtin_amdgcn_exp2f(fmaf(d[h][j][i], scale_log2, off[j][i]));
              if constexpr (decltype(masked)::value)
                colsum[h] += kpos > qpos(j, i) ? 0.f : w * sum[j][i];
              else
                colsum[h] = fmaf(w, sum[j][i], colsum[h]);
            }
        }
        // over the four lane groups: even groups collect the first tile, odd
        // ones the second
        const bool odd = grp & 1;
        float c = (odd ? colsum[1] : colsum[0]) + __shfl_xor(odd ? colsum[0] : colsum[1], 16, 64);
        c += __shfl_xor(c, 32, 64);
        const int l = fresh(threadIdx.x) & 63;    // grp * 16 + qi
        if (l < 32) out[kt * 16 + l] = c;
      }
    };
    // the sums of block b over the query groups, in their order
    auto add_block = [&](int b) {
      const int t = fresh(threadIdx.x), key = b * kBlk<NT> + t;
      if (t < kBlk<NT> && key < len) {
        float s = score[key];
        for (int w = 0; w < qgroups; ++w) s += lds.stream.sums[b % 2][w][t];
        score[key] = s;
      }
    };
    stream_blocks(Kr, P, len, lds, [&](int b, const uint16_t* lkb, const int* lpb) {
      if (b > 0) add_block(b - 1);
      float* out = lds.stream.sums[b % 2][qg];
      by_tiles([&](auto count) {
        if (lpb[kBlk<NT> - 1] > first_pos) pass2_tiles(lkb, lpb, out, count, std::true_type{});
        else pass2_tiles(lkb, lpb, out, count, std::false_type{});
      });
    });
    add_block((len - 1) / kBlk<NT>);
  }
  __syncthreads();

  const int64_t head_out = static_cast<int64_t>(slot - slot_lo) * per_seq + lg;
  if (scores_out) {
    for (int i = t; i < len; i += NT) scores_out[head_out * scores_stride + i] = score[i];
  }
  if (!drops_out || m <= 0) return;
  // max-pool and select the m lowest candidates
  uint64_t key[KPT];
  uint32_t tie[KPT];
  uint32_t valid = 0;
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const int c = t * KPT + i;
    key[i] = 0;
    tie[i] = static_cast<uint32_t>(c);      // ties by row, lower first
    if (c < n_cand) {
      float mxp = 0.f;
      for (int j = max(0, c - kPoolHalf); j <= min(len - 1, c + kPoolHalf); ++j)
        mxp = fmaxf(mxp, score[j]);
      key[i] = __float_as_uint(mxp);        // non-negative: bit order = value order
      valid |= 1u << i;
    }
  }
  const uint32_t drop = select_smallest<NT, KPT, 32>(key, tie, valid, m, lds.pick.sel);
  int* f = lds.pick.f;
  drop_list<NT, KPT>(drop, 0, f, lds.pick.sel);
  for (int k = t; k < m; k += NT) drops_out[head_out * every + k] = f[k] + k;
}

}  // namespace

hipError_t launch_window_score(const Shape& sh, const SeqMeta* meta, const void* kpool,
                               const int32_t* pos, const void* qwin, float* scores_out,
                               int32_t* drops_out, int scores_stride, int slot_lo,
                               int slot_hi, int max_len, hipStream_t s) {
  if (slot_hi <= slot_lo) return hipSuccess;
  const dim3 grid((slot_hi - slot_lo) * sh.L * sh.Hkv);
  const float scale = 1.4426950408889634f / sqrtf(static_cast<float>(kHeadDim));
  const uint16_t* k = static_cast<const uint16_t*>(kpool);
  const uint16_t* q = static_cast<const uint16_t*>(qwin);
  const int n_cand = max_len;   // upper bound of len - r
  const auto shmem = [&](size_t fixed) { return fixed + sizeof(float) * static_cast<size_t>(max_len); };
#define RA_WS_LAUNCH(NT, K)                                                                \
  hipLaunchKernelGGL((window_score_kernel<NT, K>), grid, dim3(NT), shmem(sizeof(Lds<NT>)), s, \
                     meta, k, pos, q, scores_out, drops_out, scores_stride, sh.L, sh.Hq,   \
                     sh.Hkv, sh.G, sh.r, sh.every, slot_lo, scale)
  // More heads than CUs, short caches: two workgroups of 512 threads to a CU
  // overlap their prologues, barriers and selections, where those of 1,024 run one
  // by one (1,024 and 512 threads, us at G = 4: 264 heads of 490 rows 82 and 60, of
  // 1,190 135 and 111, of 2,690 244 and 220, of 4,090 336 and 316; 512 heads of 4,090
  // alike; 256 heads of 1,190 77 and 78, of 2,690 135 and 153).  Above G = 4 they
  // would read the keys a second time.
  if (grid.x > 256 && sh.G <= 4 && n_cand <= 512 * 4) RA_WS_LAUNCH(512, 4);
  else if (grid.x > 256 && sh.G <= 4 && n_cand <= 512 * 8) RA_WS_LAUNCH(512, 8);
  else if (n_cand <= 1024 * 4) RA_WS_LAUNCH(1024, 4);
  else if (n_cand <= 1024 * 8) RA_WS_LAUNCH(1024, 8);
  else if (n_cand <= 1024 * 16) RA_WS_LAUNCH(1024, 16);
  else return hipErrorInvalidValue;
#undef RA_WS_LAUNCH
  return hipGetLastError();
}

}  // namespace ra
