// Grouped-query decode attention over the compressed per-KV-head cache, with
// the step's append fused in (Section 2, "Notation": o = sum_i alpha_i v_i,
// alpha = softmax_i(q . k_i / sqrt(d)); Appendix F: the G query heads of a
// group read their KV head's cache).
//
// Work decomposition: one workgroup of W wavefronts per (sequence, KV head,
// split of `split_keys` keys); wavefront v streams the v-th W-th of the
// split.  Each wavefront reads its keys and values exactly once for all G
// query heads of the group and keeps an online softmax (running max and sum,
// combined across lanes with wavefront shuffles); the W states merge in LDS.
// A head with one split writes its normalised output directly; otherwise
// every split writes an unnormalised partial, and the last one to finish
// merges them (the contiguous 12-wavefront build: a second kernel).  The
// step's new key/value is read from the input buffers by
// the wavefront that owns the last key, which also stores it into the cache
// after its reads, so no wavefront of the launch reads a row that is being
// written.  Value tiles are read with nontemporal loads, key rows with
// ordinary ones.
//
// bf16 path (MFMA, v_mfma_f32_16x16x32_bf16, 16x16 output tiles):
//   S^T[key][query] = K . Q^T   A = 16 key rows x 32 channels, B = Q^T with
//                               the group's G queries on the N side (padded
//                               to 16 with zeros);
//   O^T[ch][query] += V^T . P^T A = 16 channels x 32 keys from the
//                               transposed value tiles, B = P^T split into
//                               two bf16 parts (hi + lo) for precision.
// A lane's 8 operand elements come from one 16-byte global load: key rows
// are row-major and value rows are stored as transposed 8-row tiles.  The
// key rows are assigned to the two 16-row S tiles so that each lane's
// 8 softmax weights are exactly the 8 keys its P^T operand needs (tile t
// row 4a+i holds key 8a+4t+i), so no data moves between lanes except the
// two shuffles of the row maximum.
// fp32 path (MFMA, v_mfma_f32_16x16x4_f32): the same two products over
// 16-key blocks, the softmax weights kept in fp32.
#include <mutex>
#include <type_traits>

#include "ra_internal.h"

namespace ra {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kNegInf = -__builtin_huge_valf();

// The largest score of a state that has seen none but -inf (masked keys, or rows
// that score so): finite, so that the weights of such keys and the rescale come
// out 0 and 1, where the difference of two infinities would make them NaN.
constexpr float kNoScore = -3.4028234663852886e38f;

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) {
  bf16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}

__device__ __forceinline__ u32x4 ld16(const void* p) {
  return *reinterpret_cast<const u32x4*>(p);
}

// Streaming load (nontemporal): the cached rows are read once per launch, so
// they are fetched without being kept in the caches.  Used where a load
// instruction covers whole 128-byte lines (the value tiles); a key load
// covers half lines of 16 rows, whose other halves the next load reads.
__device__ __forceinline__ u32x4 ld16_stream(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}

__device__ __forceinline__ uint16_t f32_to_bf16(float x) {
  __bf16 b = static_cast<__bf16>(x);   // round to nearest even
  uint16_t h;
  __builtin_memcpy(&h, &b, 2);
  return h;
}

struct Work {
  int slot, g, split;
  int len, n_keys, k0, k1, nsplit;
  RowMap rm;       // where the rows of the (slot, layer, g) cache live
  bool valid;
};

__device__ __forceinline__ Work locate(const SeqMeta* meta, int layer, int Hkv,
                                       int split_keys, const Paging& pg) {
  Work w;
  w.split = blockIdx.x;
  w.g = blockIdx.y;
  w.slot = blockIdx.z;
  const SeqMeta& M = meta[w.slot];
  w.valid = false;
  if (!M.active) return w;
  w.len = M.len;
  w.n_keys = w.len + 1;
  w.k0 = w.split * split_keys;
  if (w.k0 >= w.n_keys) return w;
  w.k1 = min(w.k0 + split_keys, w.n_keys);
  w.nsplit = (w.n_keys + split_keys - 1) / split_keys;
  w.rm = row_map(M, w.slot, layer * Hkv + w.g, pg);
  w.valid = true;
  return w;
}

// Store the step's new pair into the cache (row `len` of the head).
template <typename E, bool PAGED>
__device__ __forceinline__ void append_row(const Work& w, const SeqMeta* meta,
                                           int Hkv, const E* k_new,
                                           const E* v_new, E* kpool, E* vpool,
                                           int32_t* pos) {
  const int lane = threadIdx.x & 63;   // called by one whole wavefront
  const int64_t src = (static_cast<int64_t>(w.slot) * Hkv + w.g) * kHeadDim;
  const int64_t row = pool_row<PAGED>(w.rm, w.len);
  for (int c = lane; c < kHeadDim; c += 64) {
    kpool[row * kHeadDim + c] = k_new[src + c];
    vpool[(row & ~int64_t(7)) * kHeadDim + c * 8 + (row & 7)] = v_new[src + c];
  }
  if (lane == 0) pos[row] = meta[w.slot].prompt_len + meta[w.slot].step;
}

// Merge the split partials of one (sequence, KV head) into the output, for
// the 12-wavefront contiguous bf16 build (heads of one split write their
// output themselves).
// One workgroup per head, launched after the attention kernel (the kernel
// boundary makes every partial visible).  Partial layout:
//   ws_o[((head * split_stride + split) * G + q) * 128 + c]  numerator / 2^m
//   ws_ml[((head * split_stride + split) * G + q) * 2 + {0,1}] = (m, l)
// with m the running max of the scores in log2 units and l the sum of
// 2^(s - m) over the split's keys.
__global__ __launch_bounds__(256) void combine_kernel(AttnLaunch a, int G, int Hq, int Hkv) {
  __shared__ float sm[kMaxSplits * kMaxGroup];   // split maxima, then weights
  __shared__ float sl[kMaxSplits * kMaxGroup];   // split sums
  __shared__ float inv_l[kMaxGroup];
  const int g = blockIdx.x, slot = blockIdx.y;
  const SeqMeta& M = a.meta[slot];
  if (!M.active) return;
  const int t = threadIdx.x;
  const int n_keys = M.len + 1;
  const int nsplit = (n_keys + a.split_keys - 1) / a.split_keys;
  if (nsplit == 1) return;
  const int head = slot * Hkv + g;
  const float* ml = a.ws_ml + static_cast<int64_t>(head) * a.split_stride * G * 2;
  const float* po = a.ws_o + static_cast<int64_t>(head) * a.split_stride * G * kHeadDim;
  for (int i = t; i < nsplit * G; i += blockDim.x) {
    sm[i] = ml[2 * i];
    sl[i] = ml[2 * i + 1];
  }
  __syncthreads();
  // per query: global max, split weights 2^(m_s - max) and the total sum
  if (t < G) {
    float mx = kNegInf;
    for (int s = 0; s < nsplit; ++s) mx = fmaxf(mx, sm[s * G + t]);
    float lsum = 0.f;
    for (int s = 0; s < nsplit; ++s) {
      const float w = exp2f(sm[s * G + t] - mx);
      sm[s * G + t] = w;
      lsum += w * sl[s * G + t];
    }
    inv_l[t] = 1.f / lsum;
  }
  __syncthreads();
  uint16_t* out = static_cast<uint16_t*>(a.out);
  // one thread per (query, 4 channels)
  for (int item = t; item < G * (kHeadDim / 4); item += blockDim.x) {
    const int q = item / (kHeadDim / 4), c4 = (item % (kHeadDim / 4)) * 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int s = 0; s < nsplit; ++s) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(
          po + static_cast<int64_t>(s * G + q) * kHeadDim + c4);
      acc += v * sm[s * G + q];
    }
    acc *= inv_l[q];
    const int64_t orow = (static_cast<int64_t>(slot) * Hq + g * G + q) * kHeadDim + c4;
#pragma unroll
    for (int j = 0; j < 4; ++j) out[orow + j] = f32_to_bf16(acc[j]);
  }
}

// Partials of a head merged inside the attention kernel travel through
// device-coherent accesses (agent-scope relaxed atomics: stores written
// through to the level the chip's dies share, loads served from it), so the
// merge needs no whole-cache write-back or invalidation, which would stall
// every workgroup still streaming on the same die.
__device__ __forceinline__ void store_shared_level(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void load_shared_level(const float* p, float& x, float& y) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  x = __uint_as_float(static_cast<uint32_t>(v));
  y = __uint_as_float(static_cast<uint32_t>(v >> 32));
}

// One softmax state of two channels: running max, sum and numerators.
struct Partial {
  float m, l, o0, o1;
};

// The split partials of one head merged by the last of its splits to finish
// (outputs of element type E: bf16 bits or float).  Every split stores its
// partials with store_shared_level and waits until they are written; then one
// thread counts the split on the head's arrival counter.  The split that
// brings the count to nsplit reads every split's partials with
// load_shared_level, merges them and resets the counter for the next launch.
// Nothing waits on another workgroup: the other splits simply end.  Called by
// every thread of the workgroup after its partials are stored; the head and
// its split count are taken afresh from the grid position and the slot record
// (kept from before the key loop, they would take registers the loop needs).
//
// Bound by the latency of the shared level: a thread owns two channels of one
// query, and its splits' numerators, maxima and sums come as batches of
// 8-byte loads all in flight together (4 or 16 splits per round trip), merged
// by the thread itself with no exchange.  A thread with several items (more
// channel pairs than threads) takes 5 to 12 splits without the four loads past
// them (25 heads of 5,190 rows in 10 splits, G = 16: 27.6 -> 25.4 us).  Where the
// workgroup has more threads than the head has channel pairs, the splits are
// dealt to `parts` groups of threads, which merge in LDS in split order.
template <typename E, int NT>
__device__ void merge_if_last(const AttnLaunch& a, int G, int Hq, int Hkv) {
  __shared__ Partial s_part[NT];
  __shared__ int last;
  const int slot = blockIdx.z, g = blockIdx.y, head = slot * Hkv + g;
  const int nsplit = (a.meta[slot].len + 1 + a.split_keys - 1) / a.split_keys;
  // This thread's partial stores are written before the workgroup counts
  // itself: the wait is issued as an asm statement that clobbers memory, so
  // the compiler cannot move the stores (relaxed atomics) past it either.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int prev = __hip_atomic_fetch_add(a.arrivals + head, 1, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
    last = prev == nsplit - 1;
    if (last)
      __hip_atomic_store(a.arrivals + head, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!last) return;
  const int t = threadIdx.x;
  const float* ml = a.ws_ml + static_cast<int64_t>(head) * a.split_stride * G * 2;
  const float* po = a.ws_o + static_cast<int64_t>(head) * a.split_stride * G * kHeadDim;
  E* out = static_cast<E*>(a.out) + (static_cast<int64_t>(slot) * Hq + g * G) * kHeadDim;
  const int pairs = G * (kHeadDim / 2);
  const int parts = max(1, min(NT / pairs, (nsplit + 3) / 4));
  const int per = (nsplit + parts - 1) / parts;
  const auto gather_by = [&](auto batch, int item, int lo, int hi) {
    constexpr int kBatch = decltype(batch)::value;
    const int q = item / (kHeadDim / 2), c = 2 * (item % (kHeadDim / 2));
    Partial p{kNoScore, 0.f, 0.f, 0.f};
    for (int s0 = lo; s0 < hi; s0 += kBatch) {
      float m[kBatch], l[kBatch], x[kBatch], y[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int row = min(s0 + j, hi - 1) * G + q;
        load_shared_level(ml + 2 * row, m[j], l[j]);
        load_shared_level(po + row * kHeadDim + c, x[j], y[j]);
      }
      float mx = p.m;
#pragma unroll
      for (int j = 0; j < kBatch; ++j) mx = fmaxf(mx, m[j]);
      const float keep = exp2f(p.m - mx);
      p.m = mx;
      p.l *= keep;
      p.o0 *= keep;
      p.o1 *= keep;
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const float w = s0 + j < hi ? exp2f(m[j] - mx) : 0.f;
        p.l += w * l[j];
        p.o0 += w * x[j];
        p.o1 += w * y[j];
      }
    }
    return p;
  };
  const auto gather = [&](int item, int lo, int hi) {
    return hi - lo <= 4 ? gather_by(std::integral_constant<int, 4>{}, item, lo, hi)
                        : gather_by(std::integral_constant<int, 16>{}, item, lo, hi);
  };
  const auto put = [&](int item, const Partial& p) {
    const float inv = 1.f / p.l;
    if constexpr (sizeof(E) == 2) {
      *reinterpret_cast<uint32_t*>(out + 2 * item) =
          f32_to_bf16(p.o0 * inv) | static_cast<uint32_t>(f32_to_bf16(p.o1 * inv)) << 16;
    } else {
      *reinterpret_cast<float2*>(out + 2 * item) = make_float2(p.o0 * inv, p.o1 * inv);
    }
  };
  if (pairs > NT && nsplit > 4 && nsplit <= 12) {
    for (int item = t; item < pairs; item += NT)
      put(item, gather_by(std::integral_constant<int, 12>{}, item, 0, nsplit));
    return;
  }
  if (parts == 1) {
    for (int item = t; item < pairs; item += NT) put(item, gather(item, 0, nsplit));
    return;
  }
  const int part = t / pairs;
  if (part < parts && part * per < nsplit)
    s_part[t] = gather(t % pairs, part * per, min(part * per + per, nsplit));
  __syncthreads();
  if (t < pairs) {
    Partial p = s_part[t];
    for (int k = 1; k < parts && k * per < nsplit; ++k) {
      const Partial r = s_part[k * pairs + t];
      const float mx = fmaxf(p.m, r.m), wp = exp2f(p.m - mx), wr = exp2f(r.m - mx);
      p = Partial{mx, p.l * wp + r.l * wr, p.o0 * wp + r.o0 * wr, p.o1 * wp + r.o1 * wr};
    }
    put(t, p);
  }
}

// ---------------------------------------------------------------------------
// bf16, MFMA
// ---------------------------------------------------------------------------

struct BlockRegs {
  u32x4 k[2][4];  // [S tile][k-step]
  u32x4 v[8];     // [16-channel tile]
};

// Offsets (in elements) of this lane's operand loads within a 32-key block.
struct LaneMap {
  int krow[2];   // key row within the block for S tile 0 / 1
  int kcol;      // first channel of the lane's 16-byte chunk at k-step 0
  int vrow;      // first key row of the lane's value tile
  int vch;       // channel within each 16-channel tile
};

__device__ __forceinline__ LaneMap lane_map() {
  const int lane = threadIdx.x & 63, r = lane & 15, grp = lane >> 4;
  LaneMap m;
  m.krow[0] = 8 * (r >> 2) + (r & 3);
  m.krow[1] = 8 * (r >> 2) + 4 + (r & 3);
  m.kcol = 8 * grp;
  m.vrow = 8 * grp;
  m.vch = r;
  return m;
}

// Rows kb .. kb+31 from the key rows at Kr and the value tiles at Vr (the
// head's region; in the paged layout the block's page, with kb = 0).
__device__ __forceinline__ void load_block(BlockRegs& b, const uint16_t* Kr,
                                           const uint16_t* Vr, int kb,
                                           const LaneMap& lm) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint16_t* row = Kr + static_cast<int64_t>(kb + lm.krow[t]) * kHeadDim + lm.kcol;
#pragma unroll
    for (int s = 0; s < 4; ++s) b.k[t][s] = ld16(row + 32 * s);
  }
  const uint16_t* vt = Vr + static_cast<int64_t>(kb + lm.vrow) * kHeadDim + lm.vch * 8;
#pragma unroll
  for (int u = 0; u < 8; ++u) b.v[u] = ld16_stream(vt + 16 * 8 * u);
}

struct Softmax {
  float m;      // running max of the scaled scores (log2 units), per query
  float l;      // this lane's share of the running sum
  f32x4 acc[8]; // O^T tile u: channels 16u + 4*grp + i, query lane & 15
};

// One 32-key block.  `limit`: keys with index >= limit (block-relative) are
// masked out (32 for a full block); with MASKED, so are the keys whose bit is
// set in `dropped`.
template <bool MASKED = false>
__device__ __forceinline__ void compute_block(Softmax& st, const BlockRegs& b,
                                              const bf16x8 (&qop)[4],
                                              float scale_log2, int limit,
                                              uint32_t dropped = 0) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(b.k[0][s]), qop[s], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(b.k[1][s]), qop[s], s1, 0, 0, 0);
  }
  const int grp = (threadIdx.x & 63) >> 4;
  float x[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[i] = s0[i] * scale_log2;
    x[4 + i] = s1[i] * scale_log2;
  }
  if (limit < 32) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (8 * grp + e >= limit) x[e] = kNegInf;
  }
  if constexpr (MASKED) {
    if (dropped) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if ((dropped >> (8 * grp + e)) & 1u) x[e] = kNegInf;
    }
  }
  float bm = x[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) bm = fmaxf(bm, x[e]);
  bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
  bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
  const float mn = fmaxf(st.m, bm);
  const float alpha = exp2f(st.m - mn);
  // P = hi + lo, both bf16, so the weights keep ~16 significant bits through
  // the bf16 MFMA (the remainder of a bf16 rounding is exact in fp32)
  bf16x8 p_hi, p_lo;
  float psum = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float pf = exp2f(x[e] - mn);
    const __bf16 hi = static_cast<__bf16>(pf);
    p_hi[e] = hi;
    p_lo[e] = static_cast<__bf16>(pf - static_cast<float>(hi));
    psum += pf;
  }
  st.l = st.l * alpha + psum;
  st.m = mn;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    st.acc[u] *= alpha;
    st.acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(b.v[u]), p_hi, st.acc[u], 0, 0, 0);
    st.acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(b.v[u]), p_lo, st.acc[u], 0, 0, 0);
  }
}

// The W wavefronts of a work item merge their states in LDS; an item that is
// a whole head writes the normalised output, another one its partial (merged
// by the head's last item, or with FUSED false by combine_kernel).
template <typename E, int W, bool FUSED>
__device__ __forceinline__ void finish_item(const AttnLaunch& a, const Work& w, int wave,
                                            int qi, int grp, const Softmax& st, int G, int Hq, int Hkv,
                                            float (&s_m)[W][kMaxGroup],
                                            float (&s_l)[W][kMaxGroup],
                                            float (&s_o)[W][kMaxGroup][kHeadDim]) {
  const int head = w.slot * Hkv + w.g;
  const int64_t item = static_cast<int64_t>(head) * a.split_stride + w.split;
  E* out = static_cast<E*>(a.out);
  // merge the W wavefronts in LDS
  if (qi < G) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      *reinterpret_cast<f32x4*>(&s_o[wave][qi][16 * u + 4 * grp]) = st.acc[u];
    if (grp == 0) {
      s_m[wave][qi] = st.m;
      s_l[wave][qi] = st.l;
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * kHeadDim; idx += 64 * W) {
    const int q = idx / kHeadDim, c = idx % kHeadDim;
    float mx = kNegInf;
#pragma unroll
    for (int v = 0; v < W; ++v) mx = fmaxf(mx, s_m[v][q]);
    float lsum = 0.f, o = 0.f;
#pragma unroll
    for (int v = 0; v < W; ++v) {
      const float sc = exp2f(s_m[v][q] - mx);
      lsum += s_l[v][q] * sc;
      o += s_o[v][q][c] * sc;
    }
    if (w.nsplit == 1) {
      const int64_t idx_out = (static_cast<int64_t>(w.slot) * Hq + w.g * G + q) * kHeadDim + c;
      if constexpr (sizeof(E) == 2) out[idx_out] = f32_to_bf16(o / lsum);
      else out[idx_out] = o / lsum;
    } else if constexpr (FUSED) {
      store_shared_level(a.ws_o + (item * G + q) * kHeadDim + c, o);
      if (c == 0) {
        store_shared_level(a.ws_ml + (item * G + q) * 2, mx);
        store_shared_level(a.ws_ml + (item * G + q) * 2 + 1, lsum);
      }
    } else {
      a.ws_o[(item * G + q) * kHeadDim + c] = o;
      if (c == 0) {
        a.ws_ml[(item * G + q) * 2] = mx;
        a.ws_ml[(item * G + q) * 2 + 1] = lsum;
      }
    }
  }
  if constexpr (FUSED) {
    if (w.nsplit > 1) merge_if_last<E, 64 * W>(a, G, Hq, Hkv);
  }
}

// W wavefronts per workgroup share one (sequence, KV head, split) work item:
// wavefront v takes the v-th W-th of the split's keys, and the wavefronts
// merge their online-softmax states in LDS at the end.  When the
// head needs a single split, the workgroup writes the normalised output
// itself and no merge kernel runs.  MINW is the number of wavefronts per
// SIMD the build must allow (1 lets the accumulators live in the
// accumulation registers, 2 keeps each wavefront within 256 registers).
template <int W, int MINW, bool PAGED>
__global__ __launch_bounds__(64 * W, MINW) void attn_bf16_kernel(
    AttnLaunch a, Paging pg, int G, int Hq, int Hkv, float scale_log2) {
  constexpr int kNBuf = 2;   // register buffers (3 or 4 measured no faster)
  // heads of several splits merged by their last split (merge_if_last); the
  // contiguous 12-wavefront build has no registers to spare for it, and its
  // multi-split heads are merged by combine_kernel
  constexpr bool kFusedMerge = W != 12 || PAGED;
  __shared__ float s_m[W][kMaxGroup];
  __shared__ float s_l[W][kMaxGroup];
  __shared__ float s_o[W][kMaxGroup][kHeadDim];
  const Work w = locate(a.meta, a.layer, Hkv, a.split_keys, pg);
  if (!w.valid) return;
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63, qi = lane & 15, grp = lane >> 4;
  const LaneMap lm = lane_map();
  const uint16_t* kpool = static_cast<const uint16_t*>(a.kpool);
  const uint16_t* vpool = static_cast<const uint16_t*>(a.vpool);
  const uint16_t* Kr = kpool + w.rm.region * kHeadDim;
  const uint16_t* Vr = vpool + w.rm.region * kHeadDim;
  // key block kb (a multiple of 32): its 32 rows lie in one page of the paged
  // layout, found through the block table; contiguous layouts index the region
  auto load = [&](BlockRegs& b, int kb) {
    if constexpr (PAGED) {
      const int64_t br = pool_row<true>(w.rm, kb);
      load_block(b, kpool + br * kHeadDim, vpool + br * kHeadDim, 0, lm);
    } else {
      load_block(b, Kr, Vr, kb, lm);
    }
  };
  const uint16_t* kn = static_cast<const uint16_t*>(a.k_new) +
                       (static_cast<int64_t>(w.slot) * Hkv + w.g) * kHeadDim;
  const uint16_t* vn = static_cast<const uint16_t*>(a.v_new) +
                       (static_cast<int64_t>(w.slot) * Hkv + w.g) * kHeadDim;

  // Q^T operand: query qi of the group, channels 32*s + 8*grp + [0, 8) at
  // k-step s (the key operand uses the same channel order, so a row's four
  // lane groups read 64 contiguous bytes per load)
  bf16x8 qop[4];
  {
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) +
        (static_cast<int64_t>(w.slot) * Hq + w.g * G + qi) * kHeadDim + 8 * grp;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x4 z = {0u, 0u, 0u, 0u};
      qop[s] = as_bf16x8(qi < G ? ld16(qrow + 32 * s) : z);
    }
  }

  Softmax st;
  st.m = kNoScore;
  st.l = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u) st.acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};

  // this wavefront's keys: [k0, k1) within the split (a multiple of 32 long
  // except where it ends at the new key)
  const int kpw = a.split_keys / W;
  // the same in every lane of the wavefront; in the paged builds of up to 8
  // wavefronts, made scalar, so that block-table entries are scalar loads
  // and block bases scalar sums (the 12-wavefront build has no registers to
  // spare for it and looks the table up per lane)
  constexpr bool kScalarTable = PAGED && W <= 8;
  const int k0 = kScalarTable ? __builtin_amdgcn_readfirstlane(w.k0 + wave * kpw)
                              : w.k0 + wave * kpw;
  const int k1 = min(k0 + kpw, w.k1);
  const bool has = k0 < k1;
  const bool owns_last = has && k1 == w.n_keys;
  const int nfull = !has ? 0 : (owns_last ? (w.len - k0) / 32 : (k1 - k0) / 32);
  if (nfull > 0) {
    // register buffers in rotation; every prefetch is unconditional (clamped
    // to the last block, whose repeated loads hit in cache) and the loop body
    // has no conditional code, so the loads it issues are consumed by the
    // next iteration and the compiler can neither sink them nor make the wait
    // before a block's compute also wait for later blocks' loads
    const int last = nfull - 1;
    BlockRegs buf[kNBuf];
#pragma unroll
    for (int j = 0; j < kNBuf; ++j) load(buf[j], k0 + 32 * min(j, last));
    int i = 0;
    for (; i + kNBuf - 1 < nfull; i += kNBuf) {
#pragma unroll
      for (int j = 0; j < kNBuf; ++j) {
        compute_block(st, buf[j], qop, scale_log2, 32);
        load(buf[j], k0 + 32 * min(i + kNBuf + j, last));
      }
    }
#pragma unroll
    for (int j = 0; j < kNBuf - 1; ++j)
      if (i + j < nfull) compute_block(st, buf[j], qop, scale_log2, 32);
  }
  if (owns_last) {
    // tail block: cached rows below len, the new pair at len, masked above
    const int kb = k0 + 32 * nfull;
    const int limit = w.n_keys - kb;       // 1..32 valid keys
    // rows of this block below len lie in one page of the paged layout (only
    // rows below len are read from the pools: the page of row len may not be
    // in the table yet when len is a multiple of 32)
    const uint16_t* Kb = Kr + static_cast<int64_t>(kb) * kHeadDim;
    const uint16_t* Vb = Vr + static_cast<int64_t>(kb) * kHeadDim;
    if constexpr (PAGED) {
      const int64_t br = kb < w.len ? pool_row<true>(w.rm, kb) : 0;
      Kb = kpool + br * kHeadDim;
      Vb = vpool + br * kHeadDim;
    }
    BlockRegs b;
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int key = kb + lm.krow[t];
      const uint16_t* row = key < w.len ? Kb + lm.krow[t] * kHeadDim : kn;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        b.k[t][s] = key <= w.len ? ld16(row + lm.kcol + 32 * s) : z;
    }
    const int key0 = kb + lm.vrow;         // first key of this lane's tile
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int ch = 16 * u + lm.vch;
      u32x4 v = key0 < w.len ? ld16(Vb + lm.vrow * kHeadDim + ch * 8) : z;
      uint16_t e8[8];
      __builtin_memcpy(e8, &v, 16);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (key0 + e == w.len) e8[e] = vn[ch];
        else if (key0 + e > w.len) e8[e] = 0;
      }
      __builtin_memcpy(&v, e8, 16);
      b.v[u] = v;
    }
    compute_block(st, b, qop, scale_log2, limit);
  }

  // lane sums of the same query -> the wavefront's sum
  st.l += __shfl_xor(st.l, 16, 64);
  st.l += __shfl_xor(st.l, 32, 64);

  if (owns_last)
    append_row<uint16_t, PAGED>(w, a.meta, Hkv, static_cast<const uint16_t*>(a.k_new),
                         static_cast<const uint16_t*>(a.v_new),
                         static_cast<uint16_t*>(a.kpool),
                         static_cast<uint16_t*>(a.vpool), a.pos);

  finish_item<uint16_t, W, kFusedMerge>(a, w, wave, qi, grp, st, G, Hq, Hkv, s_m, s_l, s_o);
}

// A block of 32 rows for the short build, rows at or past len included: row
// len is the step's new pair, rows past it are read from some cached row and
// masked by the caller (keys) or replaced by zero in patch_values.  Every
// lane issues the same sixteen loads whatever the block holds.
__device__ __forceinline__ void load_block_any(BlockRegs& b, const uint16_t* Kb,
                                               const uint16_t* Vb, const uint16_t* kn, int kb,
                                               int len, const LaneMap& lm) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint16_t* row = (kb + lm.krow[t] < len ? Kb + lm.krow[t] * kHeadDim : kn) + lm.kcol;
#pragma unroll
    for (int s = 0; s < 4; ++s) b.k[t][s] = ld16(row + 32 * s);
  }
  // an 8-row tile with no row below len reads the block's first tile instead
  const uint16_t* vt = Vb + (kb + lm.vrow < len ? lm.vrow * kHeadDim : 0) + lm.vch * 8;
#pragma unroll
  for (int u = 0; u < 8; ++u) b.v[u] = ld16_stream(vt + 16 * 8 * u);
}

// The new value at row len, zeros above it (vn: the lane's channel of each
// 16-channel tile).
__device__ __forceinline__ void patch_values(BlockRegs& b, const uint16_t (&vn)[8], int kb,
                                             int len, const LaneMap& lm) {
  const int at = len - kb - lm.vrow;         // the new row within the lane's tile
  if (at < 8) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      uint16_t e8[8];
      __builtin_memcpy(e8, &b.v[u], 16);
#pragma unroll
      for (int e = 0; e < 8; ++e) e8[e] = e < at ? e8[e] : e == at ? vn[u] : uint16_t(0);
      __builtin_memcpy(&b.v[u], e8, 16);
    }
  }
}

// Decode attention where the launch is bound by latency, not by bytes: at
// most 64 keys per wavefront (see plan_for).  A wavefront issues the loads of
// all its keys, the step's new pair among them, before it uses any: one round
// trip to memory, where the streaming build takes one for its full blocks and
// another for the block of the new pair, and reads its last block again for
// every prefetch that runs out of blocks.
template <int W, bool PAGED>
__global__ __launch_bounds__(64 * W, 1) void attn_bf16_short_kernel(
    AttnLaunch a, Paging pg, int G, int Hq, int Hkv, float scale_log2) {
  __shared__ float s_m[W][kMaxGroup];
  __shared__ float s_l[W][kMaxGroup];
  __shared__ float s_o[W][kMaxGroup][kHeadDim];
  const Work w = locate(a.meta, a.layer, Hkv, a.split_keys, pg);
  if (!w.valid) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, qi = lane & 15, grp = lane >> 4;
  const LaneMap lm = lane_map();
  const uint16_t* kpool = static_cast<const uint16_t*>(a.kpool);
  const uint16_t* vpool = static_cast<const uint16_t*>(a.vpool);
  const int64_t new_row = (static_cast<int64_t>(w.slot) * Hkv + w.g) * kHeadDim;
  const uint16_t* kn = static_cast<const uint16_t*>(a.k_new) + new_row;
  const uint16_t* vn = static_cast<const uint16_t*>(a.v_new) + new_row;
  const int kpw = a.split_keys / W;            // 32 or 64
  const int k0 = w.k0 + wave * kpw;
  const int k1 = min(k0 + kpw, w.k1);
  const bool has = k0 < k1, two = k0 + 32 < k1;
  const bool owns_last = has && k1 == w.n_keys;
  auto load = [&](BlockRegs& b, int kb) {
    // the block's first row; a block that starts at row len holds no cached
    // row and reads (and does not use) the pool's first rows
    const int64_t br = kb < w.len ? pool_row<PAGED>(w.rm, kb) : 0;
    load_block_any(b, kpool + br * kHeadDim, vpool + br * kHeadDim, kn, kb, w.len, lm);
  };

  Softmax st;
  st.m = kNoScore;
  st.l = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u) st.acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (has) {
    bf16x8 qop[4];
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) +
        (static_cast<int64_t>(w.slot) * Hq + w.g * G + (qi < G ? qi : 0)) * kHeadDim + 8 * grp;
    uint16_t vnew[8];
    if (owns_last) {
#pragma unroll
      for (int u = 0; u < 8; ++u) vnew[u] = vn[16 * u + lm.vch];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x4 z = {0u, 0u, 0u, 0u};
      const u32x4 x = ld16(qrow + 32 * s);
      qop[s] = as_bf16x8(qi < G ? x : z);
    }
    BlockRegs b0;
    load(b0, k0);
    if (two) {
      BlockRegs b1;
      load(b1, k0 + 32);
      compute_block(st, b0, qop, scale_log2, 32);
      if (owns_last) patch_values(b1, vnew, k0 + 32, w.len, lm);
      compute_block(st, b1, qop, scale_log2, min(32, k1 - k0 - 32));
    } else {
      if (owns_last) patch_values(b0, vnew, k0, w.len, lm);
      compute_block(st, b0, qop, scale_log2, k1 - k0);
    }
    st.l += __shfl_xor(st.l, 16, 64);
    st.l += __shfl_xor(st.l, 32, 64);
  }
  finish_item<uint16_t, W, true>(a, w, wave, qi, grp, st, G, Hq, Hkv, s_m, s_l, s_o);
  if (owns_last)
    append_row<uint16_t, PAGED>(w, a.meta, Hkv, static_cast<const uint16_t*>(a.k_new),
                                static_cast<const uint16_t*>(a.v_new),
                                static_cast<uint16_t*>(a.kpool),
                                static_cast<uint16_t*>(a.vpool), a.pos);
}

// ---------------------------------------------------------------------------
// bf16, MFMA, moving the rows of a deferred eviction on the way
// ---------------------------------------------------------------------------

// The last block of a head's source rows, kb .. kb+31, reaching past the
// cached rows: it is loaded as a full block (rows past the region's end read
// its row 0, so every lane issues the same sixteen loads as for any block and
// the loads in flight stay countable) and, once the data has arrived, row
// n_rows becomes the step's new pair (staged in LDS: nk, nv) and the rows
// above it zero.
__device__ __forceinline__ void load_block_clamped(BlockRegs& b, const uint16_t* Kr,
                                                   const uint16_t* Vr, int kb, int n_rows,
                                                   const LaneMap& lm) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int key = kb + lm.krow[t];
    const uint16_t* row = Kr + static_cast<int64_t>(key < n_rows ? key : 0) * kHeadDim + lm.kcol;
#pragma unroll
    for (int s = 0; s < 4; ++s) b.k[t][s] = ld16(row + 32 * s);
  }
  const int key0 = kb + lm.vrow;                      // a tile's first row (8-aligned)
  const uint16_t* vt = Vr + static_cast<int64_t>(key0 < n_rows ? key0 : 0) * kHeadDim + lm.vch * 8;
#pragma unroll
  for (int u = 0; u < 8; ++u) b.v[u] = ld16_stream(vt + 16 * 8 * u);
}

__device__ __forceinline__ void patch_block_tail(BlockRegs& b, const uint16_t* nk,
                                                 const uint16_t* nv, int kb, int n_rows,
                                                 const LaneMap& lm) {
  const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int key = kb + lm.krow[t];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (key == n_rows) b.k[t][s] = *reinterpret_cast<const u32x4*>(nk + lm.kcol + 32 * s);
      else if (key > n_rows) b.k[t][s] = z;
    }
  }
  const int key0 = kb + lm.vrow;
  if (key0 + 8 > n_rows) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      uint16_t e8[8];
      __builtin_memcpy(e8, &b.v[u], 16);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (key0 + e == n_rows) e8[e] = nv[16 * u + lm.vch];
        else if (key0 + e > n_rows) e8[e] = 0;
      }
      __builtin_memcpy(&b.v[u], e8, 16);
    }
  }
}

// Decode attention for the step after a deferred eviction (contiguous
// chronological layout, bf16, one workgroup of W wavefronts per (sequence,
// KV head), the whole head).  A sequence whose event deferred its row moves
// (due == kDueMovePending) holds its key/value rows in the order before the
// event, rows [0, plan_len), and the event's drop slots; its positions are
// already compacted and len = plan_len - m.  Attention runs over the
// surviving rows and the step's new pair (the dropped rows are masked), and
// every surviving row j after the first drop moves down to its compacted
// slot j - #{drops below j}, so the rows end as a full event would leave
// them, without reading them a second time.  The blocks are dealt in rounds,
// block r * W + v to wavefront v; every wavefront's loads of a round have
// returned (the round's softmax consumed them) before the barrier that
// precedes the round's moves.  A row moves only down, into a block of its
// own round or of an earlier one, which was read before that barrier, and
// no round reads a row that an earlier round wrote; the next round's loads,
// issued before the barrier, read only rows above every destination of the
// round, except that loads of blocks past the last key, and of tail rows
// past the cached ones, read the region's row 0 (which a round may be
// writing when the prompt is empty): those values are never used, being
// replaced by the new pair or zero, or belonging to no block.  The new pair
// is stored at len after the last round.  Sequences with nothing to move
// take the same path without moves.
template <int W>
__global__ __launch_bounds__(64 * W, 1) void attn_bf16_move_kernel(
    AttnLaunch a, int L, int G, int Hq, int Hkv, float scale_log2) {
  __shared__ float s_m[W][kMaxGroup];
  __shared__ float s_l[W][kMaxGroup];
  __shared__ float s_o[W][kMaxGroup][kHeadDim];
  __shared__ int s_drop[kMaxEvery];
  // a round's surviving value rows in destination order, per channel, offset
  // by the round's first destination row mod 8 so that destination tiles
  // start on 16-byte boundaries
  constexpr int kStage = W * 32 + 16;
  __shared__ __align__(16) uint16_t s_v[kHeadDim][kStage];
  __shared__ __align__(16) uint16_t s_new[2][kHeadDim];  // the step's key, value
  const int g = blockIdx.y, slot = blockIdx.z;
  const SeqMeta& M = a.meta[slot];
  if (!M.active) return;
  const bool moving = M.due == kDueMovePending;
  const int len = M.len;                              // rows once compacted
  const int n_rows = moving ? M.plan_len : len;       // rows in the region now
  const int m = min(n_rows - len, kMaxEvery);        // <= evict_every (host)
  const int lg = a.layer * Hkv + g;
  const int64_t region = M.base + static_cast<int64_t>(lg) * M.cap;
  // wavefront-uniform (the block indices and the drop scans below are scalar)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, qi = lane & 15, grp = lane >> 4;
  if (moving) {
    const int32_t* d = a.drops + (static_cast<int64_t>(slot) * L * Hkv + lg) * a.drop_stride;
    for (int k = threadIdx.x; k < min(m, kMaxEvery); k += 64 * W) s_drop[k] = d[k];
  }
  {
    const uint16_t* src = threadIdx.x < kHeadDim ? static_cast<const uint16_t*>(a.k_new)
                                                 : static_cast<const uint16_t*>(a.v_new);
    if (threadIdx.x < 2 * kHeadDim)
      (&s_new[0][0])[threadIdx.x] =
          src[(static_cast<int64_t>(slot) * Hkv + g) * kHeadDim + (threadIdx.x & (kHeadDim - 1))];
  }
  __syncthreads();
  const LaneMap lm = lane_map();
  uint16_t* kpool = static_cast<uint16_t*>(a.kpool);
  uint16_t* vpool = static_cast<uint16_t*>(a.vpool);
  const uint16_t* Kr = kpool + region * kHeadDim;
  const uint16_t* Vr = vpool + region * kHeadDim;

  bf16x8 qop[4];
  {
    const uint16_t* qrow = static_cast<const uint16_t*>(a.q) +
        (static_cast<int64_t>(slot) * Hq + g * G + qi) * kHeadDim + 8 * grp;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const u32x4 z = {0u, 0u, 0u, 0u};
      qop[s] = as_bf16x8(qi < G ? ld16(qrow + 32 * s) : z);
    }
  }
  Softmax st;
  st.m = kNoScore;
  st.l = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u) st.acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int n_keys = n_rows + 1;                      // the region's rows + the new pair
  const int nblk = (n_keys + 31) / 32;
  const int rounds = (nblk + W - 1) / W;
  auto load = [&](BlockRegs& b, int blk) {
    const int kb = blk * 32;
    if (kb + 32 <= n_rows) load_block(b, Kr, Vr, kb, lm);
    else load_block_clamped(b, Kr, Vr, kb, n_rows, lm);
  };
  // two register buffers, each named (an array indexed by the round's parity
  // would live in scratch memory): the loop below runs two rounds per pass
  // every round issues its sixteen prefetch loads, also for blocks past the
  // last key (they read the region's row 0 and are never used): with a fixed
  // count of loads after each block's, the wait for a block leaves the next
  // block's loads in flight
  BlockRegs buf0, buf1;
  load(buf0, wave);
  int di = 0;                 // drops below the current block (wavefront-uniform)
  auto round = [&](int r, BlockRegs& cur, BlockRegs& nxt) {
    const int blk = r * W + wave;
    const int kb = blk * 32;
    const bool have = blk < nblk;
    load(nxt, blk + W);
    uint32_t dropped = 0;
    if (have) {
      if (kb + 32 > n_rows) patch_block_tail(cur, s_new[0], s_new[1], kb, n_rows, lm);
      while (di < m && s_drop[di] < kb) ++di;
      for (int k = di; k < m && s_drop[k] < kb + 32; ++k) dropped |= 1u << (s_drop[k] - kb);
      compute_block<true>(st, cur, qop, scale_log2, min(32, n_keys - kb), dropped);
    }
    __syncthreads();          // every load of the round has been consumed
    if (moving && have) {
      const BlockRegs& b = cur;
      // key rows: this lane's two rows, four 16-byte chunks each
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int rr = lm.krow[t], j = kb + rr;
        if (j < n_rows && !((dropped >> rr) & 1u)) {
          const int dst = j - di - __popc(__builtin_amdgcn_ubfe(dropped, 0, rr));
          if (dst != j) {
            uint16_t* row = kpool + (region + dst) * kHeadDim + lm.kcol;
#pragma unroll
            for (int s = 0; s < 4; ++s) *reinterpret_cast<u32x4*>(row + 32 * s) = b.k[t][s];
          }
        }
      }
    }
    if (moving) {
      // values: the round's survivors go to LDS in destination order, then the
      // workgroup writes whole destination tiles (16 bytes per channel); only
      // the round's first and last tiles, shared with the neighbouring rounds,
      // are written element by element
      const int r0 = r * W * 32;                                 // round's first source row
      int fr = 0;                                                // drops below r0
      while (fr < m && s_drop[fr] < r0) ++fr;
      const int r1 = min(r0 + W * 32, n_rows);                   // round's source rows [r0, r1)
      int fe = fr;
      while (fe < m && s_drop[fe] < r1) ++fe;
      const int d_lo = r0 - fr, d_hi = r1 - fe;                  // destinations [d_lo, d_hi)
      const int off = d_lo & 7;
      if (have && kb < n_rows) {
        const BlockRegs& b = cur;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int rr = lm.vrow + e, j = kb + rr;
          if (j < n_rows && !((dropped >> rr) & 1u)) {
            const int dst = j - di - __popc(__builtin_amdgcn_ubfe(dropped, 0, rr));
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              uint16_t e8[8];
              __builtin_memcpy(e8, &b.v[u], 16);
              s_v[16 * u + lm.vch][off + dst - d_lo] = e8[e];
            }
          }
        }
      }
      __syncthreads();
      if (d_hi > d_lo && r1 > s_drop[0]) {
        const int t_lo = d_lo >> 3, t_hi = (d_hi - 1) >> 3;       // destination tiles
        const int items = (t_hi - t_lo + 1) * kHeadDim;
        for (int it = threadIdx.x; it < items; it += 64 * W) {
          const int tile = t_lo + it / kHeadDim, ch = it % kHeadDim;
          const int lo = max(tile * 8, d_lo), hi = min(tile * 8 + 8, d_hi);
          const int64_t row0 = region + tile * 8;                // 8-aligned (region is)
          uint16_t* dstp = vpool + row0 * kHeadDim + ch * 8;
          const uint16_t* src = &s_v[ch][off + tile * 8 - d_lo];
          if (lo == tile * 8 && hi == tile * 8 + 8) {
            *reinterpret_cast<u32x4*>(dstp) = *reinterpret_cast<const u32x4*>(src);
          } else {
            for (int x = lo; x < hi; ++x) dstp[x - tile * 8] = src[x - tile * 8];
          }
        }
      }
    }
  };
  for (int r = 0; r < rounds; r += 2) {
    round(r, buf0, buf1);
    if (r + 1 < rounds) round(r + 1, buf1, buf0);
  }
  st.l += __shfl_xor(st.l, 16, 64);
  st.l += __shfl_xor(st.l, 32, 64);
  // lane indices taken afresh (kept from before the rounds, they would be
  // spilled: the rounds hold every register)
  const int lane_e = __lane_id(), qe = lane_e & 15, ge = lane_e >> 4;
  const int tid = wave * 64 + lane_e;
  __syncthreads();            // every move is done: the new pair goes to row len
  if (wave == 0) {
    const int64_t row = region + len;
    for (int c = lane_e; c < kHeadDim; c += 64) {
      kpool[row * kHeadDim + c] = s_new[0][c];
      vpool[(row & ~int64_t(7)) * kHeadDim + c * 8 + (row & 7)] = s_new[1][c];
    }
    if (lane_e == 0) a.pos[row] = M.prompt_len + M.step;
  }

  // merge the W wavefronts in LDS and write the normalised output
  if (qe < G) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      *reinterpret_cast<f32x4*>(&s_o[wave][qe][16 * u + 4 * ge]) = st.acc[u];
    if (ge == 0) {
      s_m[wave][qe] = st.m;
      s_l[wave][qe] = st.l;
    }
  }
  __syncthreads();
  uint16_t* out = static_cast<uint16_t*>(a.out);
  for (int idx = tid; idx < G * kHeadDim; idx += 64 * W) {
    const int q = idx / kHeadDim, c = idx % kHeadDim;
    float mx = kNegInf;
#pragma unroll
    for (int v = 0; v < W; ++v) mx = fmaxf(mx, s_m[v][q]);
    float lsum = 0.f, o = 0.f;
#pragma unroll
    for (int v = 0; v < W; ++v) {
      const float sc = exp2f(s_m[v][q] - mx);
      lsum += s_l[v][q] * sc;
      o += s_o[v][q][c] * sc;
    }
    out[(static_cast<int64_t>(slot) * Hq + g * G + q) * kHeadDim + c] = f32_to_bf16(o / lsum);
  }
}

// ---------------------------------------------------------------------------
// fp32, MFMA
// ---------------------------------------------------------------------------

// A block of 16 keys in the operand registers of v_mfma_f32_16x16x4_f32
// (lane r = lane & 15, group = lane >> 4).
struct BlockF32 {
  f32x4 k[8];   // key row r, channels 16t + 4*group + [0, 4)
  f32x4 v[8];   // channel 16u + r, rows 4*group + [0, 4)
};

// The block whose `rows` first rows are cached (key rows at Kb, value tiles at
// Vb).  Rows past them read the block's first row or tile instead, so that
// every lane issues the same loads whatever the block holds.
__device__ __forceinline__ void load_block(BlockF32& b, const float* Kb, const float* Vb,
                                           int rows) {
  const int r = threadIdx.x & 15, grp = (threadIdx.x & 63) >> 4, tile = 8 * (grp >> 1);
  const int k = (r < rows ? r * kHeadDim : 0) + 4 * grp;
  const int v = (tile < rows ? tile * kHeadDim : 0) + r * 8 + 4 * (grp & 1);
#pragma unroll
  for (int t = 0; t < 8; ++t) b.k[t] = *reinterpret_cast<const f32x4*>(Kb + k + 16 * t);
#pragma unroll
  for (int u = 0; u < 8; ++u)
    b.v[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(Vb + v + 16 * 8 * u));
}

// One 16-key block at row kb.  S^T[key][query] = K . Q^T leaves each lane the
// scores of keys 4*group + i of query r, which is the P^T operand of
// O^T[channel][query] += V^T . P^T at key step i: no lane exchange but the
// two shuffles of the row maximum.  Keys at `limit` and above are masked.
__device__ __forceinline__ void compute_block(Softmax& st, const BlockF32& b,
                                              const f32x4 (&qop)[8], float scale_log2,
                                              int limit) {
  // four accumulators: short sums (and independent products)
  f32x4 sp[4] = {};
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      sp[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(b.k[t][i], qop[t][i], sp[i], 0, 0, 0);
  float x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    x[i] = ((sp[0][i] + sp[1][i]) + (sp[2][i] + sp[3][i])) * scale_log2;
  if (limit < 16) {
    const int grp = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * grp + i >= limit) x[i] = kNegInf;
  }
  float bm = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
  bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
  bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
  const float mn = fmaxf(st.m, bm);
  const float alpha = exp2f(st.m - mn);
  float p[4], psum = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = exp2f(x[i] - mn);
    psum += p[i];
  }
  st.l = st.l * alpha + psum;
  st.m = mn;
  // the block's own sum first, then one addition per block: the running sum
  // rounds once per 16 keys
#pragma unroll
  for (int u0 = 0; u0 < 8; u0 += 2) {
    f32x4 o[2] = {};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        o[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(b.v[u0 + u][i], p[i], o[u], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        st.acc[u0 + u][i] = fmaf(st.acc[u0 + u][i], alpha, o[u][i]);
  }
}

// fp32 decode attention: a workgroup of W wavefronts (four; one for many heads
// of few keys, see plan_f32) per (sequence, KV
// head, split), each streaming a W-th of the split's keys in 16-key blocks, two
// blocks in flight.  Bound by HBM where the rows are many and by latency where
// they are few; the group's queries are padded to 16, which the matrix cores
// still do in a third of the time the rows take to arrive (64 products of 32
// cycles per 16 KB block).  8 sequences of 8 heads, 2,900 rows: 40 us per
// launch (4.7 TB/s) where single wavefronts on the vector ALU, one key per
// lane, took 81 us (2.4 TB/s); 256 heads of 3,000 rows: 6.0 TB/s.
template <int W, bool PAGED>
__global__ __launch_bounds__(64 * W, 2) void attn_f32_kernel(AttnLaunch a, Paging pg, int G, int Hq,
                                                             int Hkv, float scale_log2) {
  __shared__ float s_m[W][kMaxGroup];
  __shared__ float s_l[W][kMaxGroup];
  __shared__ float s_o[W][kMaxGroup][kHeadDim];
  __shared__ __align__(16) float s_new[2][kHeadDim];   // the new pair, for its wavefront
  const Work w = locate(a.meta, a.layer, Hkv, a.split_keys, pg);
  if (!w.valid) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, qi = lane & 15, grp = lane >> 4;
  const float* kpool = static_cast<const float*>(a.kpool);
  const float* vpool = static_cast<const float*>(a.vpool);
  const int64_t new_row = (static_cast<int64_t>(w.slot) * Hkv + w.g) * kHeadDim;
  const int kpw = a.split_keys / W;            // a multiple of 16
  const int k0 = __builtin_amdgcn_readfirstlane(w.k0 + wave * kpw);
  const int k1 = min(k0 + kpw, w.k1);
  const bool has = k0 < k1;
  const bool owns_last = has && k1 == w.n_keys;
  auto load = [&](BlockF32& b, int kb) {
    // a block that starts at row len holds no cached row: it reads (and does
    // not use) the block before it
    const int64_t br = pool_row<PAGED>(w.rm, min(kb, max(0, w.len - 1) & ~15));
    load_block(b, kpool + br * kHeadDim, vpool + br * kHeadDim, w.len - kb);
  };

  Softmax st;
  st.m = kNoScore;
  st.l = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u) st.acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (has) {
    const float2 kn = reinterpret_cast<const float2*>(static_cast<const float*>(a.k_new) + new_row)[lane];
    const float2 vn = reinterpret_cast<const float2*>(static_cast<const float*>(a.v_new) + new_row)[lane];
    // Q^T operand: query qi, channels as the key rows' (zero past G)
    f32x4 qop[8];
    const float* qrow = static_cast<const float*>(a.q) +
        (static_cast<int64_t>(w.slot) * Hq + w.g * G + (qi < G ? qi : 0)) * kHeadDim + 4 * grp;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(qrow + 16 * t);
      qop[t] = qi < G ? x : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int last = (k1 - k0 - 1) / 16;       // blocks 0 .. last
    BlockF32 b0, b1;
    load(b0, k0);
    load(b1, k0 + 16 * min(1, last));
    if (owns_last) {
      reinterpret_cast<float2*>(s_new[0])[lane] = kn;
      reinterpret_cast<float2*>(s_new[1])[lane] = vn;
    }
    int i = 0;
    for (; i + 1 < last; i += 2) {
      // (the loads stay where they are: moved up among the products, they
      // would need registers of their own)
      compute_block(st, b0, qop, scale_log2, 16);
      __builtin_amdgcn_sched_barrier(0);
      load(b0, k0 + 16 * (i + 2));
      __builtin_amdgcn_sched_barrier(0);
      compute_block(st, b1, qop, scale_log2, 16);
      __builtin_amdgcn_sched_barrier(0);
      load(b1, k0 + 16 * min(i + 3, last));
      __builtin_amdgcn_sched_barrier(0);
    }
    if (i < last) {
      compute_block(st, b0, qop, scale_log2, 16);
      b0 = b1;
    }
    if (owns_last) {
      // row len takes the new pair, the values past it zero
      const int at_row = w.len - (k0 + 16 * last), at = at_row - 4 * grp;
      if (qi == at_row) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
          b0.k[t] = *reinterpret_cast<const f32x4*>(&s_new[0][16 * t + 4 * grp]);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) b0.v[u][e] = e < at ? b0.v[u][e] : e == at ? s_new[1][16 * u + qi] : 0.f;
    }
    compute_block(st, b0, qop, scale_log2, k1 - (k0 + 16 * last));
    st.l += __shfl_xor(st.l, 16, 64);
    st.l += __shfl_xor(st.l, 32, 64);
  }
  finish_item<float, W, true>(a, w, wave, qi, grp, st, G, Hq, Hkv, s_m, s_l, s_o);
  if (owns_last)
    append_row<float, PAGED>(w, a.meta, Hkv, static_cast<const float*>(a.k_new),
                             static_cast<const float*>(a.v_new), static_cast<float*>(a.kpool),
                             static_cast<float*>(a.vpool), a.pos);
}

template <bool PAGED>
hipError_t launch_attention_t(const Shape& sh, const AttnLaunch& a, hipStream_t s) {
  const dim3 grid(a.max_splits, sh.Hkv, a.max_seqs);
  // scores in log2 units: q.k / sqrt(d) * log2(e)
  const float scale_log2 = 1.4426950408889634f / sqrtf(static_cast<float>(kHeadDim));
  const dim3 cgrid(sh.Hkv, a.max_seqs);
  if (sh.dtype == 1 && a.move) {
    // one workgroup per head (max_splits == 1), rows of deferred events moved;
    // eight wavefronts (256 registers each: two per SIMD; a four-wavefront
    // build needs more than 256 and would run one per SIMD)
    const dim3 mgrid(1, sh.Hkv, a.max_seqs);
    hipLaunchKernelGGL((attn_bf16_move_kernel<8>), mgrid, dim3(512), 0, s, a, sh.L, sh.G,
                       sh.Hq, sh.Hkv, scale_log2);
  } else if (sh.dtype == 1) {
    if (a.short_runs && a.waves == 4)
      hipLaunchKernelGGL((attn_bf16_short_kernel<4, PAGED>), grid, dim3(256), 0, s, a, sh.pg,
                         sh.G, sh.Hq, sh.Hkv, scale_log2);
    else if (a.short_runs && a.waves == 8)
      hipLaunchKernelGGL((attn_bf16_short_kernel<8, PAGED>), grid, dim3(512), 0, s, a, sh.pg,
                         sh.G, sh.Hq, sh.Hkv, scale_log2);
    else if (a.waves == 12)
      hipLaunchKernelGGL((attn_bf16_kernel<12, 1, PAGED>), grid, dim3(768), 0, s, a, sh.pg,
                         sh.G, sh.Hq, sh.Hkv, scale_log2);
    else if (a.waves == 8)
      hipLaunchKernelGGL((attn_bf16_kernel<8, 1, PAGED>), grid, dim3(512), 0, s, a, sh.pg,
                         sh.G, sh.Hq, sh.Hkv, scale_log2);
    else if (a.waves == 4 && a.wide_regs)
      hipLaunchKernelGGL((attn_bf16_kernel<4, 1, PAGED>), grid, dim3(256), 0, s, a, sh.pg,
                         sh.G, sh.Hq, sh.Hkv, scale_log2);
    else if (a.waves == 4)
      hipLaunchKernelGGL((attn_bf16_kernel<4, 2, PAGED>), grid, dim3(256), 0, s, a, sh.pg,
                         sh.G, sh.Hq, sh.Hkv, scale_log2);
    else
      return hipErrorInvalidConfiguration;
    // a head with several splits is merged by its last split (merge_if_last),
    // except in the contiguous 12-wavefront build
    if (a.max_splits > 1 && a.waves == 12 && !PAGED)
      hipLaunchKernelGGL(combine_kernel, cgrid, dim3(256), 0, s, a, sh.G, sh.Hq, sh.Hkv);
  } else {
    if (a.waves == 4)
      hipLaunchKernelGGL((attn_f32_kernel<4, PAGED>), grid, dim3(256), 0, s, a, sh.pg, sh.G,
                         sh.Hq, sh.Hkv, scale_log2);
    else if (a.waves == 1)
      hipLaunchKernelGGL((attn_f32_kernel<1, PAGED>), grid, dim3(64), 0, s, a, sh.pg, sh.G,
                         sh.Hq, sh.Hkv, scale_log2);
    else
      return hipErrorInvalidConfiguration;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention(const Shape& sh, const AttnLaunch& a, hipStream_t s) {
  return sh.pg.tables ? launch_attention_t<true>(sh, a, s) : launch_attention_t<false>(sh, a, s);
}

// Partials of the allocation-free attention entry point.  Every GPU the
// library runs on holds its own copy until the process ends.  In host code
// `scratch` names a host-side stand-in, not device memory: host code uses
// only the address scratch_address returns.
static __device__ __align__(256) float scratch[kNoAllocScratchBytes / sizeof(float)];

hipError_t scratch_address(void** out) {
  static std::mutex mu;
  static void* addr[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

}  // namespace ra
