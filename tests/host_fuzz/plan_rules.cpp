// Prints the launches that the host library makes for given caches (test
// infrastructure): api.cpp with the stand-ins of stub_launchers.cpp.
//
// Usage: plan_rules DTYPE LAYOUT Q_HEADS KV_HEADS BUDGET RECENT EVERY FORWARD STEPS LEN...
// One layer; a sequence per LEN (its prompt), all fast-forwarded by FORWARD
// steps, then STEPS decode steps, one JSON line each.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include <hip/hip_runtime.h>

#include "ra_internal.h"
#include "randattn.h"

extern "C" void stub_configure(int64_t pool_rows, int64_t n_groups, int max_seqs, int page_rows);
extern ra::AttnLaunch g_attention;
extern int g_event_chunks;

#define CHECK(x)                                                          \
  do {                                                                    \
    const long long v_ = (x);                                             \
    if (v_ < 0) { std::fprintf(stderr, "%s: %lld\n", #x, v_); return 1; } \
  } while (0)

int main(int argc, char** argv) {
  if (argc < 11) return 2;
  const auto arg = [&](int i) { return std::atoi(argv[i]); };
  ra_config c{};
  c.num_layers = 1;
  c.dtype = arg(1);
  c.layout = arg(2);
  c.num_q_heads = arg(3);
  c.num_kv_heads = arg(4);
  c.head_dim = 128;
  c.budget_k = arg(5);
  c.recent_r = arg(6);
  c.evict_every = arg(7);
  c.budget_mode = RA_BUDGET_EVICTABLE;
  c.policy_block = 1;
  c.page_rows = 64;
  std::vector<int32_t> lens;
  for (int i = 10; i < argc; ++i) lens.push_back(arg(i));
  c.max_seqs = static_cast<int32_t>(lens.size());
  for (int32_t n : lens) c.max_prompt_len = std::max(c.max_prompt_len, n);
  const int64_t rows = (ra_required_slots(&c, lens.data(), c.max_seqs) + 31) / 32 * 32;
  CHECK(rows);
  const int64_t group = static_cast<int64_t>(c.num_kv_heads) * c.page_rows;
  stub_configure(rows, rows / group, c.max_seqs, c.page_rows);
  alignas(16) static char pool[16];      // the stand-ins touch no row
  std::vector<char> meta(ra_meta_bytes(&c) + 16);
  char* m = meta.data() + (16 - reinterpret_cast<uintptr_t>(meta.data()) % 16) % 16;
  ra_cache* cache = nullptr;
  CHECK(ra_cache_create(&c, pool, pool, reinterpret_cast<int32_t*>(pool), rows, m,
                        ra_meta_bytes(&c), nullptr, &cache));
  for (int i = 0; i < c.max_seqs; ++i)
    CHECK(ra_seq_begin(cache, i, lens[i], 1, i, nullptr, nullptr, nullptr));
  CHECK(ra_fast_forward(cache, arg(8), nullptr));
  const size_t q = static_cast<size_t>(c.max_seqs) * c.num_q_heads * ra::kHeadDim * 4;
  std::vector<char> in(q), out(q), ws(ra_workspace_bytes(&c));
  for (int t = 0; t < arg(9); ++t) {
    CHECK(ra_decode_attention(cache, 0, in.data(), in.data(), in.data(), out.data(), ws.data(),
                              ws.size(), nullptr));
    int32_t evicted = 0;
    CHECK(ra_end_step(cache, nullptr, &evicted));
    const ra::AttnLaunch& a = g_attention;
    ra_seq_info info;
    CHECK(ra_get_seq_info(cache, 0, &info));
    std::printf("{\"waves\":%d,\"wide\":%d,\"short\":%d,\"keys\":%d,\"splits\":%d,\"move\":%d,"
                "\"evicted\":%d,\"pending\":%d,\"len\":%d,\"chunks\":%d}\n",
                a.waves, a.wide_regs, a.short_runs, a.split_keys, a.max_splits, a.move, evicted,
                info.move_pending, info.len, g_event_chunks);
  }
  CHECK(ra_cache_destroy(cache));
  return 0;
}
