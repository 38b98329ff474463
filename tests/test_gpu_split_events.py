"""Events of few heads: every head's rows moved by several workgroups.

Sequences on their own eviction phases, so that an event concerns one or two
of them; budgets whose moved rows are a little less, exactly and a little more
than a whole number of chunks (512 rows of bf16, 256 of fp32), or than the 1,152
(few drops) and 896 rows from which bf16 moves of small caches split, and drop
lists up to the longest that a chunk may have.  After every event the kept sets and
rows equal the oracle's, and the counters that order the moves are zero.
"""

import pytest
import torch

from gpu_harness import OracleSeq, Run, check_heads, log
from paper_2609_03430_amd import binding as B

pytestmark = pytest.mark.gpu

# (dtype, layout, layers, KV heads, K, r, every, prompts)
CASES = [
    (B.RA_BF16, B.RA_LAYOUT_CHRONOLOGICAL, 1, 2, 505, 0, 16, [3, 40]),
    (B.RA_BF16, B.RA_LAYOUT_CHRONOLOGICAL, 1, 2, 1140, 0, 16, [3, 40]),    # first event whole
    (B.RA_BF16, B.RA_LAYOUT_CHRONOLOGICAL, 1, 2, 850, 0, 50, [3, 40]),
    (B.RA_BF16, B.RA_LAYOUT_CHRONOLOGICAL, 2, 2, 1024, 64, 64, [0, 17, 130]),
    (B.RA_BF16, B.RA_LAYOUT_CHRONOLOGICAL, 1, 4, 9000, 64, 64, [7, 1000]),
    (B.RA_BF16, B.RA_LAYOUT_CHRONOLOGICAL, 1, 1, 1500, 20, 500, [9, 100]),
    (B.RA_BF16, B.RA_LAYOUT_PAGED, 2, 2, 1100, 64, 64, [5, 90, 300]),
    (B.RA_BF16, B.RA_LAYOUT_PAGED, 1, 2, 961, 0, 32, [31, 64]),
    (B.RA_BF16, B.RA_LAYOUT_PAGED, 1, 2, 960, 0, 64, [31, 64]),           # a third chunk for the alignment alone
    (B.RA_F32, B.RA_LAYOUT_CHRONOLOGICAL, 1, 2, 768, 8, 16, [1, 50]),
    (B.RA_F32, B.RA_LAYOUT_PAGED, 1, 2, 600, 64, 200, [10, 33]),
]


@pytest.mark.parametrize("dtype,layout,L,Hkv,K,r,every,lps", CASES)
def test_split_events(dtype, layout, L, Hkv, K, r, every, lps):
    log("split events dtype=%d layout=%d K=%d every=%d" % (dtype, layout, K, every))
    run = Run(L=L, Hq=Hkv, Hkv=Hkv, K=K, lps=lps, r=r, every=every, dtype=dtype, layout=layout,
              page_rows=32)
    oracles = [OracleSeq(run, s) for s in range(run.n)]
    for s in range(run.n):
        # up to a few steps before an event, each sequence on its own phase
        to = ((K + r) // every + 1 + s) * every - 2 - 3 * s
        B.ra_seq_fast_forward(run.h, s, to)
        oracles[s].advance(to)
        run.steps[s] = to
        run.materialise(s)
    events = 0
    for _ in range(3 * run.n):
        _, ev = run.step()
        for o in oracles:
            o.rep.append()
            o.rep.end_step()
        if ev:
            assert ev < run.n
            events += 1
            check_heads(run, oracles)
    assert events == run.n
    B.ra_evict_now(run.h, 0)
    torch.cuda.synchronize()
    n = -(-4 * run.max_seqs * Hkv // 256) * 256        # the counters: the metadata's tail
    assert int(run.cache.meta[-n:].count_nonzero()) == 0
    run.close()
