"""Attention plans of 257 to 767 heads: long heads of about equal length are
halved up to 384 of them, long ragged ones of a contiguous layout take the build
for one wavefront per SIMD, the rest is whole.  Outputs, events and rows against
the oracle for the cases on both sides of each line."""

import numpy as np
import pytest
import torch

from gpu_harness import OracleSeq, Run, attn_err, check_heads, log
from paper_2609_03430_amd import binding as B

pytestmark = pytest.mark.gpu

CHRON, HOLE, PAGED = B.RA_LAYOUT_CHRONOLOGICAL, B.RA_LAYOUT_HOLE_FILL, B.RA_LAYOUT_PAGED


@pytest.mark.parametrize("n,Hkv,lo,hi,rows,layout,splits", [
    (33, 8, 20, 20, 3072, CHRON, 2),      # the event's moves ride a step of whole heads
    (33, 8, 20, 20, 3071, CHRON, 1),
    (65, 4, 0, 150, 3300, PAGED, 2),
    (48, 8, 31, 31, 3100, HOLE, 2),       # 384 heads
    (39, 10, 31, 31, 3100, CHRON, 1),     # 390
    (33, 8, 0, 1900, 3200, CHRON, 1),     # ragged
    (33, 8, 0, 1900, 3200, PAGED, 1),
])
def test_mid_plan(n, Hkv, lo, hi, rows, layout, splits):
    log("mid plan n=%d Hkv=%d rows=%d layout=%d" % (n, Hkv, rows, layout))
    r, every = 16, 16
    lps = [lo + (hi - lo) * (i % 7) // 6 for i in range(n)]
    K = rows - hi - r - every
    run = Run(L=1, Hq=Hkv * 5, Hkv=Hkv, K=K, lps=lps, r=r, every=every, layout=layout)
    picked = [0, 6, n // 2, n - 1]
    oracles = [OracleSeq(run, s, heads=[(0, g) for g in range(Hkv)]) for s in picked]
    steps = -(-(K + r + every) // every) * every - 1     # the longest cache: `rows` keys at most
    steps -= (hi + steps + 1) - rows if hi + steps + 1 > rows else 0
    run.fast_forward(steps)
    for o in oracles:
        o.advance(steps)
    for s in range(n):
        run.materialise(s)
    worst, seen = 0.0, False
    for t in range(every + 3):
        longest = max(B.ra_get_seq_info(run.h, s).len for s in range(n)) + 1
        if longest == rows:
            assert B.ra_attention_plan(run.h)[1] == splits
            seen = True
        outs, _ = run.step()
        outs = outs.float().cpu()
        for o in oracles:
            o.rep.append()
            worst = max(worst, attn_err(outs[0, o.slot], o.attend(0, o.rep.step - 1), B.RA_BF16,
                                        (t, o.slot)))
            o.rep.end_step()
    assert seen
    check_heads(run, oracles)
    log("  worst %.3g" % worst)
    run.close()


def test_whole_heads_where_halves_outgrow_the_no_alloc_array():
    """33 of 70 slots active: the halves' partials of 70 slots are over the
    array's 8 MiB, so the heads stay whole and the entry point accepts them."""
    n, Hkv, G, K = 70, 8, 16, 3200
    cfg = B.make_config(1, Hkv * G, Hkv, K, max_seqs=n)
    cache = B.Cache(cfg, n * B.ra_seq_rows(cfg, 8))
    for s in range(n):
        B.ra_seq_begin(cache.handle, s, 8, 1, s)
    for s in range(n - 33):
        B.ra_seq_end(cache.handle, s)
    B.ra_fast_forward(cache.handle, 3150)
    cache.k_pool.zero_()
    cache.v_pool.fill_(0.5)
    assert B.ra_attention_plan(cache.handle)[1] == 1
    q = torch.zeros(n, Hkv * G, 128, dtype=torch.bfloat16, device="cuda")
    kv = torch.full((n, Hkv, 128), 0.5, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros_like(q)
    cache.decode_noalloc(0, q, kv, kv, out)
    assert np.all(out[n - 33:].float().cpu().numpy() == 0.5)
    cache.close()
