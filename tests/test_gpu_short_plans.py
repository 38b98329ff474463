"""Attention launches of few keys: single-wavefront work items, grouped.

Each case fixes the cached length by its prompts, so that the new row falls
first or last in a block, in an item, in a workgroup, or in a workgroup of its
own, for every geometry the plan picks for small launches; the partials of a
head number from none to many.  Two steps, every query head of every sequence
against the fp64 oracle, with the tolerances of the other attention tests.
"""

import pytest

from gpu_harness import OracleSeq, Run, attn_err, check_heads, log
from paper_2609_03430_amd import binding as B

pytestmark = pytest.mark.gpu

# (KV heads, group, prompts): cached rows per sequence before the first step
CASES = [
    (1, 1, [0]), (2, 5, [30, 31]), (8, 4, [31, 0, 63]),           # one workgroup per head
    (2, 2, [255]), (1, 16, [256, 129]), (4, 3, [511, 480, 1]),
    (8, 4, [512]), (2, 16, [639, 513, 128]), (8, 5, [1535, 1407, 0]),   # 4 x 32 keys
    (8, 1, [1536]), (1, 4, [2047, 2048]), (8, 8, [3135, 31]),           # 4 x 64 keys
    (4, 2, [4095, 4351, 700, 4223] * 4), (1, 2, [16500]),               # 8 x 64 keys
]


@pytest.mark.parametrize("layout", [B.RA_LAYOUT_CHRONOLOGICAL, B.RA_LAYOUT_PAGED])
@pytest.mark.parametrize("Hkv,G,lps", CASES)
def test_short_plan(Hkv, G, lps, layout):
    log("short plan Hkv=%d G=%d keys=%d layout=%d" % (Hkv, G, max(lps) + 1, layout))
    run = Run(L=1, Hq=Hkv * G, Hkv=Hkv, K=64, lps=lps, layout=layout, page_rows=32)
    run.cache.workspace.fill_(0xff)      # partials no launch wrote: NaN
    oracles = [OracleSeq(run, s) for s in range(run.n)]
    for t in range(2):
        outs, _ = run.step()
        outs = outs.float().cpu()
        for o in oracles:
            o.rep.append()
            attn_err(outs[0, o.slot], o.attend(0, t), B.RA_BF16, (t, o.slot))
            o.rep.end_step()
    check_heads(run, oracles)
    run.close()


# fp32, 16-key blocks: the new row at every kind of place, one wavefront with
# keys to many workgroups per head, an odd and an even number of blocks
F32_CASES = [(1, 1, [0]), (2, 5, [14, 15, 16, 17]), (2, 2, [31, 47, 48, 63]), (1, 16, [64, 65]),
             (8, 4, [511, 512, 300]), (2, 3, [1039, 1055]), (4, 8, [2047, 2030] * 16),
             (8, 2, [700, 32, 0] * 12), (8, 1, [130, 1025] * 50),
             (8, 3, [0, 15, 16, 17, 31, 32, 62] * 10), (8, 16, [64, 0] * 33)]   # one wavefront, four


@pytest.mark.parametrize("layout", [B.RA_LAYOUT_CHRONOLOGICAL, B.RA_LAYOUT_PAGED])
@pytest.mark.parametrize("Hkv,G,lps", F32_CASES)
def test_f32_plan(Hkv, G, lps, layout):
    log("f32 plan Hkv=%d G=%d keys=%d layout=%d" % (Hkv, G, max(lps) + 1, layout))
    run = Run(L=1, Hq=Hkv * G, Hkv=Hkv, K=64, lps=lps, dtype=B.RA_F32, layout=layout,
              page_rows=32)
    run.cache.workspace.fill_(0xff)
    oracles = [OracleSeq(run, s) for s in range(0, run.n, max(1, run.n // 4))]
    for t in range(2):
        outs, _ = run.step()
        outs = outs.cpu()
        for o in oracles:
            o.rep.append()
            attn_err(outs[0, o.slot], o.attend(0, t), B.RA_F32, (t, o.slot))
            o.rep.end_step()
    check_heads(run, oracles)
    run.close()
