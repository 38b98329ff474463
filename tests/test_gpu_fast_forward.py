"""Fast forwards over several events, in one launch per call, against the oracle.

The kernel keeps a head's generated positions in LDS, up to 9,216 of them, and a
key for each in registers, 2 to 8 on 512 threads or 5 to 9 on 1,024, by the most
rows that any sequence holds on the way; rows past the keys are among the most
recent, one to a thread.  Above that, for hole-fill and for several paged
sequences the events are launched one by one.  Every head
must hold the oracle's positions, and later decode steps and events must agree.
"""

import numpy as np
import pytest

from gpu_harness import OracleSeq, Run, log
from paper_2609_03430_amd import binding as B

pytestmark = pytest.mark.gpu

CHRON, PAGED = B.RA_LAYOUT_CHRONOLOGICAL, B.RA_LAYOUT_PAGED


def _check(run, oracles):
    for o in oracles:
        info = B.ra_get_seq_info(run.h, o.slot)
        for l in range(run.L):
            for g in range(run.Hkv):
                want = o.rep.P[(l, g)]
                got = run.positions(o.slot, l, g)
                assert info.len == len(want) and np.array_equal(got, want), (o.slot, l, g)


@pytest.mark.parametrize("K,lps,r,every,layout,policy,block", [
    (0, [0, 5], 0, 1, CHRON, B.RA_POLICY_RANDOM, 1),           # one row kept out of one
    (3, [7], 5, 3, PAGED, B.RA_POLICY_RANDOM, 1),
    (896, [130, 0, 33], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1),     # exactly 1,024 rows
    (897, [40], 64, 64, PAGED, B.RA_POLICY_RANDOM, 1),             # one more
    (2944, [9, 300], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1),        # 3,072
    (2945, [64], 64, 64, CHRON, B.RA_POLICY_SHARED, 1),
    (9088, [31], 64, 64, PAGED, B.RA_POLICY_RANDOM, 1),            # 9,216
    (9089, [31], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1),            # event by event
    # the builds full to their last recent row, and one row more
    (960, [130, 0], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1), (961, [33], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1),
    (1472, [5], 64, 64, PAGED, B.RA_POLICY_SHARED, 1), (1985, [77], 64, 64, CHRON, B.RA_POLICY_BLOCK, 3),
    (2496, [8], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1), (3009, [1], 64, 64, PAGED, B.RA_POLICY_RANDOM, 1),
    (3520, [64], 64, 64, CHRON, B.RA_POLICY_RECENCY, 1), (4032, [9], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1),
    (4033, [9], 64, 64, PAGED, B.RA_POLICY_RANDOM, 1), (5057, [2], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1),
    (6080, [40], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1), (7105, [3], 64, 64, CHRON, B.RA_POLICY_RANDOM, 1),
    (772, [20], 700, 64, CHRON, B.RA_POLICY_RANDOM, 1), (773, [20], 700, 64, CHRON, B.RA_POLICY_RANDOM, 1),
    (100, [12, 90], 16, 16, CHRON, B.RA_POLICY_BLOCK, 4),
    (100, [12, 90], 50, 16, CHRON, B.RA_POLICY_RECENCY, 1),
    (300, [50, 80], 33, 64, PAGED, B.RA_POLICY_RANDOM, 1),         # two paged sequences
])
def test_fast_forward_events(K, lps, r, every, layout, policy, block):
    log("fast forward events K=%d lps=%s layout=%d policy=%d" % (K, lps, layout, policy))
    run = Run(L=2, Hq=2, Hkv=2, K=K, lps=lps, r=r, every=every, layout=layout, policy=policy,
              block=block, seeds=[2**63 + 3 + i for i in range(len(lps))])
    oracles = [OracleSeq(run, s) for s in range(run.n)]
    first = -(-(K + r + 1) // every) * every
    # several events; from mid-period to mid-period; a slot on its own phase; one event
    for slot, n in [(None, first + 5 * every + every // 2), (None, 3 * every),
                    (0, 2 * every + 1), (None, 2 * every), (None, every)]:
        if slot is None:
            run.fast_forward(n)
        else:
            B.ra_seq_fast_forward(run.h, slot, n)
            run.steps[slot] += n
        for o in oracles:
            if slot is None or o.slot == slot:
                o.advance(n)
        _check(run, oracles)
    for s in range(run.n):
        run.materialise(s)
    for _ in range(every + 1):             # the slot records hold for the event that follows
        run.step()
        for o in oracles:
            o.rep.append()
            o.rep.end_step()
    _check(run, oracles)
    run.close()
