"""Tile edges of the score-based evictors' kernels against their oracles.

The window scorer divides a head's 4 G query tiles and the keys of a block
between its wavefronts by G, with two rounds of query tiles above G = 8: the
groups below take every split between the ones other tests take.  More than 256 heads of a short cache take workgroups of 512 threads.
R-KV's similarities run over 512-row chunks against 128-column blocks, the chunks of a
head on one die of eight: several chunks, a ragged last column tile, and
near-duplicates inside a row's own tile, across tiles and across chunks.
"""

import numpy as np
import pytest
import torch

from gpu_harness import OracleSeq, Run, log
from oracle.scored import rkv_redundancy, rkv_scores
from paper_2609_03430_amd import binding as B
from test_gpu_window_score import _select_and_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [2, 3, 6, 9, 11, 13])
@pytest.mark.parametrize("K,steps", [(40, 128), (170, 300)])   # 128 and 161 rows (one block, and a part); 258 and 291
def test_window_query_groups(G, K, steps):
    log("window scorer G=%d K=%d" % (G, K))
    lps = [0, 33]
    run = Run(L=1, Hq=G, Hkv=1, K=K, lps=lps, r=63, every=64, policy=B.RA_POLICY_EXTERNAL)
    oracles = [OracleSeq(run, s) for s in range(run.n)]
    for t in range(min(steps, K + 63 + 25)):
        run.step()
        for o in oracles:
            o.rep.append()
    _select_and_check(run, oracles, min(steps, K + 63 + 25), stride=512)
    run.close()


@pytest.mark.parametrize("Hkv,G,K", [
    (129, 4, 40), (129, 1, 41), (129, 3, 1840), (129, 2, 1900), (129, 5, 60), (128, 2, 40)])
def test_window_many_heads(Hkv, G, K):
    """258 heads (512 threads; G = 5 not) and 256; 2,048 rows and fewer take 4 candidates
    per thread, more take 8."""
    log("window scorer Hkv=%d G=%d K=%d" % (Hkv, G, K))
    steps = K + 63 + 33
    run = Run(L=1, Hq=Hkv * G, Hkv=Hkv, K=K, lps=[90, 33], r=63, every=64,
              policy=B.RA_POLICY_EXTERNAL)
    run.fast_forward(steps)
    oracles = [OracleSeq(run, s, heads=[(0, g) for g in (0, Hkv // 2, Hkv - 1)])
               for s in range(run.n)]
    for s in range(run.n):
        run.materialise(s)
    for o in oracles:
        for _ in range(steps):
            o.rep.append()
    _select_and_check(run, oracles, steps, stride=2176)
    run.close()


@pytest.mark.parametrize("heads,keep,recent_dups", [(9, 1100, 2), (1, 429, 1), (3, 20, 0)])
def test_rkv_similarities(heads, keep, recent_dups):
    log("R-KV similarities heads=%d keep=%d" % (heads, keep))
    lp, r, every = 30, 64, 64
    steps = keep + r + 50
    n = lp + steps                      # 1,244, 573 or 164 rows: 50 to drop
    cfg = B.make_config(heads, 1, 1, keep, r, every, max_seqs=1,
                        policy=B.RA_POLICY_EXTERNAL)
    cache = B.Cache(cfg, B.ra_seq_rows(cfg, lp))
    B.ra_seq_begin(cache.handle, 0, lp, 3, 4)
    B.ra_seq_fast_forward(cache.handle, 0, steps)
    gen = torch.Generator().manual_seed(11 + heads)
    keys = torch.randn(heads, 1, n, 128, generator=gen)
    # near-duplicates (cosine about 0.95): rows 5, 7, 14 in one tile, others far apart
    for row, of in [(7, 5), (14, 5), (40, 20), (n - 2, 20), (n - 70, 21), (n // 2, 21), (60, 21)]:
        keys[:, :, row] = keys[:, :, of] + 0.3 * torch.randn(heads, 1, 128, generator=gen)
    keys = keys.to(torch.bfloat16)
    B.ra_write_rows(cache.handle, 0, keys.cuda(), torch.zeros_like(keys).cuda())
    window = torch.randn(1, heads, 1, 64, 128, generator=gen).to(torch.bfloat16).cuda()
    scratch = torch.empty(B.ra_scored_scratch_bytes(cfg, lp), dtype=torch.uint8, device="cuda")
    # lambda = 0: the score is the softmax of the redundancy alone
    params = B.make_scorer(B.RA_SCORER_RKV, rkv_lambda=0.0, rkv_threshold=0.9,
                           rkv_recent_dups=recent_dups)
    B.ra_scored_evict(cache.handle, 0, 1, params, window, scratch)
    for h in range(heads):
        got = B.ra_read_positions(cache.handle, 0, h, 0, n)
        drops = np.setdiff1d(np.arange(n), got)
        assert drops.shape[0] == 50
        cbar = rkv_redundancy(keys[h, 0].double().numpy(), np.arange(n), 0.9, recent_dups)
        s = rkv_scores(np.zeros(n), cbar, n - r, 0.0)
        # an fp32 sum of n similarities in 16 lanes, then the softmax in fp32
        tol = np.abs(s).max() * ((n / 16 + 16) * 2.0 ** -24)
        edge = np.sort(s)[49]
        kept = np.setdiff1d(np.arange(n - r), drops)
        assert drops.max() < n - r
        assert np.all(s[drops] <= edge + tol) and np.all(s[kept] >= edge - tol), h
    cache.close()
