"""Attention over rows whose scores are -inf: they weigh nothing.

Channel 0 of some cached keys is -inf and of every query positive, so the
softmax over the cached rows is the one over the other rows.  Such rows fill
the first block, a wavefront's whole run, whole work items and all of a head
but the step's new row, in every plan whose runs are short: few keys (bf16),
fp32, halved heads, and the merges of their partials.
"""

import numpy as np
import pytest
import torch

from gpu_harness import attn_err, log
from oracle.attention import softmax_attention
from paper_2609_03430_amd import binding as B

pytestmark = pytest.mark.gpu

CHRON, PAGED = B.RA_LAYOUT_CHRONOLOGICAL, B.RA_LAYOUT_PAGED


@pytest.mark.parametrize("dtype,n,Hkv,G,rows,layout", [
    (B.RA_BF16, 1, 8, 4, 200, CHRON),        # one workgroup per head
    (B.RA_BF16, 2, 4, 1, 500, PAGED),
    (B.RA_BF16, 1, 8, 4, 1090, CHRON),       # nine workgroups of 4 x 32 keys
    (B.RA_BF16, 1, 2, 16, 6300, PAGED),      # 4 x 64 keys, 25 partials per head
    (B.RA_BF16, 4, 8, 2, 5000, CHRON),       # 8 x 64 keys
    (B.RA_BF16, 25, 1, 16, 5190, CHRON),     # ten streamed items, several channel pairs a thread
    (B.RA_BF16, 1, 1, 16, 1450, PAGED),      # twelve of 4 x 32 keys, the same
    (B.RA_BF16, 33, 8, 2, 3100, CHRON),      # halved heads
    (B.RA_BF16, 1, 8, 4, 40000, CHRON),      # 12 wavefronts, merged by a kernel of its own
    (B.RA_F32, 1, 2, 2, 130, CHRON),
    (B.RA_F32, 2, 8, 4, 1100, PAGED),
    (B.RA_F32, 40, 8, 1, 900, CHRON),
    (B.RA_F32, 25, 1, 12, 9100, CHRON),      # ten items
    (B.RA_F32, 1, 1, 16, 9000, CHRON),
])
def test_rows_of_infinite_scores(dtype, n, Hkv, G, rows, layout):
    log("infinite scores dtype=%d n=%d Hkv=%d rows=%d layout=%d" % (dtype, n, Hkv, rows, layout))
    dt = torch.bfloat16 if dtype == B.RA_BF16 else torch.float32
    gen = torch.Generator().manual_seed(rows + n)
    cfg = B.make_config(1, Hkv * G, Hkv, 64, dtype=dtype, max_seqs=n, layout=layout, page_rows=32,
                        max_prompt_len=rows)
    for hidden in [(0, 16), (0, 32), (0, 64), (32, 96), (0, rows // 2), (rows // 2, rows - 1),
                   (0, rows - 1), (0, rows)]:
        cache = B.Cache(cfg, n * B.ra_seq_rows(cfg, rows))
        k = torch.randn(1, Hkv, rows, 128, generator=gen)
        v = torch.randn(1, Hkv, rows, 128, generator=gen)
        k[:, :, hidden[0]:hidden[1], 0] = -np.inf
        k, v = k.to(dt), v.to(dt)
        q = torch.randn(n, Hkv * G, 128, generator=gen)
        q[..., 0] = q[..., 0].abs() + 0.1
        q = q.to(dt)
        k_new, v_new = (torch.randn(n, Hkv, 128, generator=gen).to(dt) for _ in range(2))
        for s in range(n):
            B.ra_seq_begin(cache.handle, s, rows, 1, s, k.cuda(), v.cuda())
        cache.workspace.fill_(0xff)          # partials no launch wrote: NaN
        out = torch.zeros(n, Hkv * G, 128, dtype=dt, device="cuda")
        cache.decode(0, q.cuda(), k_new.cuda(), v_new.cuda(), out)
        out = out.float().cpu()
        seen = np.r_[0:hidden[0], hidden[1]:rows]
        for s in {0, n - 1}:
            for g in {0, Hkv - 1}:
                kd = torch.cat([k[0, g, seen], k_new[s, g:g + 1]]).double().numpy()
                vd = torch.cat([v[0, g, seen], v_new[s, g:g + 1]]).double().numpy()
                for h in {g * G, g * G + G - 1}:
                    want = softmax_attention(q[s, h].double().numpy(), kd, vd)
                    attn_err(out[s, h], want, dtype, (hidden, s, h))
        cache.close()
