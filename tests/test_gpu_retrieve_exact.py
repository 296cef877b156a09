"""The retrieval operator's lists, exactly, where every score is a small whole number: keys with one nonzero
channel and constant queries, so that no summation order can move a score and ties are everywhere
(lower row first).  Windows that overlap, touch, nest at the clipped ends and are cut by R; every chunk size
of the scan; one anchor and the most there can be; hidden rows.  Oracle: the literal operator."""
import numpy as np
import pytest
import torch

import paper_2605_11744_amd as sa
import workloads as W
from gpu_util import Cache
from oracle import segattn_oracle as orc

pytestmark = pytest.mark.gpu


def _lists(w, pools, evict, params, R):
    """pools [B, n] whole-number scores of PAST head 0; returns idx [B, R]."""
    B, n = pools.shape
    c = Cache(w, past_capacity=n + w.seg_len)
    try:
        for b in range(B):
            kd, _ = c.rows_view(b, 0)
            kd[:n] = 0
            kd[:n, 5] = torch.from_numpy(pools[b].astype(np.float32)).cuda().to(torch.bfloat16)
        sa.seg_kv_set_lengths(c.ctx, [n] * B, [0] * B, [0] * B, c.stream)
        if evict:
            sa.seg_kv_past_evict(c.ctx, 0, evict, c.stream)
        g = w.n_q_heads // w.n_kv_heads
        q = torch.ones((B, 8, w.n_q_heads, w.head_dim), dtype=torch.bfloat16, device="cuda")
        r = sa.make_retrieval(**params)
        nws = sa.seg_kv_retrieve_workspace_bytes(c.ctx, r)
        ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
        idx = torch.full((B, 1, R), -1, dtype=torch.int32, device="cuda")
        sa.seg_kv_retrieve(c.ctx, r, q, 8, R, idx, ws, nws, c.stream)
        torch.cuda.synchronize()
        return idx.cpu().numpy()[:, 0], g
    finally:
        c.close()


def _expect(scores, evict, params, R, g, D):
    q = np.ones((8, g, D))
    k = np.zeros((scores.size, D))
    k[:, 5] = scores
    return orc.retrieve_indices(q, k, R=R, evicted=evict, **params)


@pytest.mark.parametrize("D,n,spread", [(128, 640, 3), (64, 1536, 1), (128, 5120, 100), (64, 8192, 4)])
@pytest.mark.parametrize("anchors,before,after,R,evict", [
    (16, 8, 23, 512, 0),
    (1, 0, 0, 1, 0),
    (32, 0, 0, 33, 7),
    (32, 40, 40, 300, 0),       # windows overlap everywhere, R cuts one of them
    (7, 3, 0, 640, 0),          # padding takes everything at the smallest size
    (5, 3000, 3000, 500, 111),  # windows longer than the pool, clipped at both ends
])
def test_lists_of_whole_number_scores(D, n, spread, anchors, before, after, R, evict):
    params = dict(n_queries=8, pool_window=4, tail_avg=4, n_anchors=anchors, win_before=before, win_after=after)
    w = W.small("rex", seq_len=0, seg_len=128, tail_len=0, n_q_heads=4, n_kv_heads=2, head_dim=D, kv_policy=[2, 0], batch=3)
    rng = np.random.default_rng(n + anchors)
    pools = rng.integers(-spread, spread + 1, size=(3, n))
    pools[1] = 0                                       # nothing but ties
    pools[2, n // 2:n // 2 + 60] += spread             # the best rows side by side
    R = min(R, n - evict)
    got, g = _lists(w, pools, evict, params, R)
    for b in range(3):
        assert list(got[b]) == list(_expect(pools[b], evict, params, R, g, D)), b


def test_lists_of_the_longest_pools():
    """Pools long enough for the largest chunks of the scan (4096 rows, over 3072 chunks)."""
    n, B, D = 1 << 20, 13, 64
    params = dict(n_queries=8, pool_window=8, tail_avg=1, n_anchors=32, win_before=5, win_after=10)
    w = W.small("rexl", seq_len=0, seg_len=4096, tail_len=0, n_q_heads=1, n_kv_heads=1, head_dim=D, kv_policy=[2], batch=B)
    rng = np.random.default_rng(3)
    pools = rng.integers(-120, 101, size=(B, n - 4096))
    pools[1] = 1
    pools[2, 700000:700100] = 110
    got, g = _lists(w, pools, 0, params, 512)
    for b in (0, 1, 2):
        s = pools[b]
        # the literal description (a million rows sorted in Python would take minutes in the oracle)
        order = np.lexsort((np.arange(s.size), -s))[:32]
        chosen, inside = [], set()
        for a in order:
            for r in range(max(0, a - 5), min(s.size, a + 11)):
                if len(chosen) < 512 and r not in inside:
                    inside.add(r)
                    chosen.append(r)
        r = 0
        while len(chosen) < 512:
            if r not in inside:
                inside.add(r)
                chosen.append(r)
            r += 1
        assert list(got[b]) == sorted(chosen), b
