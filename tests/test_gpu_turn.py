"""GPU parity of a chunk of new rows on a filled cache (seg_attn_fwd with few rows and long
histories), where the library cuts the heads' prefixes into pieces and merges them: sequences of
different lengths in one call (so that heads have different numbers of pieces, one of them none),
prefixes that end on and off a piece, both head dimensions, a workspace of its own and the decode
path's.  Compared with the oracle.  Then the commit of such a chunk in one launch: rows and counters bit for
bit, and the decode step that reads them."""
import numpy as np
import pytest
import torch

import paper_2605_11744_amd as sa
import workloads as W
from gpu_util import Cache, assert_parity, dev_bf16, fill_cache_for_decode, full_history
from oracle import segattn_oracle as orc

pytestmark = pytest.mark.gpu

CASES = [
    # D, Hq, Hkv, policy, S, T, closed segments per sequence, open rows, new rows
    (128, 8, 2, (3, 1), 512, 64, (9, 1, 0), 100, 1),
    (128, 8, 2, (3, 1), 512, 64, (12, 2), 37, 65),
    (128, 8, 2, (2, 0), 1024, 0, (6,), 0, 33),
    (128, 16, 4, (1, 3, 2, 3), 256, 256, (17, 3), 5, 251),   # fills the segment; no workspace of its own
    (128, 4, 4, (3, 3, 1, 1), 512, 128, (11,), 64, 7),
    (64, 16, 4, (3, 1, 1, 2), 512, 128, (13, 4), 11, 40),
    (64, 4, 4, (1, 1, 3, 3), 512, 512, (8,), 300, 130),
    (128, 4, 1, (1,), 2048, 2048, (1,), 1500, 20),           # tail and open rows alone are long enough
    # few rows: pieces whose keys the waves of a workgroup share out (blocks of 8, 16 or 32 rows, the last one short)
    (128, 8, 2, (3, 1), 512, 64, (20, 1, 0), 100, 8),
    (128, 8, 2, (3, 1), 512, 64, (40, 3), 101, 9),
    (128, 4, 2, (3, 1), 512, 64, (24,), 31, 17),
    (128, 2, 2, (3, 2), 512, 0, (24,), 0, 33),
    (64, 8, 2, (3, 1), 512, 128, (20, 2), 5, 3),
    (64, 2, 2, (2, 1), 512, 128, (16,), 9, 31),              # no room for them: uncut
    (64, 2, 2, (2, 1), 512, 128, (40,), 9, 7),
    (64, 4, 2, (3, 1), 512, 128, (40, 2), 77, 9),
    # nothing to cut: a short chain, eight waves
    (64, 8, 2, (1, 1), 512, 128, (3,), 100, 40),
    # no room for pieces: one chain of up to 530 steps, sixteen waves (test_launch_forms.py), one, two or four heads a workgroup
    (64, 16, 4, (3, 1, 1, 1), 2048, 512, (8,), 11, 68),
    (64, 2, 2, (3, 1), 2048, 512, (4,), 11, 40),
    (64, 4, 2, (1, 3), 2048, 512, (4,), 1999, 33),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_chunk_on_a_filled_cache(case):
    D, Hq, Hkv, policy, S, T, closed, fill, m = CASES[case]
    B = len(closed)
    w = W.Workload(f"turn{case}", 700 + case, B, 0, Hq, Hkv, D, S, T, policy, decode=True,
                   max_context=S * (max(closed) + 1))
    k_done, c_fill = np.array(closed), np.full(B, fill + 1)
    _, ks, vs, _, _ = W.decode_inputs(w, k_done, c_fill)
    q = W.normal_bf16(w.seed, 0, B, m, Hq, D)
    k = W.normal_bf16(w.seed, 1, B, m, Hkv, D)
    v = W.normal_bf16(w.seed, 2, B, m, Hkv, D)
    c = Cache(w, past_capacity=w.max_context)
    try:
        fill_cache_for_decode(c, w, ks, vs, k_done, c_fill)  # declares fill open rows per sequence
        o, l = c.fwd(q, k, v)
        for b in range(B):
            n0 = closed[b] * S + fill
            kf, vf = full_history(ks[b], vs[b], n0 + 1, Hkv, D)
            kk = np.concatenate([kf[:n0], orc.widen(k[b])])[None]
            vv = np.concatenate([vf[:n0], orc.widen(v[b])])[None]
            qq = np.zeros((1, n0 + m, Hq, D))
            qq[0, n0:] = orc.widen(q[b])
            o_ref, l_ref = orc.attend(qq, kk, vv, seg_len=S, tail_len=T, kv_policy=policy,
                                      rows=np.arange(n0, n0 + m))
            assert_parity(o[b][None], l[b][None], o_ref, l_ref, fp32_check=False, what=f"case {case} sequence {b}")
    finally:
        c.close()


# One launch (up to 512 rows) with one to four workgroups per head, which count their arrivals at the
# head's counters; retrieved: the long-range heads' open rows are mirrored into their attention views.
COMMITS = [
    # D, Hq, Hkv, policy, S, T, closed segments per sequence, open rows, new rows, retrieval mode
    (128, 4, 2, (3, 1), 1024, 128, (3, 1), 611, 173, False),
    (128, 2, 2, (1, 2), 1024, 1024, (2, 1), 100, 400, False),
    (64, 4, 2, (2, 1), 2048, 64, (2, 0), 5, 512, False),
    (64, 4, 4, (0, 3, 1, 2), 512, 512, (1, 4), 17, 257, False),
    (128, 4, 4, (3, 1, 0, 2), 512, 128, (2, 1), 0, 512, False),  # whole segments: closed by the same launch
    (64, 2, 2, (2, 1), 300, 32, (1, 3), 0, 300, False),
    (128, 4, 2, (2, 1), 1024, 64, (3, 1), 0, 300, True),
    (64, 4, 2, (1, 2), 512, 0, (2, 1), 0, 512, True),
]


@pytest.mark.parametrize("case", range(len(COMMITS)))
def test_commit_of_a_chunk_leaves_rows_and_counters(case):
    D, Hq, Hkv, policy, S, T, closed, fill, m, retrieved = COMMITS[case]
    B = len(closed)
    w = W.Workload(f"commit{case}", 800 + case, B, 0, Hq, Hkv, D, S, T, policy, decode=True,
                   max_context=S * (max(closed) + 3))
    k_done, c_fill = np.array(closed), np.full(B, fill + 1)
    _, ks, vs, _, _ = W.decode_inputs(w, k_done, c_fill)
    k = W.normal_bf16(w.seed, 1, B, m, Hkv, D)
    v = W.normal_bf16(w.seed, 2, B, m, Hkv, D)
    c = Cache(w, past_capacity=w.max_context, retrieved_capacity=64 if retrieved else 0)
    try:
        fill_cache_for_decode(c, w, ks, vs, k_done, c_fill)
        want = [[[t.clone() for t in c.rows_view(b, h)] for h in range(Hkv)] for b in range(B)]
        kd, vd = dev_bf16(k), dev_bf16(v)
        sa.seg_kv_commit(c.ctx, kd, vd, m, c.stream)
        torch.cuda.synchronize()
        closes = fill + m == S
        counters = c.arena[:B * Hkv * 32].view(torch.int32).view(B, Hkv, 8).cpu().tolist()
        for b in range(B):
            for h, pol in enumerate(policy):
                pool = (closed[b] + closes) * S if pol & 2 else 0
                tail = T if closes else min(T, closed[b] * S)
                assert counters[b][h] == [pool, tail, 0 if closes else fill + m, 0, 0, 0, 0, 0], (b, h)
                skip = S - T if closes and not pol & 2 else 0
                at = closed[b] * S + fill if pol & 2 else 0 if closes else T + fill
                for have, exp, new in zip(c.rows_view(b, h), want[b][h], (kd, vd)):
                    exp[at:at + m - skip] = new[b, skip:, h]
                    assert torch.equal(have.view(torch.int16), exp.view(torch.int16)), (b, h)
        assert sa.seg_kv_lengths(c.ctx, B, Hkv)[2] == [0 if closes else fill + m] * B
        q1 = W.normal_bf16(w.seed, 3, B, 1, Hq, D)
        k1 = W.normal_bf16(w.seed, 4, B, 1, Hkv, D)
        v1 = W.normal_bf16(w.seed, 5, B, 1, Hkv, D)
        o, l = c.decode(q1[:, 0], k1[:, 0], v1[:, 0])
        seen = [0 if retrieved and pol & 2 else pol for pol in policy]  # no retrieved prefix: the own segment
        for b in range(B):
            n0 = closed[b] * S + fill
            kf, vf = full_history(ks[b], vs[b], n0 + 1, Hkv, D)
            kk = np.concatenate([kf[:n0], orc.widen(k[b]), orc.widen(k1[b])])[None]
            vv = np.concatenate([vf[:n0], orc.widen(v[b]), orc.widen(v1[b])])[None]
            qq = np.zeros((1, n0 + m + 1, Hq, D))
            qq[0, n0 + m:] = orc.widen(q1[b])
            o_ref, l_ref = orc.attend(qq, kk, vv, seg_len=S, tail_len=T, kv_policy=seen, rows=np.array([n0 + m]))
            assert_parity(o[b][None, None], l[b][None, :, None], o_ref, l_ref, fp32_check=False, what=f"case {case} sequence {b}")
    finally:
        c.close()
