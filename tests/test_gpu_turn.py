"""GPU parity of a chunk of new rows on a filled cache (seg_attn_fwd with few rows and long
histories), where the library cuts the heads' prefixes into pieces and merges them: sequences of
different lengths in one call (so that heads have different numbers of pieces, one of them none),
prefixes that end on and off a piece, both head dimensions, a workspace of its own and the decode
path's.  The oracle is the judge."""
import numpy as np
import pytest

import workloads as W
from gpu_util import Cache, assert_parity, fill_cache_for_decode, full_history
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
