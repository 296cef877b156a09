"""GPU parity of a decode step whose windows have many partial results to merge: more slices than the chip
holds workgroups (so that windows share them), with two or three, a dozen and dozens of partials in a
window, more than one batch of the merge kernel, a short sequence beside a long one.  Two tokens, so that the
second reads the first one's row and count.  Compared with the oracle."""
import numpy as np
import pytest

import workloads as W
from gpu_util import Cache, assert_parity, fill_cache_for_decode, full_history
from oracle import segattn_oracle as orc

pytestmark = pytest.mark.gpu

CASES = [
    # D, Hq, Hkv, policy, S, T, closed segments per sequence, open rows
    (64, 8, 8, (3,) * 8, 1024, 128, (60, 3), 700),              # about 60 partials in the longest windows
    (128, 16, 8, (3,) * 8, 1024, 1024, (12, 12, 11), 1),         # about 20
    (128, 8, 8, (3,) * 8, 1024, 256, (8, 7, 8, 8, 7), 513),      # a dozen
    (64, 12, 3, (3, 1, 2), 2048, 512, (90, 40), 31),             # windows of one slice beside long ones
    # few slices: numbered by the longest window, the shorter ones' last numbers empty
    (128, 8, 4, (1, 3, 0, 2), 1024, 256, (9, 1, 2), 77),
    (64, 4, 2, (1, 1), 2048, 512, (3, 1), 600),                  # no head with the past
    (128, 4, 2, (3, 3), 1024, 128, (5, 2), 511),                 # none without
    # every window cut by itself, but a slice searched for: numbers by the longest windows would be mostly empty
    (128, 16, 8, (3,) * 8, 1024, 128, (20, 2, 2), 77),
    (64, 12, 3, (3, 1, 2), 1024, 256, (80, 1, 0, 3), 300),
    (64, 8, 2, (3, 2), 1024, 256, (70, 3), 511),
]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_windows_of_many_partials(case, fp32):
    D, Hq, Hkv, policy, S, T, closed, fill = CASES[case]
    B = len(closed)
    w = W.Workload(f"partials{case}", 900 + case, B, 0, Hq, Hkv, D, S, T, policy, decode=True,
                   max_context=S * (max(closed) + 1))
    k_done, c_fill = np.array(closed), np.full(B, fill + 1)
    q, ks, vs, _, _ = W.decode_inputs(w, k_done, c_fill)
    c = Cache(w, past_capacity=w.max_context, fp32_check=fp32)
    try:
        k_new, v_new = fill_cache_for_decode(c, w, ks, vs, k_done, c_fill)
        hist = [full_history(ks[b], vs[b], closed[b] * S + fill + 1, Hkv, D) for b in range(B)]
        for token in range(2):
            o, l = c.decode(q, k_new, v_new)
            for b in range(B):
                if token:  # the same row again
                    hist[b] = tuple(np.concatenate([h, orc.widen(new[b])[None]]) for h, new in zip(hist[b], (k_new, v_new)))
                o_ref, l_ref = orc.decode_attend(q[b], *hist[b], seg_len=S, tail_len=T, kv_policy=policy)
                assert_parity(o[b], l[b], o_ref, l_ref, fp32_check=fp32, what=f"case {case} sequence {b} token {token}")
    finally:
        c.close()


@pytest.mark.parametrize("D,S,closed", [(128, 1024, 4), (64, 1024, 4), (128, 2048, 24)])
def test_not_a_number_in_a_whole_slice_reaches_the_output(D, S, closed):
    """Keys of one head are NaN in every fourth slice of 512 rows, so that one wave of the merge kernel holds
    nothing but partials without a maximum: that group's rows are NaN, the other group's are not."""
    policy, Hq, Hkv = (3, 2), 4, 2
    w = W.Workload("nan", 760 + D, 1, 0, Hq, Hkv, D, S, 64, policy, decode=True, max_context=S * (closed + 1))
    k_done, c_fill = np.array([closed]), np.array([33])
    q, ks, vs, _, _ = W.decode_inputs(w, k_done, c_fill)
    c = Cache(w, past_capacity=w.max_context)
    try:
        k_new, v_new = fill_cache_for_decode(c, w, ks, vs, k_done, c_fill)
        keys, _ = c.rows_view(0, 0)
        keys[:closed * S].view(-1, 4, 512, D)[:, 1] = float("nan")
        o, l = c.decode(q, k_new, v_new)
        assert np.isnan(o[0, :2]).all() and np.isnan(l[0, :2]).all()
        assert np.isfinite(o[0, 2:]).all() and np.isfinite(l[0, 2:]).all()
    finally:
        c.close()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("closed,fill", [(0, 0), (0, 1), (0, 31), (1, 0), (1, 32), (3, 95), (5, 512)])
def test_what_lies_in_the_newest_rows_place_does_not_count(D, closed, fill):
    """The split kernel takes the newest row from the caller; its place in the cache, and everything behind it,
    holds NaN.  Windows of one row, of a whole number of 32-row tiles and one more, and slices (of 512 rows)
    that hold nothing but the newest row."""
    policy, S, T = (3, 1, 2, 0), 1024, 64
    w = W.Workload("place", 770 + D + fill, 1, 0, 8, 4, D, S, T, policy, decode=True, max_context=S * (closed + 1))
    k_done, c_fill = np.array([closed]), np.array([fill + 1])
    q, ks, vs, _, _ = W.decode_inputs(w, k_done, c_fill)
    c = Cache(w, past_capacity=w.max_context)
    try:
        for h in range(4):
            for rows in c.rows_view(0, h):
                rows.fill_(float("nan"))
        k_new, v_new = fill_cache_for_decode(c, w, ks, vs, k_done, c_fill)
        o, l = c.decode(q, k_new, v_new)
        kf, vf = full_history(ks[0], vs[0], closed * S + fill + 1, 4, D)
        o_ref, l_ref = orc.decode_attend(q[0], kf, vf, seg_len=S, tail_len=T, kv_policy=policy)
        assert_parity(o[0], l[0], o_ref, l_ref, fp32_check=False, what=f"{closed} segments, {fill} rows")
    finally:
        c.close()
