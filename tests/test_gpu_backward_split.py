"""GPU parity of the backward pass at the sizes where the library shares a workgroup's steps out among its
waves (small windows), or dQ's and dK/dV's items share a launch: lengths around the 32-row step, fewer steps than waves,
every number of query heads per workgroup, carried tails that end inside a key block, segments that are no multiple of a
block, packed batches with empty and one-token sequences, and enough key blocks for the four-wave
dK/dV form.  Compared with the oracle; bars as in test_gpu_backward.py."""
import numpy as np
import pytest
import torch

import paper_2605_11744_amd as sa
import workloads as W
from gpu_util import config_of, dev_bf16, to_f64
from oracle import segattn_oracle as orc
from test_gpu_backward import assert_grad_parity, run_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,g", [(64, 1), (64, 2), (64, 4), (128, 1), (128, 3), (128, 4)])
@pytest.mark.parametrize("n,S,T", [(1, 64, 8), (33, 32, 32), (65, 40, 33), (255, 256, 0), (300, 128, 31), (411, 200, 100)])
def test_small_windows(n, S, T, D, g):
    w = W.small("bws", index=850 + n % 40, seq_len=n, seg_len=S, tail_len=T, n_q_heads=2 * g, n_kv_heads=2, head_dim=D,
                kv_policy=[1, 3 if n % 2 else 2], batch=2 if n < 100 else 1)
    q, k, v = W.prefill_inputs(w)
    go = W.grad_inputs(w)
    ref = orc.attend_backward(q, k, v, go, seg_len=S, tail_len=T, kv_policy=w.kv_policy)
    assert_grad_parity(run_backward(w, q, k, v, go, fp32_check=False), ref, fp32_check=False, what=f"n={n}")


@pytest.mark.parametrize("D,g", [(64, 8), (128, 2), (128, 8)])
@pytest.mark.parametrize("n,S,T", [(31, 64, 8), (129, 128, 128), (430, 200, 64)])
def test_windows_whose_gradients_share_a_launch(n, S, T, D, g):
    """Chains that are long against the work (groups of several heads, few keys): dQ and dK/dV items in one launch behind
    the row statistics; a last block of one row, a short last segment; the same bits twice."""
    w = W.small("bwb", index=930 + n % 40, seq_len=n, seg_len=S, tail_len=T, n_q_heads=g, n_kv_heads=1, head_dim=D,
                kv_policy=[3], batch=2)
    q, k, v = W.prefill_inputs(w)
    go = W.grad_inputs(w)
    ref = orc.attend_backward(q, k, v, go, seg_len=S, tail_len=T, kv_policy=w.kv_policy)
    a = run_backward(w, q, k, v, go, fp32_check=False)
    assert_grad_parity(a, ref, fp32_check=False, what=f"n={n}")
    b = run_backward(w, q, k, v, go, fp32_check=False)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))  # sums in a fixed order


@pytest.mark.parametrize("D,Hkv,g,S,T,lens", [
    (64, 2, 4, 64, 16, (0, 1, 150, 33, 0, 64, 129)),
    (128, 2, 2, 100, 100, (257, 3, 96)),
    (128, 2, 4, 96, 32, (1,) * 70 + (200,)),
    (64, 16, 1, 64, 16, (130, 31, 32, 33, 95, 96, 97, 200) * 2),   # over 640 key blocks: the four-wave form
    (64, 8, 1, 32, 7, (64,) * 60),
])
def test_packed_small_windows(D, Hkv, g, S, T, lens):
    run_packed(D, g, S, T, [(3, 1, 0, 2)[h % 4] for h in range(Hkv)], lens)


# Windows of several short segments whose two passes are launches of their own, the forms of each asked from the rules by
# test_launch_forms.py: dQ (split or not, query heads of a workgroup), waves of the split dK/dV form (0: the other one).
TWO_LAUNCHES = [
    # D, query heads of a KV head, S, T, policy, windows, rows: forms
    (64, 3, 200, 0, (0,), 1, 97, "split 8 1"),
    (64, 3, 48, 12, (3,), 1, 72, "split 4 1"),
    (64, 2, 200, 50, (1,), 1, 162, "split 8 2"),
    (64, 2, 200, 0, (3,), 1, 70, "split 4 2"),
    (64, 4, 128, 16, (2,), 1, 584, "split 8 4"),
    (64, 4, 32, 8, (2,), 1, 136, "split 4 4"),
    (64, 4, 97, 24, (2, 2, 0), 2, 591, "items 8 4"),
    (64, 4, 48, 6, (0, 0, 3), 2, 281, "items 4 4"),
    (128, 3, 32, 32, (2, 2), 1, 595, "split 4 1"),
    (128, 2, 32, 8, (2, 2), 1, 596, "split 4 2"),
    (128, 4, 32, 4, (2,), 2, 591, "split 4 4"),
    (128, 2, 48, 0, (0, 2), 2, 1612, "split 0 2"),
    (128, 2, 97, 24, (2, 3), 2, 777, "items 4 2"),
    (128, 4, 32, 4, (2, 3, 3), 2, 378, "items 4 4"),
]
TWO_LAUNCHES_PACKED = [  # the last: sequence lengths
    (64, 3, 200, 0, (0,), (122, 1, 0, 17, 1), "split 8 1"),
    (64, 2, 128, 16, (1,), (0, 73) + (0, 1) * 30, "split 4 2"),
    (64, 4, 97, 24, (3,), (1, 590) + (6,) * 15 + (1,), "split 8 4"),
    (64, 4, 32, 4, (2,), (144, 1, 1) + (0,) * 12, "split 4 4"),
    (128, 3, 32, 0, (3,), (1,) * 33 + (811,) + (3,) * 24, "split 4 1"),
    (128, 2, 32, 0, (2,), (4,) * 30 + (726,) + (5,) * 29, "split 4 2"),
    (128, 4, 32, 32, (2,), (9,) * 12 + (769,) + (9,) * 11, "split 4 4"),
]
ONE_LAUNCH_PACKED = [
    (64, 4, 64, 16, (3,), (150, 0, 33, 1, 64), "both 4 4"),
    (128, 3, 64, 16, (3,), (150, 0, 33, 1, 64), "both 4 1"),
    (128, 2, 96, 96, (1,), (97, 1, 200), "both 4 2"),
    (128, 4, 96, 32, (3,), (1,) * 20 + (193,), "both 4 4"),
]


@pytest.mark.parametrize("D,g,S,T,policy,B,n,forms", TWO_LAUNCHES)
def test_windows_of_two_launches(D, g, S, T, policy, B, n, forms):
    w = W.small("bwt", index=950 + n % 40, seq_len=n, seg_len=S, tail_len=T, n_q_heads=len(policy) * g, n_kv_heads=len(policy),
                head_dim=D, kv_policy=list(policy), batch=B)
    q, k, v = W.prefill_inputs(w)
    go = W.grad_inputs(w)
    ref = orc.attend_backward(q, k, v, go, seg_len=S, tail_len=T, kv_policy=w.kv_policy)
    assert_grad_parity(run_backward(w, q, k, v, go, fp32_check=False), ref, fp32_check=False, what=f"{forms} n={n}")


@pytest.mark.parametrize("D,g,S,T,policy,lens,forms", TWO_LAUNCHES_PACKED + ONE_LAUNCH_PACKED)
def test_packed_windows_of_known_forms(D, g, S, T, policy, lens, forms):
    run_packed(D, g, S, T, list(policy), lens)


def run_packed(D, g, S, T, policy, lens):
    total, Hkv = sum(lens), len(policy)
    w = W.small("bwsp", index=890 + len(lens) % 50, seq_len=total, seg_len=S, tail_len=T, n_q_heads=Hkv * g, n_kv_heads=Hkv,
                head_dim=D, kv_policy=policy)
    q, k, v = W.prefill_inputs(w)
    go = W.grad_inputs(w)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cfg = config_of(w, out_fp32=True, batch=len(lens))
    qd, kd, vd, gd, cud = dev_bf16(q[0]), dev_bf16(k[0]), dev_bf16(v[0]), dev_bf16(go[0]), torch.from_numpy(cu).cuda()
    nan = lambda *shape: torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    out, lse, dq, dk, dv = nan(total, Hkv * g, D), nan(Hkv * g, total), nan(total, Hkv * g, D), nan(total, Hkv, D), nan(total, Hkv, D)
    nws = sa.seg_attn_bwd_varlen_workspace_bytes(cfg, total)
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    sa.seg_attn_fwd_varlen(cfg, qd, kd, vd, cud, total, max(lens), out, lse, st)
    sa.seg_attn_bwd_varlen(cfg, qd, kd, vd, out, lse, gd, cud, total, max(lens), dq, dk, dv, ws, nws, st)
    torch.cuda.synchronize()
    ref = orc.attend_backward_packed(q[0], k[0], v[0], go[0], cu, seg_len=S, tail_len=T, kv_policy=w.kv_policy)
    assert_grad_parity((to_f64(dq), to_f64(dk), to_f64(dv)), ref, fp32_check=False, what=str(lens[:8]))
