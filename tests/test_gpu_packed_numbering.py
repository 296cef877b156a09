"""GPU parity of packed batches under both numberings of their items (row blocks there are, or every sequence
padded to the longest, whichever is fewer): sequences of one length, more than 64 of them (the search for
a block's sequence takes several steps), a long one among short ones; with the kernels for small
launches and, under item_queues = 3, with the general ones.  Compared with the oracle."""
import numpy as np
import pytest
import torch

import gpu_util
import paper_2605_11744_amd as sa
import workloads as W
from gpu_util import assert_parity, config_of, dev_bf16, to_f64
from oracle import segattn_oracle as orc
from test_gpu_backward import assert_grad_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("item_queues", [0, gpu_util.QUEUES_ON_SMALL_GRID])
@pytest.mark.parametrize("D,Hkv,g,S,T", [(64, 2, 4, 64, 16), (128, 2, 2, 100, 40)])
@pytest.mark.parametrize("lens", [(64,) * 40, (33,) * 70, (1,) * 3, (9, 10) * 65 + (400,), (500,) + (7, 0, 20) * 50],
                         ids=["40x64", "70x33", "3x1", "long_last", "long_first"])
def test_packed_batches(lens, D, Hkv, g, S, T, item_queues, monkeypatch):
    monkeypatch.setitem(gpu_util.TUNING, "item_queues", item_queues)
    total = sum(lens)
    w = W.small("pnum", index=940 + len(lens) % 50, seq_len=total, seg_len=S, tail_len=T, n_q_heads=Hkv * g, n_kv_heads=Hkv,
                head_dim=D, kv_policy=[3, 1])
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
    kw = dict(seg_len=S, tail_len=T, kv_policy=w.kv_policy)
    assert_parity(to_f64(out), to_f64(lse), *orc.attend_packed(q[0], k[0], v[0], cu, **kw), fp32_check=False, what=str(lens[:8]))
    ref = orc.attend_backward_packed(q[0], k[0], v[0], go[0], cu, **kw)
    assert_grad_parity((to_f64(dq), to_f64(dk), to_f64(dv)), ref, fp32_check=False, what=str(lens[:8]))
