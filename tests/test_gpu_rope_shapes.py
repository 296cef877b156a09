"""GPU parity of seg_rope_apply over the shapes its workgroups divide up: fewer pieces of a row than threads
and more, numbers of heads that do not divide a workgroup, one row, rows that end inside a workgroup's
share or inside a sequence.  Every element against the textbook rotation in float64, half a bf16 ulp."""
import numpy as np
import pytest
import torch

import paper_2605_11744_amd as sa
from gpu_util import to_f64
from oracle import segattn_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hq,hkv", [(64, 1, 1), (64, 6, 3), (128, 5, 1), (128, 36, 4), (128, 96, 96)])
@pytest.mark.parametrize("B,rows", [(1, 1), (3, 17), (2, 700), (1, 16391)])
def test_rope_apply_shapes(D, hq, hkv, B, rows):
    if hq * B * rows > 600_000:
        rows = 600_000 // (hq * B)
    g = torch.Generator(device="cuda").manual_seed(7)
    x = [torch.randn((B, rows, h, D), generator=g, device="cuda").to(torch.bfloat16) for h in (hq, hkv)]
    before = [to_f64(t) for t in x]
    pos0 = [1000 * b for b in range(B)]
    cfg = sa.make_config(batch=B, n_q_heads=hq, n_kv_heads=hkv, head_dim=D, seg_len=64, tail_len=0, kv_policy=[1] * hkv,
                         rope_theta=10000.0)
    sa.seg_rope_apply(cfg, x[0], x[1], rows, torch.tensor(pos0, dtype=torch.int64, device="cuda"),
                      torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for t, ref in zip(x, before):
        for b in range(B):
            exact = orc.rope_rotate(ref[b], pos0[b] + np.arange(rows), 10000.0)
            err = np.abs(to_f64(t[b]) - exact)
            assert (err <= 2.0 ** -8 * np.abs(exact) + 1e-5).all(), (b, err.max())
