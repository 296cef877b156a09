"""GPU parity of the forward pass at the sizes where the library shares a workgroup's keys out among its
waves (few query rows): lengths around the 32-key step, the 32-column block and the eight waves of a
workgroup (fewer key steps than waves, a last round of one), every number of query heads per
workgroup, segments that are no multiple of a block, packed batches with empty and one-token
sequences, bf16 and fp32 results.  Compared with the oracle."""
import numpy as np
import pytest
import torch

import paper_2605_11744_amd as sa
import workloads as W
from gpu_util import assert_parity, config_of, dev_bf16, fwd_seq, to_f64
from oracle import segattn_oracle as orc

pytestmark = pytest.mark.gpu

DENSE = [(n, S, T) for n, S, T in ((1, 64, 0), (31, 64, 64), (33, 32, 32), (65, 100, 33), (255, 512, 128), (257, 256, 100),
                                   (289, 32, 7), (530, 200, 200), (777, 1000, 0))]


@pytest.mark.parametrize("D,g", [(64, 1), (64, 4), (128, 1), (128, 2), (128, 3), (128, 8)])
@pytest.mark.parametrize("n,S,T", DENSE)
def test_short_prompts(n, S, T, D, g):
    w = W.small("ks", index=760 + n % 40, seq_len=n, seg_len=S, tail_len=min(T, S), n_q_heads=2 * g, n_kv_heads=2, head_dim=D,
                kv_policy=[1 if n % 2 else 0, 3 if g % 2 else 2], batch=2 if n < 300 else 1)
    q, k, v = W.prefill_inputs(w)
    o_ref, l_ref = orc.attend(q, k, v, seg_len=S, tail_len=w.tail_len, kv_policy=w.kv_policy)
    o, l = fwd_seq(w, q, k, v)
    assert_parity(o, l, o_ref, l_ref, fp32_check=False, what=f"n={n} S={S}")
    o, l = fwd_seq(w, q, k, v, out_fp32=False)
    assert np.abs(o - o_ref).max() <= 1e-2 + 2.0 ** -8 * np.abs(o_ref).max()  # bf16 results: half an ulp more


@pytest.mark.parametrize("D,g,S,T", [(64, 4, 64, 16), (64, 1, 100, 100), (128, 4, 96, 32), (128, 2, 33, 5), (128, 1, 512, 128)])
@pytest.mark.parametrize("lens", [(0, 1, 300, 0, 33, 64, 129, 0), (257,), (1,) * 70 + (200,), (31, 32, 33, 95, 96, 97)])
def test_packed_short_sequences(lens, D, g, S, T):
    total, Hkv = sum(lens), 2
    w = W.small("ksp", index=810 + len(lens), seq_len=total, seg_len=S, tail_len=T, n_q_heads=Hkv * g, n_kv_heads=Hkv,
                head_dim=D, kv_policy=[3, 1])
    q, k, v = W.prefill_inputs(w)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = torch.full((total, Hkv * g, D), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((Hkv * g, total), float("nan"), dtype=torch.float32, device="cuda")
    cud = torch.from_numpy(cu).cuda()
    sa.seg_attn_fwd_varlen(config_of(w, out_fp32=True, batch=len(lens)), dev_bf16(q[0]), dev_bf16(k[0]), dev_bf16(v[0]), cud,
                           total, max(lens), out, lse, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    o_ref, l_ref = orc.attend_packed(q[0], k[0], v[0], cu, seg_len=S, tail_len=T, kv_policy=w.kv_policy)
    assert_parity(to_f64(out), to_f64(lse), o_ref, l_ref, fp32_check=False, what=str(lens[:8]))


def test_reference_maximum_is_raised_late():
    """Scores that grow along the keys by more than the 2^8 a weight may reach: the reference maximum has to be
    raised again and again, in every wave at other steps."""
    n, D = 520, 128
    w = W.small("ksmax", index=840, seq_len=n, seg_len=n, tail_len=0, n_q_heads=2, n_kv_heads=1, head_dim=D, kv_policy=[0])
    q, k, v = W.prefill_inputs(w)
    q = W.f32_to_bf16_bits(np.ones((1, n, 2, D), dtype=np.float32))
    ramp = np.linspace(0.0, 40.0, n, dtype=np.float32)[None, :, None, None] / np.sqrt(D)
    k = W.f32_to_bf16_bits(np.broadcast_to(ramp, (1, n, 1, D)) + 0.01 * np.sign(orc.widen(k)).astype(np.float32))
    o_ref, l_ref = orc.attend(q, k, v, seg_len=n, tail_len=0, kv_policy=[0])
    o, l = fwd_seq(w, q, k, v)
    assert_parity(o, l, o_ref, l_ref, fp32_check=False, what="ramp")


LONG = [(3073, 4096, 512, 1), (3110, 4000, 0, 2), (4001, 2048, 2048, 1)]  # n, S, T, query heads of one KV head


@pytest.mark.parametrize("n,S,T,g", LONG)
def test_long_chains_of_few_heads(n, S, T, g):
    """Prompts of one KV head of 64 with 96 and more key steps in a row (sixteen waves share them out): a last row
    block of one row and a step of one key, a last round of the waves that most have no step in."""
    w = W.small("ksl", index=845 + n % 10, seq_len=n, seg_len=S, tail_len=T, n_q_heads=g, n_kv_heads=1, head_dim=64, kv_policy=[1])
    q, k, v = W.prefill_inputs(w)
    rows = np.unique(np.r_[0:70, 1500:1600, n - 130:n])
    o_ref, l_ref = orc.attend(q, k, v, seg_len=S, tail_len=T, kv_policy=[1], rows=rows)
    o, l = fwd_seq(w, q, k, v)
    assert np.isfinite(o).all() and np.isfinite(l).all()
    assert_parity(o[:, rows], l[:, :, rows], o_ref, l_ref, fp32_check=False, what=f"n={n}")
