"""Attention on both sides of 128 positions: scores of any magnitude give finite
contexts (the largest score's exponent is exactly 0), and a causal prompt's
first positions have the same bits whatever its length."""
import numpy as np
import pytest
import torch

import paper_2503_05130_amd as ie
import workloads as W
from oracle import forward as F
from tests.gpu_util import DEV, f64, instance_config, sync, to_dev
from tests.test_gpu_kernels import UBF, attn_inputs

pytestmark = pytest.mark.gpu


def context(q, k, v, causal):
    B, H, S, dh = q.shape
    vt = torch.zeros((B, H, dh, (S + 63) // 64 * 64), dtype=torch.bfloat16)
    vt[..., :S] = v.transpose(2, 3)
    ctx = torch.full((B, S, H * dh), float("nan"), dtype=torch.bfloat16, device=DEV)
    ie.test_attention(to_dev(q), to_dev(k), to_dev(vt), ctx, B, H, S, dh, causal)
    sync()
    return ctx


@pytest.mark.parametrize("scale", [2.0 ** 12, 2.0 ** 16, 2.0 ** 30])
@pytest.mark.parametrize("S,dh,causal", [(128, 64, False), (129, 64, False), (160, 64, True), (300, 128, False),
                                         (513, 128, True)])
def test_large_scores(S, dh, causal, scale):
    print(f"attention S={S} dh={dh} causal={causal} scale={scale}", flush=True)
    q, k, v = attn_inputs(2, 3, S, dh, seed=S + dh, scale=scale)
    got = f64(context(q, k, v, causal)).reshape(2, S, 3, dh).transpose(0, 2, 1, 3)
    assert np.all(np.isfinite(got))
    # such a softmax has all its weight on one key wherever the two largest scores are further apart than
    # their rounding: dh fp32 terms and the scale, at most (dh + 2) 2^-23 of the terms' magnitudes
    s = f64(q) @ f64(k).transpose(0, 1, 3, 2) / np.sqrt(dh)
    mag = np.abs(f64(q)) @ np.abs(f64(k)).transpose(0, 1, 3, 2) / np.sqrt(dh)
    if causal:
        s = np.where(np.tril(np.ones((S, S), bool)), s, -np.inf)
        mag = np.where(np.tril(np.ones((S, S), bool)), mag, 0.0)
    top = np.sort(np.concatenate([s, np.full(s.shape[:-1] + (1,), -np.inf)], -1), -1)
    sure = top[..., -1] - top[..., -2] > 2 * (dh + 2) * 2.0 ** -23 * mag.max(-1) + 40
    assert sure.mean() > 0.9
    want = np.take_along_axis(f64(v), s.argmax(-1)[..., None], 2)
    err = np.abs(got - want)
    assert np.all(err[sure] <= 2 * UBF * np.abs(f64(v)).max())


@pytest.mark.parametrize("S,dh", [(129, 64), (300, 64), (1000, 64), (300, 128)])
def test_causal_prefix_has_the_same_bits(S, dh):
    print(f"attention prefix S={S} dh={dh}", flush=True)
    q, k, v = attn_inputs(1, 9, S, dh, seed=S, scale=1.5)
    full = context(q, k, v, True)
    for n in (97, 128):
        part = context(q[:, :, :n].contiguous(), k[:, :, :n].contiguous(), v[:, :, :n].contiguous(), True)
        assert torch.equal(part[0].view(torch.int16), full[0, :n].view(torch.int16)), n


@pytest.mark.parametrize("size", [1e5, 1e6])
@pytest.mark.parametrize("seq", [128, 129, 256])
def test_post_ln_block_with_large_inputs(seq, size):
    """The first layer's Q and K are not normalised: scores grow with the input's square."""
    shape = W.model_shape("bert_base_l12_d768_s128", n_layers=1, n_out=0)
    x = W.make_input(71, 1, seq, 768).astype(np.float32) * np.float32(size)
    print(f"post-LN block seq={seq} inputs of {size}", flush=True)
    with ie.Instance(**instance_config(shape, 1, seq)) as inst:
        inst.submit(x)
        got = inst.read_logits()
    assert np.all(np.isfinite(got))
