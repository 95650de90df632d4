"""One training step at the shapes where the grouped weight gradients, the
batched transposes, the FFN-up product that keeps both its outputs and the
attention backward's 32-token blocks can go wrong: widths that only 64 divides,
an odd number of K tiles in either K order, sequences of one to four blocks with
and without a remainder.  Every gradient against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2503_05130_amd as ie
from oracle import train as T
from tests.gpu_util import instance_config
from tests.test_gpu_train import GRAD_REL_L2, LOSS_REL, SMALL, make_batch, oracle_tensors, rel_l2, shape_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,d,F,causal", [
    (64, 1, 128, 64, 0),      # one K tile, one token a sequence
    (2, 96, 128, 320, 0),     # three K tiles, three blocks
    (4, 112, 256, 192, 1),    # seven K tiles, four blocks with a remainder
    (1, 64, 384, 704, 0),
    (64, 3, 128, 1088, 1),
    (16, 128, 256, 320, 0),   # 2048 tokens: the even/odd order
    (66, 32, 128, 192, 1),    # 33 K tiles of it
])
def test_every_gradient(B, S, d, F, causal):
    shape = shape_of(dict(SMALL, n_layers=2 if B * S < 2048 else 1, d_model=d, n_heads=d // 64, d_ff=F, causal=causal))
    print(f"train step B={B} S={S} d={d} F={F} causal={causal}", flush=True)
    x, labels = make_batch(shape, B, S, 700 + S)
    params = T.initial_params(shape)
    loss_ref, grads_ref, _ = T.loss_and_grads(params, x, labels, shape)
    with ie.Trainer(**instance_config(shape, B, S)) as tr:
        tr.step(x, labels)
        assert abs(tr.loss() - loss_ref) <= LOSS_REL * abs(loss_ref)
        for layer, slot, name, ref in oracle_tensors(grads_ref, shape):
            if S == 1 and slot in (0, 1):   # one key: the softmax is constant, Q and K get no gradient
                ref = ref[..., 2 * d:]
                g = tr.export(layer, slot, ie.TRAIN_GRAD, (d, 3 * d) if slot == 0 else (3 * d,))
                assert np.all(np.abs(g[..., :2 * d]) <= 1e-6), name
                g = g[..., 2 * d:]
            else:
                g = tr.export(layer, slot, ie.TRAIN_GRAD, ref.shape)
            assert np.all(np.isfinite(g)), name
            assert rel_l2(g, ref) <= GRAD_REL_L2, (name, rel_l2(g, ref))


def test_trainer_memory_per_token():
    """The weight gradients' operands are transposed into activations that the layer's backward has read: a token
    takes 141.25 d bytes of a one-layer trainer's workspace and scratch (d_ff = 4 d, 64-wide heads, 128 positions: the forward's workspace 40 d, the layer's saved activations 36 d, the backward's fp32 rows 16 d, its
    bf16 rows 18 d, two transposed operands 16 d, attention scratch 12 d, column sums 3.25 d)."""
    d, used = 768, []
    shape = shape_of(dict(SMALL, n_layers=1, d_model=d, n_heads=d // 64, d_ff=4 * d))
    for B in (32, 32, 96):   # the first one also allocates what the process keeps
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        with ie.Trainer(**instance_config(shape, B, 128)):
            used.append(before - torch.cuda.mem_get_info()[0])
    per_token = (used[2] - used[1]) / (64 * 128)
    print(f"trainer bytes {used}: {per_token / d:.1f} d a token", flush=True)
    assert per_token <= 145 * d, per_token / d


@pytest.mark.parametrize("d,F,group,wide", [(768, 3072, (256, 128), (128, 192)), (512, 2048, (128, 128), (128, 128))])
def test_every_gradient_of_4096_tokens(d, F, group, wide):
    """The tiles of a BERT-width step: the four weight gradients' one launch, and the FFN-up and dv products."""
    B, S = 32, 128
    assert ie.test_gemm_group(256, [(d, F), (F, d), (d, d), (3 * d, d)], B * S) == group
    assert ie.test_gemm_plan(B * S, F, d, F, 256)[2:] == wide
    shape = shape_of(dict(SMALL, n_layers=1, d_model=d, n_heads=d // 64, d_ff=F, causal=0))
    print(f"train step B={B} S={S} d={d} F={F}", flush=True)
    x, labels = make_batch(shape, B, S, 811)
    loss_ref, grads_ref, _ = T.loss_and_grads(T.initial_params(shape), x, labels, shape)
    with ie.Trainer(**instance_config(shape, B, S)) as tr:
        tr.step(x, labels)
        assert abs(tr.loss() - loss_ref) <= LOSS_REL * abs(loss_ref)
        for layer, slot, name, ref in oracle_tensors(grads_ref, shape):
            g = tr.export(layer, slot, ie.TRAIN_GRAD, ref.shape)
            assert np.all(np.isfinite(g)) and rel_l2(g, ref) <= GRAD_REL_L2, (name, rel_l2(g, ref))
