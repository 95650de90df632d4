"""Host inputs and outputs give the bits that device ones give, on both sides of
the size (65536 floats) up to which they go through the instance's pinned
buffers, and batch after batch (the buffers are used again)."""
import numpy as np
import pytest
import torch

import paper_2503_05130_amd as ie
import workloads as W
from tests.gpu_util import DEV, instance_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,seq,n_out", [
    (1, 1, 1), (3, 5, 3),
    (4, 128, 0),     # input and output exactly at the limit
    (3, 171, 0),     # one row past it
    (4, 128, 2), (5, 103, 3),
])
def test_host_equals_device(batch, seq, n_out):
    print(f"host staging batch={batch} seq={seq} n_out={n_out}", flush=True)
    shape = W.model_shape("encoder_l1_d128_s32_b2", n_out=n_out)
    with ie.Instance(**instance_config(shape, batch, seq)) as inst:
        for k in range(3):
            x = W.make_input(500 + k, batch, seq, 128)
            xd = torch.from_numpy(x).to(DEV)
            inst.submit(xd)
            want = inst.read_logits()
            out = torch.empty((batch, seq, inst.out_width), device=DEV)
            inst.read_logits(out)
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
            inst.submit(x)
            x[:] = np.nan   # the input was copied before submit returned
            assert np.array_equal(inst.read_logits().view(np.uint32), want.view(np.uint32)), k
            assert inst.last_batch_ms() > 0
