"""The attention kernel's placement of (query group, head) on the grid: head
counts that do not fill the 8 XCDs, group counts that leave the reversed rows of
32 workgroups partly filled, chunks of which only the first 32 keys are visible.
Every output element is written and within the kernel's bound of the oracle."""
import numpy as np
import pytest
import torch

import paper_2503_05130_amd as ie
from oracle import forward as F
from tests.gpu_util import DEV, f64, sync, to_dev
from tests.test_gpu_kernels import UBF, attn_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,S,dh", [
    (1, 1, 1, 64), (1, 1, 33, 128), (1, 7, 129, 64), (1, 9, 96, 64), (3, 3, 161, 128),
    (1, 9, 2200, 64),      # 18 groups of 2 heads an XCD: a row of 32 and one of 4
    (1, 17, 1400, 128),    # 11 groups of 3 heads: 32 and 1
    (2, 20, 897, 64),      # 8 groups of 5 heads: 32 and 8
    (13, 20, 300, 64),     # 780 workgroups: more than three a CU, a chunk's blocks one after the other
    (12, 20, 500, 64),     # 960
    (13, 20, 300, 128),    # head dim 128: side by side at any number
])
@pytest.mark.parametrize("causal", [False, True])
def test_every_query_is_placed_once(B, H, S, dh, causal):
    print(f"attention placement B={B} H={H} S={S} dh={dh} causal={causal}", flush=True)
    q, k, v = attn_inputs(B, H, S, dh, seed=S + H, scale=1.0)
    vt = torch.full((B, H, dh, (S + 63) // 64 * 64), float("nan"), dtype=torch.bfloat16)
    vt[..., :S] = v.transpose(2, 3)
    ctx = torch.full((B, S, H * dh), float("nan"), dtype=torch.bfloat16, device=DEV)
    ie.test_attention(to_dev(q), to_dev(k), to_dev(vt), ctx, B, H, S, dh, causal)
    sync()
    got = f64(ctx).reshape(B, S, H, dh)
    assert np.all(np.isfinite(got))
    vmax = np.abs(f64(v)).max()
    for b in range(B):
        for h in range(H):
            ref = F.attention_context(f64(q[b, h]), f64(k[b, h]), f64(v[b, h]), causal)
            tol = 2.5 * UBF * vmax + UBF * 1.01 * np.abs(ref) + 1e-4 * vmax
            assert np.all(np.abs(got[b, :, h] - ref) <= tol), (b, h)
