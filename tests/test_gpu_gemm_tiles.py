"""Every output tile of the GEMM at its edges: rows one past and one short of a
tile, one to five K tiles (fewer than, as many as and more than the LDS ring
holds), an odd number of K tiles in the even/odd order.  Against the fp64
product with the accumulation bound of test_gpu_kernels.py; the last rows also
bit for bit against a launch of those rows alone, which takes another tile."""
import numpy as np
import pytest
import torch

import paper_2503_05130_amd as ie
from oracle import forward as F
from tests.gpu_util import DEV, f64, sync, to_dev
from tests.test_gpu_kernels import U32, UBF, gemm_bound, gemm_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,M,N,K", [
    ((32, 32), 1, 64, 64), ((32, 32), 33, 128, 192), ((32, 32), 31, 192, 384),
    ((32, 64), 65, 3072, 64), ((32, 64), 100, 2304, 320),
    ((64, 64), 129, 4096, 64), ((64, 64), 513, 1024, 320),
    ((64, 96), 500, 2304, 64), ((64, 96), 513, 2304, 320),
    ((128, 64), 500, 4096, 192), ((128, 64), 2000, 1024, 320),
    ((128, 96), 513, 3072, 64), ((128, 96), 4095, 768, 320),     # one workgroup per CU: 4-slot rings
    ((128, 96), 2049, 2304, 192),                                # two per CU: 2-slot rings
    ((128, 128), 513, 4096, 192), ((128, 128), 2050, 1024, 64),
    ((128, 192), 4097, 2304, 192),
    ((256, 256), 4000, 4096, 1024), ((256, 256), 4095, 4096, 1088),
    ((32, 32), 33, 64, 2048), ((32, 64), 65, 3072, 2112), ((64, 64), 129, 4096, 2048),
    ((64, 96), 513, 2304, 2112), ((128, 64), 257, 4096, 2112),
    ((128, 96), 4095, 768, 2112),
    ((128, 128), 513, 4096, 2112), ((256, 128), 4097, 1024, 2048), ((256, 128), 2047, 8192, 2112),
])
@pytest.mark.parametrize("epi", [ie.EPI_BIAS_BF16, ie.EPI_BIAS_RESID_F32])
def test_tile(tile, M, N, K, epi):
    print(f"gemm tile {tile} M={M} N={N} K={K} epi={epi}", flush=True)
    assert ie.test_gemm_plan(M, N, K, N, 256)[2:] == tile
    a, w, bias, resid = gemm_inputs(M, N, K, seed=M + N + K)
    a_d, w_d, b_d = to_dev(a), to_dev(w.t()), to_dev(bias)
    fp32 = epi == ie.EPI_BIAS_RESID_F32
    r_d = torch.from_numpy(resid).to(DEV) if fp32 else None
    out = torch.full((M, N), float("nan"), dtype=torch.float32 if fp32 else torch.bfloat16, device=DEV)
    ie.test_gemm(epi, a_d, w_d, b_d, r_d, out, M, N, K)
    n = min(M, 16)
    part = torch.empty((n, N), dtype=out.dtype, device=DEV)
    ie.test_gemm(epi, a_d[M - n:].contiguous(), w_d, b_d, r_d[M - n:].contiguous() if fp32 else None, part, n, N, K)
    sync()
    # the first, the last and some rows between, so that the fp64 reference stays small
    rows = np.unique(np.concatenate([np.arange(min(M, 40)), np.arange(max(0, M - 300), M), np.arange(0, M, 97)]))
    a64, w64 = f64(a)[rows], f64(w)
    pre = F.linear(a64, w64, f64(bias))
    bound = gemm_bound(a64, w64, K)
    got = f64(out)[rows]
    if fp32:
        r64 = resid[rows].astype(np.float64)
        ref, tol = pre + r64, bound + 2 * U32 * (np.abs(pre + r64) + np.abs(r64)) + 1e-7
    else:
        ref, tol = pre, bound + UBF * np.abs(pre) * 1.01
    assert np.all(np.isfinite(f64(out)))
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) - tol))
    assert torch.equal(part.view(torch.int32 if fp32 else torch.int16),
                       out[M - n:].view(torch.int32 if fp32 else torch.int16))
