"""The decode product's forms for 9-16 rows (two rows a wave in the LayerNorm
prologue), the order of its sums over K, and the packed copy made for one sequence
as larger decode batches (5-8 and 9-16 sequences) read it."""
import numpy as np
import pytest
import torch

import paper_2503_05130_amd as ie
import workloads as W
from oracle import forward as F
from tests.gpu_util import DEV, bf16_round, compare, f64, instance_config, sync, to_dev
from tests.test_gpu_kernels import UBF, gemm_bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,ln", [
    (9, 48, 128, True), (16, 3072, 1024, True), (13, 4096, 1024, True), (9, 384, 1792, True),
    (9, 16, 2048, False), (16, 1024, 4096, False), (12, 2048, 2080, False),
    (16, 2064, 2048, False), (16, 1024, 2016, False),
])
def test_nine_to_sixteen_rows(M, N, K, ln):
    print(f"skinny M={M} N={N} K={K} ln={ln}", flush=True)
    rng = np.random.default_rng(M + N + K)
    w = bf16_round(rng.standard_normal((K, N)) * 0.05)
    b = bf16_round(rng.standard_normal(N) * 0.1)
    w_d, b_d = to_dev(w.t()), to_dev(b)
    if ln:
        z = (rng.standard_normal((M, K)) * 2 + 0.5).astype(np.float32)
        g = (1 + 0.1 * rng.standard_normal(K)).astype(np.float32)
        be = (0.1 * rng.standard_normal(K)).astype(np.float32)
        lnarg, a_d = tuple(torch.from_numpy(t).to(DEV) for t in (z, g, be)) + (1e-5,), None
        y = F.layer_norm(z.astype(np.float64), g.astype(np.float64), be.astype(np.float64), 1e-5)
        extra = UBF * (np.abs(y) @ np.abs(f64(w)))   # the normalised rows are rounded to bf16
    else:
        a = bf16_round(rng.standard_normal((M, K)))
        lnarg, a_d, y, extra = None, to_dev(a), f64(a), 0.0
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    ie.test_gemm_skinny(ie.EPI_BIAS_BF16, a_d, w_d, b_d, None, out, M, N, K, ln=lnarg)
    packed = torch.empty(N * K, dtype=torch.bfloat16, device=DEV)
    groups = ie.test_skinny_groups(M, N, K, ln)
    ie.test_skinny_pack(w_d, packed, N, K, groups)
    out2 = torch.full_like(out, float("nan"))
    ie.test_gemm_skinny_packed(ie.EPI_BIAS_BF16, a_d, packed, groups, b_d, None, out2, M, N, K, ln=lnarg)
    sync()
    ref = F.linear(y, f64(w), f64(b))
    tol = gemm_bound(y, f64(w), K) + extra + UBF * 1.01 * np.abs(ref) + 1e-6
    assert np.all(np.abs(f64(out) - ref) <= tol)
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16))


@pytest.mark.parametrize("M,N,K", [(16, 1024, 4096), (9, 2048, 2048), (16, 512, 2080), (16, 4096, 1024), (13, 48, 800)])
def test_order_of_sums(M, N, K):
    """One K-group: wave w of 8 adds the 32-wide K steps w, w + 8, ... in turn, then the waves' sums are added in
    wave order, whatever N and K.  A feature has three terms, 2^30, s in 1 .. 63 and -2^30, in steps that order adds
    one after the other: s is lost where it follows 2^30 (whose last place is 2^7) and stays where it comes last."""
    assert ie.test_skinny_groups(M, N, K, False) == 1
    print(f"skinny order M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(N + K)
    small = rng.integers(1, 64, N).astype(np.float32)
    lost = rng.random(N) < 0.5
    v = np.zeros((N, K // 32), np.float32)
    for f in range(N):
        if rng.random() < 0.6:   # one wave's three steps
            at = np.sort(rng.choice(np.arange(rng.integers(8), K // 32, 8), 3, replace=False))
        else:                    # three waves' sums
            at = np.sort(rng.choice(8, 3, replace=False)) + 8 * rng.integers(0, K // 256, 3)
        v[f, at] = [2.0 ** 30, small[f], -2.0 ** 30] if lost[f] else [2.0 ** 30, -2.0 ** 30, small[f]]
    w, a = torch.zeros((N, K), dtype=torch.bfloat16), torch.zeros((M, K), dtype=torch.bfloat16)
    at = 32 * np.arange(K // 32) + rng.integers(0, 32, K // 32)
    w[:, at], a[:, at] = torch.from_numpy(v).bfloat16(), 1.0
    zero = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    out = torch.empty_like(zero)
    ie.test_gemm_skinny(ie.EPI_BIAS_RESID_F32, to_dev(a), to_dev(w), torch.zeros(N, dtype=torch.bfloat16, device=DEV),
                        zero, out, M, N, K)
    sync()
    assert np.array_equal(out.cpu().numpy(), np.broadcast_to(np.where(lost, 0, small), (M, N)))


@pytest.mark.parametrize("epi", [ie.EPI_BIAS_BF16, ie.EPI_BIAS_GELU_BF16, ie.EPI_BIAS_RESID_F32])
@pytest.mark.parametrize("M,N,K,groups,ln", [
    (16, 1024, 1024, 4, False), (9, 48, 128, 4, False), (16, 1024, 4096, 2, False), (13, 64, 4224, 4, False),
    (8, 1024, 4096, 4, False), (5, 48, 256, 4, False),          # 2 groups read the copy for 4
    (16, 3072, 1024, 2, True), (9, 384, 1792, 4, True), (7, 384, 2176, 4, True), (6, 512, 640, 4, True),
])
def test_copy_for_more_groups(M, N, K, groups, ln, epi):
    """A product reads a copy made for two or four times its K-groups to the same bits as row-major weights."""
    own = ie.test_skinny_groups(M, N, K, ln)
    print(f"skinny copy M={M} N={N} K={K} own={own} copy={groups} ln={ln} epi={epi}", flush=True)
    assert groups in (2 * own, 4 * own)
    rng = np.random.default_rng(M + N + K + epi)
    w_d, b_d = to_dev(bf16_round(rng.standard_normal((N, K)) * 0.05)), to_dev(bf16_round(rng.standard_normal(N) * 0.1))
    z, g, be, r = (torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(DEV) for s in ((M, K), K, K, (M, N)))
    lnarg, a_d = ((z, g, be, 1e-5), None) if ln else (None, z.bfloat16())
    fp32 = epi == ie.EPI_BIAS_RESID_F32
    want = torch.full((M, N), float("nan"), dtype=torch.float32 if fp32 else torch.bfloat16, device=DEV)
    got = torch.full_like(want, float("nan"))
    packed = torch.empty(N * K, dtype=torch.bfloat16, device=DEV)
    ie.test_skinny_pack(w_d, packed, N, K, groups)
    ie.test_gemm_skinny(epi, a_d, w_d, b_d, r if fp32 else None, want, M, N, K, ln=lnarg)
    ie.test_gemm_skinny_shared(epi, a_d, packed, groups, b_d, r if fp32 else None, got, M, N, K, ln=lnarg)
    sync()
    bits = torch.int32 if fp32 else torch.int16
    assert torch.all(torch.isfinite(want)) and torch.equal(got.view(bits), want.view(bits))


def test_copy_for_other_groups_is_refused():
    w = torch.zeros((2048, 2048), dtype=torch.bfloat16, device=DEV)
    b, a = torch.zeros(2048, dtype=torch.bfloat16, device=DEV), torch.zeros((8, 2048), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((8, 2048), dtype=torch.bfloat16, device=DEV)
    assert ie.test_skinny_groups(8, 2048, 2048, False) == 2
    for groups in (1, 3, 8):
        with pytest.raises(ie.IefwdError) as e:
            ie.test_gemm_skinny_shared(ie.EPI_BIAS_BF16, a, w, groups, b, None, out, 8, 2048, 2048)
        assert e.value.status == ie.EINVAL


def test_decode_weights_take_one_copy():
    """An instance's device memory holds one packed copy of its matrices, whatever max_batch: the same tokens in
    16 sequences take no more than in 4, but for the decode attention's partial results (under 8 MB here)."""
    shape = W.model_shape("decoder_l24_d1024_s512", n_layers=4, n_out=0)
    used = []
    for batch, seq in ((4, 256), (4, 256), (16, 64)):   # the first one also allocates what the process keeps
        sync()
        before = torch.cuda.mem_get_info()[0]
        with ie.Instance(**dict(instance_config(shape, batch, seq), kv_cache=1)):
            used.append(before - torch.cuda.mem_get_info()[0])
    print(f"decode instance bytes: {used}", flush=True)
    matrices = 4 * 12 * 1024 * 1024 * 2
    assert 2 * matrices <= used[1] and used[2] - used[1] <= (24 << 20), used


@pytest.mark.parametrize("batch", [3, 6, 16])
def test_instance_decodes_each_class(batch):
    shape = W.model_shape("decoder_l24_d1024_s512", n_layers=2, n_out=0, b_std=0.02, ln_std=0.02, qk_std=0.05)
    S = 20
    x = W.make_input(9100 + batch, batch, S + 2, 1024)
    print(f"decode class of {batch} sequences", flush=True)
    with ie.Instance(**dict(instance_config(shape, 16, S + 2), kv_cache=1)) as inst:
        inst.submit(np.ascontiguousarray(x[:, :S]))
        inst.wait()
        for i in range(2):
            inst.decode(np.ascontiguousarray(x[:, S + i]), S + i)
            got = inst.read_logits()[:, 0]
            ma, rl = compare(got, F.forward(x[:, :S + i + 1], shape)[:, -1])
            assert rl <= 1e-2 and ma <= 5e-2, (i, ma, rl)
