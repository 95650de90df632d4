"""Every output tile of the GEMM with every epilogue that the forward pass and
training use, and the grouped launch of weight gradients.  The tile is reached
through the CU count that the choice is made for; rows and K tiles leave
remainders.  Against the fp64 product with the accumulation bound of
test_gpu_kernels.py, and bit for bit against another tile of the same order."""
import itertools

import numpy as np
import pytest
import torch

import paper_2503_05130_amd as ie
from oracle import forward as F
from oracle import train as T
from tests.gpu_util import DEV, bf16_round, f64, sync, to_dev
from tests.test_gpu_kernels import U32, UBF, gemm_bound

pytestmark = pytest.mark.gpu

N_CUS = (1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256)
SEQUENTIAL = [(32, 32), (32, 64), (64, 64), (64, 96), (128, 64), (128, 96), "128 x 96, two a CU", (128, 128), (128, 192), (256, 256)]
SPLIT = [(32, 32), (32, 64), (64, 64), (64, 96), (128, 64), (128, 96), (128, 128), (256, 128)]
TILES = [(False, t) for t in SEQUENTIAL] + [(True, t) for t in SPLIT]


def pick(split, tile, plan, widths):
    """The smallest (M, N, K, n_cu) with M one short of or one past a multiple of the tile that runs on `tile`."""
    two = tile == "128 x 96, two a CU"
    bm, bn = (128, 96) if two else tile
    ks = (2112,) if split else (1088,) if bm == 256 else (320, 704)
    shapes = [(m, n, k) for m in (bm + 1, 2 * bm - 1, 3 * bm + 1, 4 * bm - 1, 6 * bm + 1, 8 * bm - 1) for n in widths(bn) for k in ks]
    for (m, n, k), c in itertools.product(sorted(shapes, key=lambda s: s[0] * s[1] * s[2]), N_CUS):
        tiles = -(-m // bm) * (n // bn)
        if plan(m, n, k, c) != (bm, bn) or ((bm, bn) == (128, 96) and not split and (tiles > c) != two):
            continue
        return m, n, k, c
    raise AssertionError(f"no product found for {tile}")


def multiples(bn):
    step = bn if bn % 64 == 0 else 64 * bn // np.gcd(64, bn)
    return [int(step * i) for i in (1, 2, 3, 4, 6)]


def operands(M, N, K, seed):
    rng = np.random.default_rng(seed)
    a, w = bf16_round(rng.standard_normal((M, K))), bf16_round(rng.standard_normal((N, K)) * 0.05)
    return rng, a, w, bf16_round(rng.standard_normal(N) * 0.1)


EPILOGUES = (ie.EPI_LN_RESID_F32, ie.EPI_F32, ie.EPI_GELU_BWD_BF16, ie.EPI_GELU2_BF16, ie.EPI_BIAS_GELU_BF16)


@pytest.mark.parametrize("split,tile,epi", [   # 128 x 192 is never chosen for the LayerNorm residual
    (s, t, e) for (s, t), e in itertools.product(TILES, EPILOGUES) if (t, e) != ((128, 192), ie.EPI_LN_RESID_F32)])
def test_epilogue(split, tile, epi):
    ln = epi == ie.EPI_LN_RESID_F32
    M, N, K, n_cu = pick(split, tile, lambda m, n, k, c: ie.test_gemm_plan(m, n, k, n, c, ln)[2:], multiples)
    print(f"gemm tile {tile} M={M} N={N} K={K} n_cu={n_cu} epi={epi}", flush=True)
    rng, a, w, b = operands(M, N, K, M + N + K + epi)
    z = (rng.standard_normal((M, N)) * 2).astype(np.float32)
    stats = np.stack([rng.standard_normal(M), rng.uniform(0.3, 2, M)], 1).astype(np.float32)
    gam, bet = (1 + 0.2 * rng.standard_normal(N)).astype(np.float32), (0.2 * rng.standard_normal(N)).astype(np.float32)
    aux = bf16_round(rng.standard_normal((M, N)) * 2)
    fp32 = epi in (ie.EPI_LN_RESID_F32, ie.EPI_F32)
    dev = {k: torch.from_numpy(v).to(DEV) for k, v in dict(resid=z, stats=stats, gamma=gam, beta=bet).items()}
    w_d, b_d = to_dev(w), to_dev(b)

    def launch(rows, cus):
        n = rows.stop - rows.start
        o = torch.full((n, N), float("nan"), dtype=torch.float32 if fp32 else torch.bfloat16, device=DEV)
        o2 = torch.full((n, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        ie.test_gemm_on(cus, epi, to_dev(a[rows]), w_d, o, n, N, K, bias=b_d, resid=dev["resid"][rows].contiguous(),
                        stats=dev["stats"][rows].contiguous(), gamma=dev["gamma"], beta=dev["beta"], aux=to_dev(aux[rows]), out2=o2)
        sync()
        return o, o2

    out, out2 = launch(slice(0, M), n_cu)
    a64, w64, b64 = f64(a), f64(w).T, f64(b)
    acc, bound, got = a64 @ w64, gemm_bound(a64, w64, K), f64(out)
    assert np.all(np.isfinite(got))
    if epi == ie.EPI_F32:
        ref, tol = acc, bound
    elif ln:
        xh = (z.astype(np.float64) - stats[:, :1]) * stats[:, 1:]
        ref = gam * xh + bet + acc + b64
        # the residual's three roundings on terms of at most |gamma| (|z| + |mean|) rstd + |beta|, the sums' two
        mag = np.abs(gam) * (np.abs(z) + np.abs(stats[:, :1])) * stats[:, 1:] + np.abs(bet)
        tol = bound + 4 * U32 * mag + 2 * U32 * (np.abs(ref) + np.abs(acc) + np.abs(b64)) + 1e-7
    elif epi == ie.EPI_GELU_BWD_BF16:
        g = T._gelu_grad(f64(aux))
        ref, tol = acc * g, bound * np.abs(g) + 1e-6 * np.abs(acc) + UBF * 1.01 * np.abs(acc * g) + 1e-7
    elif epi == ie.EPI_BIAS_GELU_BF16:
        pre = acc + b64
        ref = F.gelu(pre)
        tol = 1.13 * bound + UBF * 1.01 * np.abs(ref) + 1e-6 * np.abs(pre) + 1e-7
    else:
        ref, tol = acc + b64, bound + UBF * 1.01 * np.abs(acc + b64)
        want2 = F.gelu(got)   # of the value as rounded
        assert np.all(np.abs(f64(out2) - want2) <= UBF * 1.01 * np.abs(want2) + 1e-6 * np.abs(got) + 1e-7)
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) - tol))
    rows = slice(max(0, M - 17), M)
    part, part2 = launch(rows, 256)
    assert torch.equal(part.view(torch.int16), out[rows].view(torch.int16))
    assert epi != ie.EPI_GELU2_BF16 or torch.equal(part2.view(torch.int16), out2[rows].view(torch.int16))


@pytest.mark.parametrize("seq8", [False, True])
@pytest.mark.parametrize("split,tile", TILES)
def test_qkv_scatter(split, tile, seq8):
    """seq8: sequences of a multiple of 8 positions (16-byte stores of V^T); else odd ones (single elements)."""
    # d_model = K = N / 3, its heads 64 wide, a multiple of the tile's width
    pair = (128, 96) if isinstance(tile, str) else tile
    step = pair[1] * 64 // np.gcd(64, pair[1])
    d = int(-(-(2048 if split else 1024 if pair[0] == 256 else 320 if pair == (128, 64) else 192) // step) * step)
    found = None
    for B, S, c in itertools.product((1, 3, 5, 9, 13, 17, 25, 33), (40, 104, 200) if seq8 else (37, 93, 125), N_CUS + (512,)):
        tiles = -(-B * S // pair[0]) * (3 * d // pair[1])
        if ie.test_gemm_plan(B * S, 3 * d, d, d, c)[2:] != pair or (B * S) % pair[0] == 0 or B * S < pair[0]:
            continue
        if pair == (128, 96) and not split and (tiles > c) != isinstance(tile, str):
            continue
        if found is None or B * S < found[0] * found[1]:
            found = B, S, c
    assert found, tile
    (B, S, n_cu), H = found, d // 64
    print(f"qkv tile {tile} B={B} S={S} d={d} n_cu={n_cu}", flush=True)
    M, spad = B * S, (S + 63) // 64 * 64
    _, a, w, b = operands(M, 3 * d, d, M + d)
    q = torch.full((B, H, S, 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    k, vt = torch.full_like(q, float("nan")), torch.full((B, H, 64, spad), float("nan"), dtype=torch.bfloat16, device=DEV)
    ie.test_gemm_qkv_on(n_cu, to_dev(a), to_dev(w), to_dev(b), q, k, vt, B, S, d, H)
    sync()
    a64, w64 = f64(a), f64(w).T
    ref = (a64 @ w64 + f64(b)).reshape(B, S, 3, H, 64)
    bound = gemm_bound(a64, w64, d).reshape(B, S, 3, H, 64)
    got = [f64(q), f64(k), f64(vt)[..., :S].transpose(0, 1, 3, 2)]
    for i in range(3):
        want, tol = ref[:, :, i].transpose(0, 2, 1, 3), bound[:, :, i].transpose(0, 2, 1, 3)
        assert np.all(np.abs(got[i] - want) <= tol + UBF * 1.01 * np.abs(want) + 1e-7), "QKV"[i]
    assert torch.all(torch.isnan(vt[..., S:]))   # the padding is left alone


@pytest.mark.parametrize("split,tile", [(s, t) for s, t in TILES if not isinstance(t, str)])
def test_group_sums_like_single_products(split, tile):
    """Four products of one K in one launch have the bits of four launches, whatever the group's tile."""
    bm, bn = tile
    found = None
    for m, c, k in itertools.product((1, 2, 3, 5), N_CUS, (2048, 2112) if split else (1088,) if bm == 256 else (64, 192, 320)):
        n = multiples(bn)
        shapes = [(m * bm + 1, n[1]), (bm - 1, n[0]), (m * bm, n[2]), (17, n[1])]
        if ie.test_gemm_group(c, shapes, k) == tile:
            found = shapes, k, c
            break
    assert found, tile
    shapes, K, n_cu = found
    print(f"gemm group tile {tile} {shapes} K={K} n_cu={n_cu}", flush=True)
    ops = [operands(m, n, K, m + n) for m, n in shapes]
    a, w = [to_dev(o[1]) for o in ops], [to_dev(o[2]) for o in ops]
    out = [torch.full(s, float("nan"), device=DEV) for s in shapes]
    assert ie.test_gemm_group(n_cu, shapes, K, a, w, out) == tile
    for j, (m, n) in enumerate(shapes):
        one = torch.full((m, n), float("nan"), device=DEV)
        ie.test_gemm_on(256, ie.EPI_F32, a[j], w[j], one, m, n, K)
        sync()
        assert torch.all(torch.isfinite(one)) and torch.equal(out[j].view(torch.int32), one.view(torch.int32)), j
