"""Benchmark: batched transformer forward pass of one serverless DL instance on
one MI355X.

Workload (one "step" = one batch through the whole forward pass):
BERT-base-shaped post-LN encoder, 12 layers, d_model 768, 12 heads, FFN 3072,
GELU, per-token 768->2 head, seq 128, batch 32, seeded random-init bf16
weights, fp32 N(0,1) input embeddings already resident in HBM, full 256-CU
quota.

Prints one JSON line: inferences/s (one inference = one sequence), the
forward-level MFMA utilisation, the roofline of the dominant kernel (FFN-down
GEMM + bias + LayerNorm residual: each launch in the timed region records its own
start and end into HIP events), the aggregate throughput of two co-located instances at
CU quotas 64/192, 128/128 and 192/64 against one alone, and the fp64 CPU oracle
timed on a bounded sample, the per-batch cost of re-masking the
instance's stream between batches, throughput and MFMA utilisation at CU
quotas (BERT-base batch 32; the RoBERTa-large-sized causal decoder at batch 8,
S 512), the four GEMM classes against hipBLASLt on the same shapes, and a
training step of the same encoder (batch 32, AdamW).

  python bench.py [--steps K] [--warmup W] [--gpus 1] [--no-cpu-baseline] [--no-colocated] [--no-remask]
                  [--no-quota-sweep] [--no-gemm-reference] [--no-hbm-kernels] [--timer-every N]
                  [--no-train | --train-only] [--decode | --decode-only]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2516.6     # 256 CU x 4096 FLOP/clk x 2.4 GHz, dense bf16 MFMA
WORKLOAD = "bert_base_l12_d768_s128"
# Bytes per launch of the FFN-down kernel between the L2s and the memory side (FETCH_SIZE x
# 2.000 + WRITE_SIZE x 1.000 KiB, factors from a 256 MiB device copy in the same runs): L2
# misses, which the 256 MB MALL may serve without touching HBM.  Valid only for the GEMM
# source and build flags they were counted on; any other source reports null.
FFN2_TRAFFIC = {"source_sha256_16": "407f0ca975856833", "bytes": (37200.7 * 2.0 + 14668.0 * 1.0) * 1024}
GEMM_SOURCES = ("paper_2503_05130_amd/csrc/gemm.hip", "paper_2503_05130_amd/csrc/gemm.h", "paper_2503_05130_amd/csrc/gemm_device.h",
                "paper_2503_05130_amd/csrc/launch.h", "paper_2503_05130_amd/csrc/gelu.h",
                "paper_2503_05130_amd/build.py")


def gemm_source_hash() -> str:
    import hashlib

    h = hashlib.sha256()
    for f in GEMM_SOURCES:
        with open(os.path.join(ROOT, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def forward_flops(L, d, F, H, S, n_out, causal=False):
    """Algorithmic FLOPs of one sequence (multiply-add = 2)."""
    gemm = 2 * S * d * (3 * d) + 2 * S * d * d + 2 * S * d * F + 2 * S * F * d
    attn = (2 * (S * (S + 1) // 2) * d * 2) if causal else 4 * S * S * d
    return L * (gemm + attn) + 2 * S * d * n_out


def host_info(blas) -> dict:
    """nproc, CPU model and the BLAS library NumPy calls (threadpoolctl's view)."""
    model = ""
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    return {"nproc": len(os.sched_getaffinity(0)), "cpu_count": os.cpu_count(), "cpu_model": model,
            "blas": [{"api": p.get("internal_api"), "version": p.get("version"), "threads": p.get("num_threads"),
                      "library": os.path.basename(p.get("filepath", ""))} for p in blas]}


def cpu_baseline(shape, batch_sample: int):
    """The fp64 oracle on `batch_sample` sequences of the same workload."""
    from threadpoolctl import threadpool_info

    import workloads as W
    from oracle import forward as F
    from oracle import init_spec as I

    w = W.WORKLOADS[WORKLOAD]
    x = W.make_input(w["input_seed"], batch_sample, w["seq"], shape["d_model"])
    layers = [I.layer_weights(shape, l) for l in range(shape["n_layers"])]
    glob = I.global_weights(shape)
    t0 = time.perf_counter()
    F.forward_with(x, shape, lambda l: layers[l], glob)
    dt = time.perf_counter() - t0
    blas = [p for p in threadpool_info() if p.get("user_api") == "blas"]
    threads = max([p.get("num_threads", 1) for p in blas] or [os.cpu_count() or 1])
    return {"value": round(batch_sample / dt, 4), "unit": "inferences/s", "cores": int(threads),
            "kind": "oracle", "host": host_info(blas),
            "sample": f"{batch_sample} sequences of the same workload (seq 128), NumPy fp64 forward, "
                      f"weights pre-generated; {dt:.2f} s"}


def oracle_timing() -> dict:
    """The fp64 oracle timed on this host's cores on every workload of the
    plan: the single-layer encoder (batch 2), BERT-base at batch 1 / 8 / 32
    (median of 3 runs), the RoBERTa-large-sized causal decoder at batch 8 and
    the d = 2048 decoder at batch 2 (one run each), plus single-thread runs of
    the two smallest.  Weights are generated before the clock starts; inputs
    are the workloads' seeded inputs.  inferences/s = batch / wall time."""
    import statistics

    from threadpoolctl import threadpool_info, threadpool_limits

    import workloads as W
    from oracle import forward as F
    from oracle import init_spec as I

    plan = [("encoder_l1_d128_s32_b2", 2, 3, None), ("encoder_l1_d128_s32_b2", 2, 3, 1),
            ("bert_base_l12_d768_s128", 1, 3, None), ("bert_base_l12_d768_s128", 1, 3, 1),
            ("bert_base_l12_d768_s128", 8, 3, None), ("bert_base_l12_d768_s128", 32, 3, None),
            ("decoder_l24_d1024_s512", 8, 1, None), ("decoder_l24_d2048_s1024", 2, 1, None)]
    rows, weights = [], {}
    for name, batch, runs, threads in plan:
        shape = W.model_shape(name)
        w = W.WORKLOADS[name]
        if name not in weights:
            weights.clear()
            weights[name] = ([I.layer_weights(shape, l) for l in range(shape["n_layers"])], I.global_weights(shape))
        layers, glob = weights[name]
        x = W.make_input(w["input_seed"], batch, w["seq"], shape["d_model"])
        times = []
        with threadpool_limits(limits=threads):
            used = max([p.get("num_threads", 1) for p in threadpool_info() if p.get("user_api") == "blas"] or [1])
            for _ in range(runs):
                t0 = time.perf_counter()
                F.forward_with(x, shape, lambda l: layers[l], glob)
                times.append(time.perf_counter() - t0)
        t = statistics.median(times)
        rows.append({"workload": name, "batch": batch, "blas_threads": used, "runs": runs,
                     "seconds": round(t, 3), "inferences_s": round(batch / t, 4)})
        print(json.dumps(rows[-1]), file=sys.stderr, flush=True)
    blas = [p for p in threadpool_info() if p.get("user_api") == "blas"]
    return {"kind": "oracle", "host": host_info(blas), "rows": rows}


def colocated(ie, W, shape, cfg, quota_pairs, batch=8, window_s=1.0):
    """Aggregate throughput of two co-located instances (independent seeds) on
    disjoint CU sets, each driven by its own host thread with back-to-back
    batches, against one instance alone at the full quota.  Inputs are device-resident.  Each leg
    runs for a fixed wall-clock window and counts the batches that completed
    inside it, so an instance at a small quota does not stretch the window of
    the other one."""
    import threading

    import torch

    w = W.WORKLOADS[WORKLOAD]
    S, d = w["seq"], shape["d_model"]
    insts = [ie.Instance(device=0, max_batch=batch, max_seq=S, **dict(cfg, seed=31 + i)) for i in range(2)]
    xs = [torch.from_numpy(W.make_input(31000 + 1000 * i, batch, S, d)).to("cuda:0") for i in range(2)]
    torch.cuda.synchronize()

    def drive(i, deadline, done):
        n = 0
        while True:
            insts[i].submit(xs[i])
            insts[i].wait()
            if time.perf_counter() > deadline:
                break
            n += 1
        done[i] = n

    def window(active):
        for i in active:                      # warm the re-masked streams
            for _ in range(5):
                insts[i].submit(xs[i])
                insts[i].wait()
        done = [0, 0]
        t0 = time.perf_counter()
        ths = [threading.Thread(target=drive, args=(i, t0 + window_s, done)) for i in active]
        for t in ths:
            t.start()
        for t in ths:
            t.join()
        return batch * sum(done) / window_s

    insts[0].set_quota(256)
    solo = window([0])
    out = {"workload": f"2 x {WORKLOAD}, batch {batch} each", "window_s": window_s,
           "solo_inf_s": round(solo, 1), "pairs": []}
    for qa, qb in quota_pairs:
        insts[0].set_quota(qa, 0)          # disjoint CUs: bits [0, qa) and [qa, qa + qb)
        insts[1].set_quota(qb, qa)
        agg = window([0, 1])
        out["pairs"].append({"quotas": [qa, qb], "aggregate_inf_s": round(agg, 1),
                             "vs_solo": round(agg / solo, 3)})
    for inst in insts:
        inst.close()
    return out


def remask_overhead(inst, x, n=40):
    """Cost of re-masking between batches: mean batch time with the quota
    alternating 128 <-> 256 on every batch, against the mean of the two fixed
    quotas.  Each batch is waited for, so the figures are per-batch latencies."""
    import torch

    def run(quotas):
        for q in quotas[:4]:
            inst.set_quota(q)
            inst.submit(x)
            inst.wait()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for q in quotas:
            inst.set_quota(q)
            inst.submit(x)
            inst.wait()
        return (time.perf_counter() - t0) * 1e3 / len(quotas)

    t256 = run([256] * n)
    t128 = run([128] * n)
    alt = run([128, 256] * (n // 2))
    inst.set_quota(256)
    base = (t128 + t256) / 2
    return {"ms_fixed_256": round(t256, 4), "ms_fixed_128": round(t128, 4), "ms_alternating": round(alt, 4),
            "overhead_pct": round((alt - base) / base * 100, 2)}


def decode_leg(ie, W, batch=2, prompt=512, steps=64):
    """Decode phase of the d = 2048 causal decoder (24 layers, 16 heads, FFN
    8192): a prompt of `prompt` tokens per sequence, then `steps` decode steps
    of one token per sequence (fresh synthetic embeddings each step).  Time per
    output token (TPOT) is the mean device time of a step; the roofline counts
    the bytes a step must read (every weight once, the KV cache up to the
    position) against 8 TB/s."""
    import torch

    name = "decoder_l24_d2048_s1024"
    shape = W.model_shape(name)
    d, L, F_, H = shape["d_model"], shape["n_layers"], shape["d_ff"], shape["n_heads"]
    cfg = {k: shape[k] for k in ("n_layers", "d_model", "n_heads", "d_ff", "pre_ln", "causal", "n_out",
                                 "ln_eps", "w_std", "b_std", "ln_std", "qk_std", "seed")}
    inst = ie.Instance(device=0, max_batch=batch, max_seq=prompt + steps, kv_cache=1, **cfg)
    rng = np.random.default_rng(9100)
    xp = torch.from_numpy(rng.standard_normal((batch, prompt, d), dtype=np.float32)).to("cuda:0")
    xs = torch.from_numpy(rng.standard_normal((steps, batch, d), dtype=np.float32)).to("cuda:0")
    kinds = {"qkv": ie.K_QKV, "attn": ie.K_ATTN, "out": ie.K_OUTPROJ, "ffn1": ie.K_FFN1, "ffn2": ie.K_FFN2,
             "ln": ie.K_LN}
    ms = []
    for rep in range(3):                      # warm-up, TPOT, per-kernel-class times
        inst.submit(xp)
        inst.wait()
        if rep == 2:
            for k in kinds.values():
                inst.time_kernel(k, True)
        for g in range(steps):
            inst.decode(xs[g], prompt + g)
            inst.wait()
            if rep == 1:
                ms.append(inst.last_batch_ms())
    per = {}
    for nm, k in kinds.items():
        t, n = inst.kernel_time(k)
        inst.time_kernel(k, False)
        per[nm] = round(t * 1e3 / steps, 2)        # us per step
    inst.close()
    tpot = float(np.mean(ms))
    wbytes = L * 2 * (3 * d * d + d * d + 2 * d * F_) + L * 2 * 4 * (2 * d) + 2 * 4 * d
    kvbytes = sum(L * batch * 2 * (prompt + g + 1) * d * 2 for g in range(steps)) / steps
    gbs = (wbytes + kvbytes) / (tpot * 1e-3) / 1e9
    return {"workload": f"{name} decode, batch {batch}, prompt {prompt}, {steps} steps", "tpot_ms": round(tpot, 4),
            "tokens_per_s": round(batch / (tpot * 1e-3), 1),
            "roofline": {"bound": "hbm", "achieved": round(gbs, 1), "peak": 8000.0, "unit": "GB/s",
                         "frac": round(gbs / 8000.0, 4), "bytes_per_step": round(wbytes + kvbytes)},
            "us_per_step": per}


def quota_sweep(ie, W, inst, x, B, S, shape):
    """Throughput and forward-level MFMA utilisation at CU quotas: the BERT-base
    batch at 64 / 128 / 192 / 256 CUs, and the RoBERTa-large-sized causal
    decoder (24 layers, d 1024, S 512, batch 8) at 64 / 128 / 256 CUs.  Device
    time per batch from the instance's own events; utilisation against the
    quota's share of the bf16 peak."""
    def run(instance, xin, quotas, flops_batch, batch, n_warm, n_time):
        out = []
        for q in quotas:
            instance.set_quota(q)
            for _ in range(n_warm):
                instance.submit(xin)
                instance.wait()
            ms = []
            for _ in range(n_time):
                instance.submit(xin)
                instance.wait()
                ms.append(instance.last_batch_ms())
            t = float(np.median(ms))
            out.append({"quota_cus": q, "ms_per_batch": round(t, 4), "inferences_s": round(batch / (t * 1e-3), 1),
                        "mfma_util_pct": round(flops_batch / (t * 1e-3) / (PEAK_BF16_TFLOPS * 1e12 * q / 256) * 100, 2)})
        instance.set_quota(256)
        return out

    d, F_, L, H = shape["d_model"], shape["d_ff"], shape["n_layers"], shape["n_heads"]
    res = {"bert": {"workload": f"{WORKLOAD}, batch {B}",
                    "points": run(inst, x, (64, 128, 192, 256), forward_flops(L, d, F_, H, S, shape["n_out"]) * B, B,
                                  3, 10)}}
    import torch

    name = "decoder_l24_d1024_s512"
    ds = W.model_shape(name)
    wd = W.WORKLOADS[name]
    cfg = {k: ds[k] for k in ("n_layers", "d_model", "n_heads", "d_ff", "pre_ln", "causal", "n_out", "ln_eps",
                              "w_std", "b_std", "ln_std", "qk_std", "seed")}
    dec = ie.Instance(device=0, max_batch=wd["batch"], max_seq=wd["seq"], **cfg)
    xd = torch.from_numpy(W.make_input(wd["input_seed"], wd["batch"], wd["seq"], ds["d_model"])).to("cuda:0")
    fl = forward_flops(ds["n_layers"], ds["d_model"], ds["d_ff"], ds["n_heads"], wd["seq"], ds["n_out"], causal=True)
    res["decoder"] = {"workload": f"{name}, batch {wd['batch']}",
                      "points": run(dec, xd, (64, 128, 256), fl * wd["batch"], wd["batch"], 2, 5),
                      "paper_context": "RoBERTa-large inference iteration 25 ms solo, 50 ms under SM contention, "
                                       "NVIDIA A100-40GB, batch / sequence / precision not stated (Sec. 3.4.1)"}
    dec.close()
    return res


def gemm_reference(ie, inst, x, B, S, shape, reps=20):
    """The forward's four GEMM classes against torch.matmul (hipBLASLt) on the
    same shapes with plain bf16 outputs: the library reference for what these
    small products reach on this chip.  `ours_us` is per launch inside the
    forward, with the fused epilogues (head scatter, residual, GELU, LayerNorm
    residual rebuild and fp32 out); `ours_plain_us` is the same product with
    the plain bias -> bf16 epilogue, timed in isolation exactly like the
    library call (the like-for-like main-loop comparison)."""
    import torch

    kinds = {"qkv": ie.K_QKV, "out_proj": ie.K_OUTPROJ, "ffn_up": ie.K_FFN1, "ffn_down": ie.K_FFN2}
    for k in kinds.values():
        inst.time_kernel(k, True)
    for _ in range(reps):
        inst.submit(x)
        inst.wait()
    ours = {}
    for nm, k in kinds.items():
        t, n = inst.kernel_time(k)
        inst.time_kernel(k, False)
        ours[nm] = t * 1e3 / max(n, 1)
    T, d, F_ = B * S, shape["d_model"], shape["d_ff"]
    shapes = {"qkv": (T, 3 * d, d), "out_proj": (T, d, d), "ffn_up": (T, F_, d), "ffn_down": (T, d, F_)}
    out = {}
    for nm, (M, N, K) in shapes.items():
        a = torch.randn(M, K, device="cuda:0", dtype=torch.bfloat16)
        w = torch.randn(N, K, device="cuda:0", dtype=torch.bfloat16)
        c = torch.empty(M, N, device="cuda:0", dtype=torch.bfloat16)
        for _ in range(5):
            torch.matmul(a, w.t(), out=c)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            torch.matmul(a, w.t(), out=c)
        e1.record()
        torch.cuda.synchronize()
        lib_us = e0.elapsed_time(e1) * 1e3 / reps
        bias = torch.zeros(N, device="cuda:0", dtype=torch.bfloat16)
        for _ in range(5):
            ie.test_gemm(0, a, w, bias, None, c, M, N, K)
        torch.cuda.synchronize()
        e0.record()
        for _ in range(reps):
            ie.test_gemm(0, a, w, bias, None, c, M, N, K)
        e1.record()
        torch.cuda.synchronize()
        plain_us = e0.elapsed_time(e1) * 1e3 / reps
        fl = 2.0 * M * N * K
        out[nm] = {"mnk": [M, N, K], "ours_us": round(ours[nm], 2), "ours_plain_us": round(plain_us, 2),
                   "hipblaslt_us": round(lib_us, 2), "ours_tflops": round(fl / ours[nm] / 1e6, 1),
                   "ours_plain_tflops": round(fl / plain_us / 1e6, 1), "hipblaslt_tflops": round(fl / lib_us / 1e6, 1)}
    return out


def hbm_kernels(ie, inst, x, B, S, shape, reps=20):
    """Achieved HBM bandwidth of the forward's memory-bound kernels: algorithmic
    bytes over device time per launch (HIP events around each launch, on the
    instance's stream).  LayerNorm class of a post-LN forward: the input cast
    (4 B in, 2 B out per element), 2L - 1 LayerNorms (4 B in, 2 B out per
    element, 8 B of statistics per row) and the last LayerNorm fused with the
    head (4 B in per element, the logits out).  Attention: Q, K and V^T read
    once (2 B each per element of the [T, d] activations), the context written
    once (2 B)."""
    T, d, L = B * S, shape["d_model"], shape["n_layers"]
    if shape["pre_ln"]:
        return None
    ln_bytes = T * d * 6 + (2 * L - 1) * (T * d * 6 + T * 8) + T * d * 4 + T * shape["n_out"] * 4
    attn_bytes = L * (3 * T * d * 2 + T * d * 2)
    kinds = {"layernorm": (ie.K_LN, ln_bytes, 2 * L + 1), "attention": (ie.K_ATTN, attn_bytes, L)}
    for k, _, _ in kinds.values():
        inst.time_kernel(k, True)
    for _ in range(reps):
        inst.submit(x)
        inst.wait()
    out = {}
    for nm, (k, nbytes, per_fwd) in kinds.items():
        ms, n = inst.kernel_time(k)
        inst.time_kernel(k, False)
        fwd = n / per_fwd
        gbs = nbytes * fwd / (ms * 1e-3) / 1e9
        out[nm] = {"launches": n, "avg_us": round(ms * 1e3 / max(n, 1), 2),
                   "bytes_per_launch": round(nbytes / per_fwd), "achieved_GBps": round(gbs, 1),
                   "frac_of_hbm_peak": round(gbs / 8000.0, 3)}
    return out


def train_flops(L, d, F, H, S, n_out, causal=False):
    """Algorithmic FLOPs of one training step per sequence: the forward, and a
    backward of twice the forward's products (input and weight gradients of
    every GEMM, the four attention products' gradients, the head's)."""
    return 3 * forward_flops(L, d, F, H, S, n_out, causal)


def train_leg(ie, W, batch=32, steps=10, warmup=3):
    """Training steps of the BERT-base-shaped post-LN encoder (batch 32, seq
    128, 2-class per-token cross-entropy, AdamW) at the full quota: device time
    per step, sequences/s, MFMA utilisation of the step's algorithmic FLOPs,
    and the split over kernel classes."""
    import torch

    name = WORKLOAD
    shape = W.model_shape(name)
    S = W.WORKLOADS[name]["seq"]
    cfg = {k: shape[k] for k in ("n_layers", "d_model", "n_heads", "d_ff", "pre_ln", "causal", "n_out", "ln_eps",
                                 "w_std", "b_std", "ln_std", "qk_std", "seed")}
    tr = ie.Trainer(device=0, max_batch=batch, max_seq=S, **cfg)
    x = torch.from_numpy(W.make_input(7100, batch, S, shape["d_model"])).to("cuda:0")
    lab = torch.from_numpy(W.make_labels(7101, batch, S, shape["n_out"])).to("cuda:0")
    for _ in range(warmup):
        tr.step(x, lab)
        tr.wait()
    ms, losses = [], []
    for _ in range(steps):
        tr.step(x, lab)
        losses.append(tr.loss())
        ms.append(tr.last_batch_ms())
    kinds = {"forward": (ie.K_QKV, ie.K_ATTN, ie.K_OUTPROJ, ie.K_FFN1, ie.K_FFN2, ie.K_LN),
             "backward_gemm": (ie.K_BWD_GEMM,), "backward_other": (ie.K_BWD,), "optimizer": (ie.K_OPTIM,)}
    for ks in kinds.values():
        for k in ks:
            tr.time_kernel(k, True)
    for _ in range(3):
        tr.step(x, lab)
        tr.wait()
    split = {}
    for nm, ks in kinds.items():
        tot = 0.0
        for k in ks:
            t, _ = tr.kernel_time(k)
            tr.time_kernel(k, False)
            tot += t
        split[nm] = round(tot / 3, 3)
    tr.close()
    t = float(np.median(ms))
    fl = train_flops(shape["n_layers"], shape["d_model"], shape["d_ff"], shape["n_heads"], S, shape["n_out"]) * batch
    return {"workload": f"{name} training step, batch {batch}, 2-class per-token cross-entropy, AdamW",
            "ms_per_step": round(t, 4), "sequences_s": round(batch / (t * 1e-3), 1),
            "tokens_s": round(batch * S / (t * 1e-3), 1),
            "mfma_util_pct": round(fl / (t * 1e-3) / (PEAK_BF16_TFLOPS * 1e12) * 100, 2),
            "loss_first_last": [round(losses[0], 5), round(losses[-1], 5)], "ms_by_class": split}


def copy_calibration(mib: int) -> None:
    """A plain device-to-device copy of `mib` MiB, for scaling the FETCH_SIZE /
    WRITE_SIZE counters of a profiling run (read once, written once)."""
    import torch

    a = torch.empty(mib * 2 ** 20, dtype=torch.uint8, device="cuda:0")
    b = torch.empty_like(a)
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()


def start_clock_sampler(path: str):
    """Starts `amd-smi metric --clock` in a loop (each sample preceded by a
    wall-clock timestamp) as a child process.  Called before this process
    touches the GPU, so no process that holds a GPU context starts another
    program.  Returns the Popen handle, or None if amd-smi is unavailable or a
    profiler is attached (its preloaded library initialises the GPU first)."""
    import shutil
    import subprocess

    if any(k.startswith("ROCPROF") for k in os.environ) or not shutil.which("amd-smi"):
        return None
    loop = "while :; do date +%s.%N; amd-smi metric --clock; sleep 0.05; done"
    return subprocess.Popen(["bash", "-c", loop], stdout=open(path, "w"), stderr=subprocess.DEVNULL,
                            start_new_session=True)


def stop_clock_sampler(proc, path: str, t0: float, t1: float):
    """Stops the sampler and returns the mean GFX clock (MHz, over all XCDs and
    the samples taken between t0 and t1 on the wall clock) and the sample count."""
    import re
    import signal

    try:
        os.killpg(proc.pid, signal.SIGTERM)
    except ProcessLookupError:
        pass
    proc.wait(timeout=10)
    with open(path) as f:
        text = f.read()
    os.remove(path)
    blocks = re.split(r"^(\d+\.\d+)\s*$", text, flags=re.M)
    means = []
    for i in range(1, len(blocks) - 1, 2):
        ts = float(blocks[i])
        vals = [float(v) for v in re.findall(r"GFX_\d+:\s*\n\s*CLK:\s*([\d.]+)\s*MHz", blocks[i + 1])]
        if t0 <= ts <= t1 and vals:
            means.append(sum(vals) / len(vals))
    if not means:
        return None, 0
    return sum(means) / len(means), len(means)


def clock_leg(inst, x, sampler, path: str, seconds: float = 3.0):
    """Mean shader clock while the same forward runs back to back for `seconds`."""
    import torch

    end = time.time() + seconds
    t0 = time.time() + 0.3          # skip the first samples while clocks ramp
    n = 0
    while time.time() < end:
        inst.submit(x)
        inst.wait()
        n += 1
    torch.cuda.synchronize()
    t1 = time.time()
    mhz, samples = stop_clock_sampler(sampler, path, t0, t1)
    return {"method": "amd-smi metric --clock sampled while the forward runs back to back "
                      f"({n} batches, {seconds:.0f} s), mean over XCDs and samples",
            "sclk_mhz": round(mhz, 1) if mhz else None, "samples": samples}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--batch", type=int, default=32)
    ap.add_argument("--quota", type=int, default=256)
    ap.add_argument("--cpu-sample", type=int, default=96)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-colocated", action="store_true")
    ap.add_argument("--no-remask", action="store_true")
    ap.add_argument("--no-quota-sweep", action="store_true")
    ap.add_argument("--no-gemm-reference", action="store_true")
    ap.add_argument("--no-train", action="store_true")
    ap.add_argument("--no-hbm-kernels", action="store_true")
    ap.add_argument("--timer-every", type=int, default=4,
                    help="per-launch events on the dominant kernel in every n-th timed batch")
    ap.add_argument("--train-only", action="store_true",
                    help="time only the training step (a profiling aid: prints {\"train\": ...})")
    ap.add_argument("--decode", action="store_true", help="also time the decode phase of the d=2048 decoder")
    ap.add_argument("--decode-only", action="store_true",
                    help="time only the decode phase (a profiling aid: prints {\"decode\": ...})")
    ap.add_argument("--copy-calibration-mib", type=int, default=0,
                    help="first run a plain device copy of this many MiB (counter calibration)")
    ap.add_argument("--no-clock", action="store_true", help="skip the measured shader clock leg")
    ap.add_argument("--oracle-timing", action="store_true",
                    help="time only the fp64 oracle on every workload (CPU; prints {\"oracle_timing\": ...})")
    args = ap.parse_args()
    if args.oracle_timing:
        print(json.dumps({"oracle_timing": oracle_timing()}))
        return 0
    if args.gpus != 1:
        print(f"bench.py measures one GPU only (the instances of this workload share one MI355X); "
              f"--gpus {args.gpus} is not supported", file=sys.stderr)
        return 2

    if args.timer_every < 1:
        print("--timer-every must be >= 1", file=sys.stderr)
        return 2

    clock_path = None
    sampler = None
    if not (args.no_clock or args.decode_only or args.train_only):
        import tempfile
        fd, clock_path = tempfile.mkstemp(prefix="bench_sclk_", suffix=".txt")
        os.close(fd)
        sampler = start_clock_sampler(clock_path)   # before anything touches the GPU
        if sampler is None:
            os.remove(clock_path)

    import torch

    import paper_2503_05130_amd as ie
    import workloads as W

    if args.copy_calibration_mib:
        copy_calibration(args.copy_calibration_mib)
    if args.decode_only:
        print(json.dumps({"decode": decode_leg(ie, W)}))
        return 0
    if args.train_only:
        print(json.dumps({"train": train_leg(ie, W)}))
        return 0
    w = W.WORKLOADS[WORKLOAD]
    shape = W.model_shape(WORKLOAD)
    B, S = args.batch, w["seq"]
    cfg = {k: shape[k] for k in ("n_layers", "d_model", "n_heads", "d_ff", "pre_ln", "causal", "n_out",
                                 "ln_eps", "w_std", "b_std", "ln_std", "qk_std", "seed")}
    inst = ie.Instance(device=0, max_batch=B, max_seq=S, **cfg)
    inst.set_quota(args.quota)
    x = torch.from_numpy(W.make_input(w["input_seed"], B, S, shape["d_model"])).to("cuda:0")
    torch.cuda.synchronize()

    for _ in range(args.warmup):
        inst.submit(x)
        inst.wait()

    # The dominant kernel's launches carry a start and a stop event on every
    # TIMER_EVERY-th batch of the timed region: events on every launch cost
    # ~5 us each (~4% of a batch), which would understate `value`.
    dominant = ie.K_FFN2
    k_ms, k_launches = 0.0, 0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        sampled = i % args.timer_every == 0
        if sampled:
            inst.time_kernel(dominant, True)
        inst.submit(x)
        inst.wait()
        if sampled:
            ms, n = inst.kernel_time(dominant)
            inst.time_kernel(dominant, False)
            k_ms, k_launches = k_ms + ms, k_launches + n
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0

    out = inst.read_logits()
    if not np.all(np.isfinite(out)):
        print("non-finite logits", file=sys.stderr)
        return 1

    d, F_, L, H = shape["d_model"], shape["d_ff"], shape["n_layers"], shape["n_heads"]
    flops_seq = forward_flops(L, d, F_, H, S, shape["n_out"])
    ms_step = elapsed * 1e3 / args.steps
    value = B * args.steps / elapsed
    mfma_util = flops_seq * B / (ms_step * 1e-3) / (PEAK_BF16_TFLOPS * 1e12 * args.quota / 256) * 100

    kernel_flops = 2.0 * (B * S) * F_ * d
    k_avg_s = k_ms * 1e-3 / max(k_launches, 1)
    achieved = kernel_flops / k_avg_s / 1e12
    peak = PEAK_BF16_TFLOPS * args.quota / 256
    roof = {"bound": "mfma", "achieved": round(achieved, 2), "peak": round(peak, 1), "unit": "TFLOP/s",
            "frac": round(achieved / peak, 4),
            "traffic": (round(FFN2_TRAFFIC["bytes"]) if gemm_source_hash() == FFN2_TRAFFIC["source_sha256_16"]
                        else None),
            "traffic_level": "L2 <-> memory side (FETCH_SIZE + WRITE_SIZE): L2 misses, possibly MALL hits",
            "kernel": "FFN-down GEMM + bias + LayerNorm residual", "avg_us": round(k_avg_s * 1e6, 2), "launches": k_launches,
            "timed_batches": f"every {args.timer_every}th of the {args.steps} timed batches"}

    result = {
        "metric": "inferences/sec (aggregate, co-located) + MFMA util % at given CU quotas, 1 GPU",
        "value": round(value, 2),
        "unit": "inferences/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (seeded N(0,1) fp32 embeddings, seeded random-init bf16 weights)",
        "config": {"workload": WORKLOAD, "n_layers": L, "d_model": d, "n_heads": H, "d_ff": F_,
                   "global_batch": B, "seq_len": S, "quota_cus": args.quota, "parallelism": "none (1 instance)"},
        "mfma_util_pct": round(mfma_util, 2),
        "roofline": roof,
    }
    if sampler is not None:
        clk = clock_leg(inst, x, sampler, clock_path)
        if clk["sclk_mhz"]:
            # the same utilisation against the peak at the clock the chip actually ran
            clk["mfma_util_pct_at_sclk"] = round(mfma_util * 2400.0 / clk["sclk_mhz"], 2)
            clk["ffn_down_frac_at_sclk"] = round(roof["frac"] * 2400.0 / clk["sclk_mhz"], 4)
        result["clock"] = clk
    if not args.no_remask:
        result["remask"] = remask_overhead(inst, x)
    if not args.no_quota_sweep:
        result["quota_sweep"] = quota_sweep(ie, W, inst, x, B, S, shape)
    if not args.no_gemm_reference:
        result["gemm_reference"] = gemm_reference(ie, inst, x, B, S, shape)
    if not args.no_hbm_kernels:
        result["hbm_kernels"] = hbm_kernels(ie, inst, x, B, S, shape)
    inst.close()
    if not args.no_colocated:
        result["colocated"] = colocated(ie, W, shape, cfg, [(64, 192), (128, 128), (192, 64)])
        # the same pairs at the headline batch: two batch-32 instances against one
        result["colocated_b32"] = colocated(ie, W, shape, cfg, [(64, 192), (128, 128), (192, 64)], batch=B)
    if args.decode:
        result["decode"] = decode_leg(ie, W)
    if not args.no_train:
        result["train"] = train_leg(ie, W)
    if not args.no_cpu_baseline:
        result["cpu_baseline"] = cpu_baseline(shape, args.cpu_sample)
    print(json.dumps(result))
    return 0


if __name__ == "__main__":
    sys.exit(main())
