"""Performance cases of libiefwd: the calls its users make, over the range of sizes they make them at.

A user of the library holds one instance per serverless function (model weights, workspace, a
compute share) and drives it through the Python binding: ``submit`` / ``read_logits`` for a batch of an
encoder or a prompt of a causal model, ``decode`` / ``read_logits`` per generated token, ``step`` /
``loss`` for a training function.  Each case is one such call (or the short loop of calls that a user
writes around it).  Most cases are stacks of one to four layers, whose outputs are the hidden
states; two are whole BERT-base-shaped models, which return logits.

Weights are the library's seeded init (written out again below, in fp64, for ``exact``) with non-zero
biases and LayerNorm affine, and Q / K columns scaled so that attention scores have a standard deviation
of about 2.8 at every width; inputs are standard normal fp32 embeddings.
"""
import math

import numpy as np
import torch

import paper_2503_05130_amd as ie

DEV = "cuda:0"


# ------------------------------------------------------------------------------------ cases
def _encode(name, layers, d, batch, seq, n_out=0, quota=0, host=False, d_ff=0):
    return dict(name=name, kind="encode", layers=layers, d=d, head_dim=64, d_ff=d_ff or 4 * d, batch=batch, seq=seq,
                n_out=n_out, quota=quota, host=host)


def _prefill(name, layers, d, head_dim, batch, seq, d_ff=0):
    return dict(name=name, kind="prefill", layers=layers, d=d, head_dim=head_dim, d_ff=d_ff or 4 * d, batch=batch,
                seq=seq)


def _decode(name, layers, d, head_dim, batch, context, steps):
    return dict(name=name, kind="decode", layers=layers, d=d, head_dim=head_dim, d_ff=4 * d, batch=batch,
                context=context, steps=steps)


def _train(name, layers, d, d_ff, batch, seq, n_out, steps, full):
    return dict(name=name, kind="train", layers=layers, d=d, head_dim=64, d_ff=d_ff, batch=batch, seq=seq,
                n_out=n_out, steps=steps, full=full)


def listed():
    return [
        # the smallest request: one small encoder layer, host buffers in and out; launches and waits count
        _encode("encode_small", 1, 128, 2, 32, host=True),
        # one request of a BERT-base-shaped service at low load: the latency of 12 layers of short launches
        _encode("bert_base_b1", 12, 768, 1, 128, n_out=2),
        # a full batch of that service: the throughput case
        _encode("bert_base_b32", 12, 768, 32, 128, n_out=2),
        # a batch as it happens to arrive: odd batch, odd sequence length
        _encode("encode_ragged", 2, 768, 7, 93),
        # the same model on a quarter of the GPU beside other instances
        _encode("encode_quota64", 2, 768, 8, 128, quota=64),
        # prompts of a RoBERTa-large-sized causal model
        _prefill("prefill_d1024", 2, 1024, 64, 8, 512),
        # prompts of the large causal model, head dim 128
        _prefill("prefill_d2048", 2, 2048, 128, 2, 1024),
        # one long odd-sized prompt: attention is most of the work
        _prefill("prefill_long", 1, 1024, 64, 1, 4001),
        # token generation of the large causal model for two sequences: bound by reading the weights
        _decode("decode_d2048_b2", 4, 2048, 128, 2, 512, 4),
        # token generation for sixteen sequences with long contexts: the KV cache is most of the bytes
        _decode("decode_d1024_b16", 4, 1024, 64, 16, 3000, 4),
        # training at BERT-base width: forward, backward and AdamW on 4096 tokens
        _train("train_d768", 2, 768, 3072, 32, 128, 2, 3, False),
        # training a small model: many short launches; the first layer's matrix gradients come back too
        _train("train_small", 2, 128, 512, 4, 32, 3, 6, True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["encode", "encode", "prefill", "decode", "train"])
    if kind == "encode":
        d = rng.choice([128, 256, 512, 768, 768, 1024])
        batch, seq = _log_int(rng, 1, 32), _log_int(rng, 16, 256)
        while batch * seq > 4096:
            batch, seq = _log_int(rng, 1, 32), _log_int(rng, 16, 256)
        c = _encode("", rng.randint(1, 4), d, batch, seq, n_out=rng.choice([0, 0, 2]), quota=rng.choice([0, 0, 0, 64, 128]),
                    host=rng.random() < 0.2, d_ff=rng.choice([4 * d, 4 * d, 2 * d, 3 * d + 64]))
    elif kind == "prefill":
        d, head_dim = rng.choice([(512, 64), (1024, 64), (1024, 128), (2048, 128)])
        batch, seq = _log_int(rng, 1, 8), _log_int(rng, 48, 4000)
        while batch * seq * d > 4096 * 1024:
            batch, seq = _log_int(rng, 1, 8), _log_int(rng, 48, 4000)
        c = _prefill("", rng.randint(1, 2), d, head_dim, batch, seq)
    elif kind == "decode":
        d, head_dim = rng.choice([(512, 64), (1024, 64), (1024, 128), (2048, 128)])
        c = _decode("", rng.randint(1, 4), d, head_dim, _log_int(rng, 1, 16), _log_int(rng, 20, 3500), rng.randint(1, 4))
        while c["batch"] * c["context"] * d > 16 * 3000 * 1024:
            c["context"] = _log_int(rng, 20, 3500)
    else:
        d = rng.choice([128, 256, 512, 768])
        full = d <= 256
        seq = rng.choice([16, 32, 48, 64, 96, 128])
        batch = _log_int(rng, 1, 4 if full else 32)
        while (batch * seq) % 64:
            batch += 1
        c = _train("", rng.randint(1, 2), d, rng.choice([4 * d, 2 * d]), batch, seq, rng.randint(2, 6), 6 if full else 3, full)
    del c["name"]
    return c


def _config(case, seed):
    """The instance configuration of a case."""
    causal = case["kind"] in ("prefill", "decode")
    seq = case["context"] + case["steps"] if case["kind"] == "decode" else case["seq"]
    return dict(n_layers=case["layers"], d_model=case["d"], n_heads=case["d"] // case["head_dim"], d_ff=case["d_ff"],
                max_batch=case["batch"], max_seq=seq, n_out=case.get("n_out", 0), pre_ln=int(causal), causal=int(causal),
                kv_cache=int(case["kind"] == "decode"), ln_eps=1e-5, w_std=0.02, b_std=0.02, ln_std=0.02,
                qk_std=math.sqrt(2.8 / case["d"]), seed=seed * 977 + 5)


def _inputs(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed * 131 + 17)
    normal = lambda *shape: torch.randn(*shape, generator=g, device=DEV, dtype=torch.float32)  # noqa: E731
    b, d = case["batch"], case["d"]
    if case["kind"] == "decode":
        return {"prompt": normal(b, case["context"], d), "x": normal(case["steps"], b, d)}
    if case["kind"] == "train":
        labels = torch.randint(0, case["n_out"], (case["steps"], b, case["seq"]), generator=g, device=DEV, dtype=torch.int32)
        return {"x": normal(case["steps"], b, case["seq"], d), "labels": labels}
    return {"x": normal(b, case["seq"], d)}


TRAIN = dict(lr=1e-4)
VECTORS = (1, 3, 4, 5, 7, 9, 10, 11)   # biases and LayerNorm parameters of a layer
MATRICES = (0, 2, 6, 8)


def prepare(case, seed):
    s = {"case": case, **_inputs(case, seed)}
    torch.cuda.synchronize()   # the inputs are made on torch's stream, the instance runs on its own
    if case["kind"] == "train":
        s["inst"] = ie.Trainer(train=TRAIN, **_config(case, seed))
        return s
    s["inst"] = ie.Instance(**_config(case, seed))
    if case.get("quota"):
        s["inst"].prepare_quota(case["quota"])
        s["inst"].set_quota(case["quota"])
    if case.get("host"):
        s["x"] = s["x"].cpu().numpy()
    if case["kind"] == "decode":
        s["inst"].submit(s["prompt"])
        s["inst"].wait()
        del s["prompt"]
    return s


def run(s):
    case, inst = s["case"], s["inst"]
    if case["kind"] in ("encode", "prefill"):
        inst.submit(s["x"])
        if case.get("host"):
            return inst.read_logits()
        out = torch.empty((case["batch"], case["seq"], inst.out_width), device=DEV)
        return inst.read_logits(out)
    if case["kind"] == "decode":   # each token's output is there before the next token's input is given
        outs = []
        for i in range(case["steps"]):
            inst.decode(s["x"][i], case["context"] + i)
            outs.append(inst.read_logits(torch.empty((case["batch"], 1, inst.out_width), device=DEV)))
        return outs
    losses = []
    for i in range(case["steps"]):
        inst.step(s["x"][i], s["labels"][i])
        losses.append(inst.loss())
    out = {"loss": np.array(losses), "logits": inst.read_logits(torch.empty((case["batch"], case["seq"], case["n_out"]), device=DEV))}
    d, f, n = case["d"], case["d_ff"], case["n_out"]
    shapes = {0: (d, 3 * d), 1: (3 * d,), 2: (d, d), 6: (d, f), 7: (f,), 8: (f, d)}
    for layer in range(case["layers"]):
        for slot in VECTORS + (MATRICES if case["full"] and layer == 0 else ()):
            out["grad_%d_%d" % (layer, slot)] = inst.export(layer, slot, ie.TRAIN_GRAD, shapes.get(slot, (d,)))
    out["grad_head"] = inst.export(case["layers"], 14, ie.TRAIN_GRAD, (d, n))
    out["grad_head_bias"] = inst.export(case["layers"], 15, ie.TRAIN_GRAD, (n,))
    return out


def work(case):
    d, f, b, layers = case["d"], case["d_ff"], case["batch"], case["layers"]
    params = 4 * d * d + 2 * d * f   # of one layer's matrices
    if case["kind"] == "decode":
        flops = bytes_ = 0
        for i in range(case["steps"]):
            keys = case["context"] + i + 1
            flops += layers * (2 * b * params + 4 * b * keys * d)
            bytes_ += layers * (2 * params + 2 * 2 * b * keys * d) + 2 * 4 * b * d
        return {"bytes": bytes_, "flops": flops}
    t, s = b * case["seq"], case["seq"]
    attn = 2 * t * (s + 1) * d if case["kind"] == "prefill" else 4 * t * s * d
    flops = layers * (2 * t * params + attn)
    width = case.get("n_out", 0) or d
    if case["kind"] == "train":
        # three products of the forward's size; 30 bytes a parameter in AdamW (gradient, master and two
        # moments read, master and moments and the bf16 copy written)
        return {"bytes": case["steps"] * (layers * params * 30 + 4 * t * d), "flops": 3 * case["steps"] * flops}
    return {"bytes": layers * 2 * params + 4 * t * d + 4 * t * width, "flops": flops}


def tolerance(case):
    # bf16 operands and intermediates with fp32 sums: the error against exact() measures 0.2 to 0.25% of the
    # output's norm for the blocks up to width 1024, 0.35 to 0.6% for width 2048 and the 12-layer models
    if case["kind"] == "train":
        # a weight's bf16 copy may round the other way after an update, and a gradient entry near zero gets
        # an AdamW step of either sign
        return {"rel": 4e-2}
    return {"rel": 2e-2 if case.get("n_out") or case["d"] * case["layers"] > 2048 else 1e-2}


# --------------------------------------------------------------------------- the same in 64 bits
def _i64(v):
    return v - (1 << 64) if v >= 1 << 63 else v


def _shift(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)   # logical


def _mix(z):
    """The SplitMix64 output function on int64 tensors (wrapping)."""
    z = z + _i64(0x9E3779B97F4A7C15)
    z = (z ^ _shift(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shift(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ _shift(z, 31)


def _normals(seed, layer, slot, n):
    one = lambda v: torch.tensor([_i64(v & ((1 << 64) - 1))], dtype=torch.int64)  # noqa: E731
    key = int(_mix(one(seed) ^ _mix(one(32 * layer + slot))))
    c = 2 * torch.arange(n, device=DEV, dtype=torch.int64) + key
    u1 = (_shift(_mix(c), 11) + 1).double() * 2.0 ** -53
    u2 = _shift(_mix(c + 1), 11).double() * 2.0 ** -53
    return torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(6.283185307179586 * u2)


def _weights(cfg):
    """Per layer {slot: fp64 tensor} and the global ones: the library's documented seeded init."""
    f32 = lambda v: float(np.float32(v))  # noqa: E731
    d, f, n, seed, layers = cfg["d_model"], cfg["d_ff"], cfg["n_out"], cfg["seed"], cfg["n_layers"]
    ws, bs, ls, qs = (f32(cfg[k]) for k in ("w_std", "b_std", "ln_std", "qk_std"))

    def bf16(layer, slot, shape, std):
        v = _normals(seed, layer, slot, math.prod(shape)).reshape(shape) * std
        return v.float().bfloat16().double()

    def affine(layer, slot, offset):
        return (offset + ls * _normals(seed, layer, slot, d)).float().double()

    std_qkv = torch.full((3 * d,), ws, dtype=torch.float64, device=DEV)
    std_qkv[:2 * d] = qs
    out = []
    for l in range(layers):
        out.append({0: bf16(l, 0, (d, 3 * d), std_qkv), 1: bf16(l, 1, (3 * d,), bs), 2: bf16(l, 2, (d, d), ws),
                    3: bf16(l, 3, (d,), bs), 4: affine(l, 4, 1.0), 5: affine(l, 5, 0.0), 6: bf16(l, 6, (d, f), ws),
                    7: bf16(l, 7, (f,), bs), 8: bf16(l, 8, (f, d), ws), 9: bf16(l, 9, (d,), bs),
                    10: affine(l, 10, 1.0), 11: affine(l, 11, 0.0)})
    top = {12: affine(layers, 12, 1.0), 13: affine(layers, 13, 0.0)}
    if n:
        top.update({14: bf16(layers, 14, (d, n), ws), 15: bf16(layers, 15, (n,), bs)})
    return out, top


def _norm(x, g, b, eps=float(np.float32(1e-5))):
    c = x - x.mean(-1, keepdim=True)
    return g * c / torch.sqrt((c * c).mean(-1, keepdim=True) + eps) + b


def _gelu(x):
    return 0.5 * x * (1.0 + torch.special.erf(x / math.sqrt(2.0)))


def _attend(y, w, heads, causal):
    b, s, d = y.shape
    q, k, v = ((y @ w[0] + w[1]).reshape(b, s, 3, heads, d // heads).permute(2, 0, 3, 1, 4)).unbind(0)
    ctx = []
    for i in range(b):   # one sequence at a time: the scores of all would not fit
        p = q[i] @ k[i].transpose(-1, -2).contiguous() / math.sqrt(d // heads)
        if causal:
            p = p.masked_fill(torch.ones(s, s, dtype=torch.bool, device=DEV).triu(1), -math.inf)
        ctx.append((torch.softmax(p, -1) @ v[i].contiguous()).transpose(0, 1).reshape(s, d))
    return torch.stack(ctx) @ w[2] + w[3]


def _forward(x, layers, top, heads, pre_ln, causal, n_out):
    h = x
    for w in layers:
        if pre_ln:
            h = h + _attend(_norm(h, w[4], w[5]), w, heads, causal)
            h = h + _gelu(_norm(h, w[10], w[11]) @ w[6] + w[7]) @ w[8] + w[9]
        else:
            h = _norm(h + _attend(h, w, heads, causal), w[4], w[5])
            h = _norm(h + _gelu(h @ w[6] + w[7]) @ w[8] + w[9], w[10], w[11])
    if pre_ln:
        h = _norm(h, top[12], top[13])
    return h @ top[14] + top[15] if n_out else h


def exact(case, seed):
    cfg, data = _config(case, seed), _inputs(case, seed)
    layers, top = _weights(cfg)
    heads, pre_ln, n_out = cfg["n_heads"], cfg["pre_ln"], cfg["n_out"]
    if case["kind"] in ("encode", "prefill"):
        out = _forward(data["x"].double(), layers, top, heads, pre_ln, cfg["causal"], n_out)
        return out.cpu().numpy() if case.get("host") else out
    if case["kind"] == "decode":
        outs = [[] for _ in range(case["steps"])]
        for b in range(case["batch"]):
            x = torch.cat([data["prompt"][b], data["x"][:, b]]).double()[None]
            h = _forward(x, layers, top, heads, 1, 1, 0)[0]
            for i in range(case["steps"]):
                outs[i].append(h[case["context"] + i])
        return [torch.stack(o)[:, None] for o in outs]
    # training: fp64 masters and moments; the forward reads the matrices and biases rounded to bf16
    affine = (4, 5, 10, 11, 12, 13)
    params = [(l, k, v) for l, w in enumerate(layers) for k, v in w.items()] + [(len(layers), k, top[k]) for k in (14, 15)]
    master = {(l, k): v.clone() for l, k, v in params}
    m, v2 = ({key: torch.zeros_like(t) for key, t in master.items()} for _ in range(2))
    lr, decay = float(np.float32(TRAIN["lr"])), float(np.float32(0.01))
    b1, b2, eps = float(np.float32(0.9)), float(np.float32(0.999)), float(np.float32(1e-8))
    losses = []
    for i in range(case["steps"]):
        leaf = {key: (t if key[1] in affine else t.float().bfloat16().double()).requires_grad_() for key, t in master.items()}
        ws = [{k: leaf[(l, k)] for k in layers[l]} for l in range(len(layers))]
        head = {k: leaf[(len(layers), k)] for k in (14, 15)}
        logits = _forward(data["x"][i].double(), ws, head, heads, 0, 0, n_out)
        loss = torch.nn.functional.cross_entropy(logits.reshape(-1, n_out), data["labels"][i].reshape(-1).long())
        grads = dict(zip(leaf, torch.autograd.grad(loss, list(leaf.values()))))
        losses.append(float(loss.detach()))
        for key, g in grads.items():
            m[key] = b1 * m[key] + (1 - b1) * g
            v2[key] = b2 * v2[key] + (1 - b2) * g * g
            w = master[key].detach()
            w = w * (1 - lr * decay) if key[1] in (0, 2, 6, 8, 14) else w
            master[key] = w - lr * (m[key] / (1 - b1 ** (i + 1))) / (torch.sqrt(v2[key] / (1 - b2 ** (i + 1))) + eps)
    out = {"loss": np.array(losses), "logits": logits.detach()}
    for l in range(len(layers)):
        for slot in VECTORS + (MATRICES if case["full"] and l == 0 else ()):
            out["grad_%d_%d" % (l, slot)] = grads[(l, slot)]
    out["grad_head"], out["grad_head_bias"] = grads[(len(layers), 14)], grads[(len(layers), 15)]
    return out
