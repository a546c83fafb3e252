"""Cases that stand for the use of the HiFT step library, for timing and for comparing results.

A case is one of the following kinds of work:
  sweep          one sweep of scheduled HiFT steps over all groups of a model (HiftModel.train): what the library is for
  lora           a short run of adapter steps, after which the adapters are read out (HiftModel.lora_step, lora_read)
  attention      one layer's attention, forward and backward
  linear         one linear layer: its product, the gradient of its input and that of its weight
  cross_entropy  the loss over a large vocabulary, with the gradient in place of the logits
  optimizer      the update of one group's parameters
  norm           a normalisation over rows
The sizes of the listed cases are those of the library's own workloads (hift_inputs) and tests: the tiny fp32 decoder,
the encoders of width 768 and 1024, the decoder of width 4096 (its depth cut to two layers, as in the tests).
"""
import math

import torch

import paper_2401_15207_amd as H

ADAMW = {"opt": "adamw", "lr": 1e-5, "wd": 0.0}
ENCODER_BASE = dict(kind="sweep", arch=1, layers=12, d=768, heads=12, ffn=3072, vocab=50265, classes=2, positions=514, dtype="bf16",
                    batch=8, seq=128, m=1, strategy="top2down", losses=False, parked=True, **ADAMW)
DECODER_4096 = dict(kind="sweep", arch=2, layers=2, d=4096, heads=32, ffn=11008, vocab=32000, classes=0, positions=512, dtype="bf16",
                    batch=4, seq=512, m=1, strategy="bottom2up", losses=False, parked=False, **ADAMW)


def listed():
    return [
        # the smallest model: every step is launches and latency; the loss is read after each step, as a training log does
        dict(name="sweep_tiny_fp32", kind="sweep", arch=0, layers=2, d=64, heads=4, ffn=256, vocab=256, classes=0, positions=32,
             dtype="fp32", batch=2, seq=32, m=1, strategy="bottom2up", losses=True, parked=False, opt="adamw", lr=1e-3, wd=0.01),
        # fine-tuning a small encoder with the state of inactive groups in pinned host memory, as the method prescribes
        dict(ENCODER_BASE, name="sweep_encoder_768_parked"),
        # the large encoder's widths, two units per group in random order
        dict(ENCODER_BASE, name="sweep_encoder_1024", layers=6, d=1024, heads=16, ffn=4096, classes=3, batch=16, m=2,
             strategy="random", parked=False),
        # the flagship's widths, batch and grouping, at the depth that the tests use
        dict(DECODER_4096, name="sweep_decoder_4096"),
        # the same model on a short batch padded to its longest sequence: ragged in every tile
        dict(DECODER_4096, name="sweep_decoder_4096_ragged", batch=3, seq=77),
        # the adapter method on the same kernels
        dict(DECODER_4096, name="lora_decoder_4096", kind="lora", rank=8, steps=4, lr=1e-4),
        # one layer's attention of the decoder of width 4096, with rotary positions
        dict(name="attention_causal_512", kind="attention", batch=4, heads=32, seq=512, head_dim=128, causal=True, rope=True),
        # and of the encoder of width 1024
        dict(name="attention_encoder_128", kind="attention", batch=16, heads=16, seq=128, head_dim=64, causal=False, rope=False),
        # the feed-forward input projection of the encoder of width 768: too few tiles for packed weights
        dict(name="linear_encoder_768", kind="linear", rows=1024, inner=768, outer=3072, dtype="bf16", packed=False, bias=True,
             residual=False),
        # the feed-forward output projection of the decoder of width 4096, weights laid out once
        dict(name="linear_decoder_4096", kind="linear", rows=2048, inner=11008, outer=4096, dtype="bf16", packed=True, bias=False,
             residual=True),
        # the language-model loss of the decoders
        dict(name="cross_entropy_32000", kind="cross_entropy", rows=2048, vocab=32000, seq=512, dtype="bf16"),
        # the update of one layer of the decoder of width 4096
        dict(name="optimizer_layer_4096", kind="optimizer", count=202383360, half=True, decay=True, opt="adamw", lr=1e-5, wd=0.01),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sweep", "sweep", "lora", "attention", "attention", "linear", "linear", "cross_entropy", "optimizer", "norm"])
    if kind in ("sweep", "lora"):
        arch = rng.choice([0, 1, 2])
        dtype = "fp32" if kind == "sweep" and rng.random() < 0.3 else "bf16"
        if dtype == "fp32":
            head, heads = rng.choice([16, 32, 64]), rng.randint(2, 4)
        else:
            head, heads = rng.choice([64, 128]), rng.randint(4, 16)
        d, classes = head * heads, rng.randint(2, 5) if arch == 1 else 0
        ffn = d * 4 if arch != 2 else (8 * d // 3 + 255) // 256 * 256
        layers, seq = rng.randint(1, 6), rng.randint(8, 256)
        c = dict(kind=kind, arch=arch, layers=layers, d=d, heads=heads, ffn=ffn, vocab=_log(rng, 256, 50272), classes=classes,
                 positions=seq + rng.choice([0, 2, 130]), dtype=dtype, batch=max(1, min(_log(rng, 1, 16), 2048 // seq)), seq=seq,
                 m=rng.randint(1, min(3, layers + 1)), strategy=rng.choice(["bottom2up", "top2down", "random"]),
                 losses=rng.random() < 0.4, parked=False, lr=1e-5, wd=rng.choice([0.0, 0.01]), opt="adamw")
        if kind == "lora":
            c.update(rank=rng.choice([8, 16]), steps=rng.randint(2, 6), lr=1e-4)
        else:
            c.update(opt=rng.choice(["adamw", "adamw", "sgdm"]), parked=rng.random() < 0.25)
        return c
    if kind == "attention":
        head_dim = rng.choice([64, 128])
        seq = 8 * _log(rng, 4, 128)
        heads = rng.choice([8, 12, 16, 20, 32, 40])
        batch = max(1, min(_log(rng, 1, 16), 2048 // seq))
        causal = rng.random() < 0.6
        return dict(kind=kind, batch=batch, heads=heads, seq=seq, head_dim=head_dim, causal=causal, rope=causal and rng.random() < 0.6)
    if kind == "linear":
        packed = rng.random() < 0.4
        dtype = "bf16" if packed or rng.random() < 0.8 else "fp32"
        if packed:  # what packed weights are for: enough tiles of 128 x 256 in either direction
            rows = rng.randint(1700, 2048)
            inner, outer = 256 * rng.randint(15, 40), 256 * rng.randint(15, 40)
        else:
            rows = _log(rng, 32, 2048)
            inner, outer = 8 * _log(rng, 8, 512), 8 * _log(rng, 8, 512)
        if dtype == "fp32":
            inner, outer = min(inner, 1024), min(outer, 1024)
        return dict(kind=kind, rows=rows, inner=inner, outer=outer, dtype=dtype, packed=packed, bias=rng.random() < 0.5,
                    residual=rng.random() < 0.4)
    if kind == "cross_entropy":
        seq = rng.randint(8, 512)
        return dict(kind=kind, rows=seq * rng.randint(1, max(1, 2048 // seq)), vocab=_log(rng, 250, 50272), seq=seq,
                    dtype=rng.choice(["bf16", "bf16", "fp32"]))
    if kind == "optimizer":
        return dict(kind=kind, count=_log(rng, 50000, 150000000), half=rng.random() < 0.8, decay=rng.random() < 0.7,
                    opt=rng.choice(["adamw", "adamw", "adagrad", "sgdm"]), lr=1e-5, wd=0.01)
    return dict(kind=kind, rows=_log(rng, 100, 8192), d=8 * _log(rng, 8, 640), rms=rng.random() < 0.5,
                dtype=rng.choice(["bf16", "bf16", "fp32"]))


# ---- inputs ---------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape, dtype=torch.float32, scale=1.0):
    return (torch.randn(*shape, generator=g, device="cuda") * scale).to(dtype)


def _dtype(case):
    return torch.bfloat16 if case.get("dtype") == "bf16" else torch.float32


def _code(case):
    return 1 if case.get("dtype") == "bf16" else 0


def _config(case):
    return dict(arch=case["arch"], n_layers=case["layers"], d_model=case["d"], n_heads=case["heads"], d_ffn=case["ffn"],
                vocab=case["vocab"], max_seq=case["positions"], n_classes=case["classes"], norm_eps=1e-5, rope_base=10000.0,
                dtype=_code(case))


def _opt(case):
    kind = "sgd" if case["opt"] == "sgdm" else case["opt"]
    return dict(kind=kind, lr=case["lr"], beta1=0.9, beta2=0.999, eps=1e-10 if kind == "adagrad" else 1e-8, weight_decay=case["wd"],
                momentum=0.9 if case["opt"] == "sgdm" else 0.0)


def _batches(case, g, n):
    """n batches: tokens by a bounded Zipf law for the rotary decoder, uniform otherwise; the next token or a class as label."""
    out = []
    b, s, v = case["batch"], case["seq"], case["vocab"]
    for _ in range(n):
        if case["arch"] == 2:
            cdf = torch.cumsum(torch.arange(1, v + 1, device="cuda", dtype=torch.float64) ** -1.1, 0)
            u = torch.rand(b, s, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
            tok = torch.searchsorted(cdf, u).clamp_(max=v - 1).to(torch.int32)
        else:
            tok = torch.randint(0, v, (b, s), generator=g, device="cuda", dtype=torch.int32)
        if case["arch"] == 1:
            lab = torch.randint(0, case["classes"], (b,), generator=g, device="cuda", dtype=torch.int32)
        else:
            lab = torch.full_like(tok, -1)
            lab[:, :-1] = tok[:, 1:]
        out.append((tok, lab))
    return out


def _weights(case, tensors, g):
    """Initial parameters unit by unit: matrices N(0, 0.02^2), gains around one, biases around zero, representable in bf16."""
    units = {}
    for _name, shape, kind, unit, _off in tensors:
        n = math.prod(shape)
        w = torch.randn(n, generator=g, device="cuda") * 0.02
        if kind == 1:
            w += 1.0
        units.setdefault(unit, []).append(w.to(torch.bfloat16).float())
    return [torch.cat(units[u]) for u in sorted(units)]


def _adapters(case, g):
    return _randn(g, case["layers"] * 4 * case["rank"] * case["d"], scale=0.02)


def _rope_table(seq, head_dim):
    p = torch.arange(seq, dtype=torch.float64, device="cuda")[:, None]
    i = torch.arange(head_dim // 2, dtype=torch.float64, device="cuda")[None, :]
    a = p * 10000.0 ** (-2.0 * i / head_dim)
    return torch.cos(a), torch.sin(a)


def _groups(case):
    n = case["layers"] + 2
    k = H.group_count(n, case["m"])
    return [list(range(j * case["m"], min((j + 1) * case["m"], n))) for j in range(k)]


def prepare(case, seed):
    g, kind, dt = _gen(seed), case["kind"], _dtype(case)
    if kind in ("sweep", "lora"):
        more = dict(lora_rank=case["rank"], lora_alpha=2.0 * case["rank"]) if kind == "lora" else {}
        model = H.HiftModel(_config(case), _opt(case), case["m"], case["batch"], case["seq"], state_on_host=int(case["parked"]), **more)
        for u, w in enumerate(_weights(case, model.tensors, g)):
            model.write_params_device(u, u + 1, w)
        s = {"case": case, "model": model}
        if kind == "lora":
            model.lora_write(_adapters(case, g).cpu().numpy())
            s["batches"] = _batches(case, g, case["steps"])
            return s
        s["k"] = model.set_group_schedule(case["strategy"], case["m"], 0)
        s["batches"] = _batches(case, g, s["k"])
        # the arena is the caller's memory: [fp32 master weights | forward copies | packed copies | gradient | optimizer state ...],
        # each as long as the memory report says, the parameters in canonical order
        rep = model.memory()
        base = -model.device_arena.data_ptr() % 256
        s["weights"] = model.device_arena[base:base + 4 * rep["n_params"]].view(torch.float32)
        if not case["parked"]:
            base += rep["device_master"] + rep["device_forward"] + rep["device_packed"] + rep["device_grad"]
            s["moment"] = model.device_arena[base:base + 4 * rep["n_params"]].view(torch.float32)
        return s
    if kind == "attention":
        b, h, n, e = case["batch"], case["heads"], case["seq"], case["head_dim"]
        s = {"case": case, "qkv": _randn(g, b * n, 3 * h * e, dtype=torch.bfloat16), "dctx": _randn(g, b * n, h * e, dtype=torch.bfloat16)}
        s["ctx"], s["dqkv"] = torch.empty_like(s["dctx"]), torch.empty_like(s["qkv"])
        s["lse"] = torch.empty(b, h, n, device="cuda")
        s["dsum"] = torch.empty(b, h, n, device="cuda")
        s["table"] = torch.stack(_rope_table(n, e), -1).float().contiguous() if case["rope"] else None
        return s
    if kind == "linear":
        r, i, o = case["rows"], case["inner"], case["outer"]
        s = {"case": case, "x": _randn(g, r, i, dtype=dt), "w": _randn(g, o, i, dtype=dt, scale=0.02), "dy": _randn(g, r, o, dtype=dt)}
        s["bias"] = _randn(g, o, dtype=dt, scale=0.5) if case["bias"] else None
        s["res"] = _randn(g, r, o, dtype=dt) if case["residual"] else None
        s["y"], s["dx"] = torch.empty_like(s["dy"]), torch.empty_like(s["x"])
        s["dw"] = torch.empty(o, i, device="cuda")
        if case["packed"]:
            s["wf"] = torch.empty(H.kernel_packed_bytes(o, i), device="cuda", dtype=torch.uint8)
            s["wb"] = torch.empty(H.kernel_packed_bytes(i, o), device="cuda", dtype=torch.uint8)
            H.kernel_pack_b(1, o, i, s["w"], i, s["wf"])
            H.kernel_pack_b(0, i, o, s["w"], i, s["wb"])
            s["ws"] = torch.zeros(H.kernel_packed_workspace_bytes(), device="cuda", dtype=torch.uint8)
        return s
    if kind == "cross_entropy":
        r, v = case["rows"], case["vocab"]
        lab = torch.randint(0, v, (r,), generator=g, device="cuda", dtype=torch.int32)
        lab[case["seq"] - 1::case["seq"]] = -1  # the last position of a sequence has no next token
        return {"case": case, "logits": _randn(g, r, v, dtype=dt, scale=2.0), "labels": lab,
                "scratch": torch.empty(r + 1, device="cuda"), "loss": torch.empty(1, device="cuda")}
    if kind == "optimizer":
        n = case["count"]
        s = {"case": case, "w": _randn(g, n, scale=0.02), "g": _randn(g, n, scale=1e-3)}
        s["s1"] = _randn(g, n, scale=1e-4)
        if case["opt"] == "adagrad":
            s["s1"].square_()
        s["s2"] = _randn(g, n, scale=1e-4).square_() if case["opt"] == "adamw" else None
        s["half"] = torch.empty(n, device="cuda", dtype=torch.bfloat16) if case["half"] else None
        return s
    r, d = case["rows"], case["d"]
    s = {"case": case, "x": _randn(g, r, d, dtype=dt), "g": (1.0 + _randn(g, d, scale=0.02)).to(dt), "b": _randn(g, d, dtype=dt, scale=0.02)}
    s["y"], s["stats"] = torch.empty_like(s["x"]), torch.empty(r, 2, device="cuda")
    return s


# ---- one pass ---------------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "sweep":
        losses = s["model"].train(s["batches"], s["k"], want_losses=case["losses"])
        out = {"weights": s["weights"]}
        if "moment" in s:
            out["moment"] = s["moment"]
        if losses is not None:
            out["losses"] = losses
        return out
    if kind == "lora":
        losses = [s["model"].lora_step(tok, lab, want_loss=case["losses"]) for tok, lab in s["batches"]]
        out = {"adapters": s["model"].lora_read(0), "moment": s["model"].lora_read(2)}
        if case["losses"]:
            out["losses"] = losses
        return out
    if kind == "attention":
        a = (case["batch"], case["heads"], case["seq"], case["head_dim"], case["causal"])
        H.kernel_attention_fwd(*a, s["qkv"], None, s["ctx"], s["lse"])
        H.kernel_attention_bwd(*a, s["qkv"], s["ctx"], s["lse"], s["dctx"], s["dsum"], s["dqkv"], s["table"])
        return {"ctx": s["ctx"], "lse": s["lse"], "dqkv": s["dqkv"]}
    if kind == "linear":
        r, i, o, dt = case["rows"], case["inner"], case["outer"], _code(case)
        if case["packed"]:
            H.kernel_gemm_packed_ws(0, r, o, i, s["x"], i, s["wf"], s["y"], o, s["bias"], s["res"], s["ws"])
            H.kernel_gemm_packed_ws(0, r, i, o, s["dy"], o, s["wb"], s["dx"], i, None, None, s["ws"])
        else:
            H.kernel_gemm(dt, 1, 1, 0, r, o, i, s["x"], i, s["w"], i, s["y"], o, s["bias"], s["res"])
            H.kernel_gemm(dt, 1, 0, 0, r, i, o, s["dy"], o, s["w"], i, s["dx"], i)
        H.kernel_gemm(dt, 0, 0, 1, o, i, r, s["dy"], o, s["x"], i, s["dw"], i)
        return {"y": s["y"], "dx": s["dx"], "dw": s["dw"]}
    if kind == "cross_entropy":
        # in place, as in a step; a pass after the first takes what the one before left, which costs the same
        H.kernel_cross_entropy(_code(case), case["rows"], case["vocab"], s["logits"], s["labels"], s["scratch"], s["loss"])
        return {"loss": s["loss"], "dlogits": s["logits"]}
    if kind == "optimizer":
        H.kernel_optimizer(_opt(case), case["count"], case["decay"], 3, s["w"], s["g"], s["s1"], s["s2"], s["half"])
        return {k: s[k] for k in ("w", "s1", "s2", "half") if s[k] is not None}
    H.kernel_norm_fwd(_code(case), case["rms"], case["rows"], case["d"], 1e-5, s["x"], s["g"], None if case["rms"] else s["b"], s["y"],
                      s["stats"])
    return {"y": s["y"], "stats": s["stats"]}


# ---- what a pass cannot do without --------------------------------------------------------------------------------
def _model_work(case):
    """(flops, bytes) of the forward pass, of the activation gradients and of the weight gradients of one hidden layer, and of the
    head; attention counts every key for the encoder and half of them under the causal mask."""
    d, f, v = case["d"], case["ffn"], case["vocab"]
    t = case["batch"] * case["seq"]
    e = 2 if case["dtype"] == "bf16" else 4
    lin = 4 * d * d + (3 if case["arch"] == 2 else 2) * d * f
    att = (4 if case["arch"] == 1 else 2) * t * case["seq"] * d
    head_rows = case["batch"] if case["arch"] == 1 else t
    head_cols = case["classes"] if case["arch"] == 1 else v
    acts = t * (8 * d + 3 * f)  # what a layer's backward pass reads again: written once
    return {"layer": (2 * t * lin + att, e * (lin + acts)), "layer_dx": (2 * t * lin + 2.5 * att, e * (lin + acts)),
            "layer_dw": (2 * t * lin, 4 * lin), "head": (2 * head_rows * d * head_cols, e * (head_cols * d + 2 * head_rows * head_cols)),
            "lin": lin, "head_params": head_cols * d}


def work(case):
    kind = case["kind"]
    if kind in ("sweep", "lora"):
        w, layers, top = _model_work(case), case["layers"], case["layers"] + 1
        flops = bytes_ = 0.0
        if kind == "lora":
            for _ in range(case["steps"]):
                for n, part in ((layers, "layer"), (layers, "layer_dx"), (2, "head")):
                    flops += n * w[part][0]
                    bytes_ += n * w[part][1]
            return {"flops": flops, "bytes": bytes_}
        words = {"adamw": 7, "sgdm": 5, "adagrad": 5}[case["opt"]]  # fp32 values read and written per parameter by the update
        per = 4 * words + (2 if case["dtype"] == "bf16" else 0)
        for units in _groups(case):
            lo = units[0]
            for u in units:  # weight gradients and update
                if 1 <= u <= layers:
                    flops += w["layer_dw"][0]
                    bytes_ += w["layer_dw"][1] + per * w["lin"]
                elif u == top:
                    flops += w["head"][0]
                    bytes_ += (4 + per) * w["head_params"]
                else:
                    bytes_ += (4 + per) * (case["vocab"] + (case["positions"] if case["arch"] != 2 else 0)) * case["d"]
            above = layers - max(lo, 1) + 1 if lo <= layers else 0  # layers that the backward pass crosses
            for n, part in ((layers, "layer"), (above, "layer_dx"), (2, "head")):
                flops += n * w[part][0]
                bytes_ += n * w[part][1]
        return {"flops": flops, "bytes": bytes_}
    if kind == "attention":
        b, h, n, e = case["batch"], case["heads"], case["seq"], case["head_dim"]
        pairs = b * h * (n * (n + 1) / 2 if case["causal"] else n * n)
        return {"flops": (4 + 10) * pairs * e, "bytes": 2 * b * n * h * e * (3 + 1 + 3 + 1 + 1 + 3) + 8 * b * h * n}
    if kind == "linear":
        r, i, o, e = case["rows"], case["inner"], case["outer"], 2 if case["dtype"] == "bf16" else 4
        res = r * o if case["residual"] else 0
        return {"flops": 6.0 * r * i * o, "bytes": e * (3 * r * i + 3 * r * o + 2 * i * o + res) + 4 * i * o}
    if kind == "cross_entropy":
        return {"flops": 0, "bytes": 2 * case["rows"] * case["vocab"] * (2 if case["dtype"] == "bf16" else 4)}
    if kind == "optimizer":
        return {"flops": 0, "bytes": case["count"] * (4 * {"adamw": 7, "sgdm": 5, "adagrad": 5}[case["opt"]] + (2 if case["half"] else 0))}
    return {"flops": 0, "bytes": 2 * case["rows"] * case["d"] * (2 if case["dtype"] == "bf16" else 4)}


def tolerance(case):
    kind, half = case["kind"], case.get("dtype") == "bf16"
    if kind == "sweep":
        if not half:
            # a key's bias has a gradient of zero but for rounding, and AdamW gives its noise the full step
            return {"rel": 5e-4, "max": 0.05}
        # weights alone (parked state): an update is at most lr a step, and its sign is rounding's where the gradient is nearly
        # zero; with the first moment: bf16 activations through every layer of the model
        return {"rel": 2e-4, "max": 0.05} if case["parked"] else {"rel": 0.03, "max": 1.0 - 1e-9}
    if kind == "lora":
        return {"rel": 0.03, "max": 1.0 - 1e-9}
    if kind == "attention":
        return {"rel": 0.015, "max": 0.3}
    if kind == "optimizer":
        return {"rel": 1e-4, "max": 0.01}  # a bf16 copy that rounds the other way at a tie is one of its units off
    return {"rel": 0.008, "max": 0.1} if half else {"rel": 1e-5, "max": 1e-3}


# ---- the same in 64 bits ------------------------------------------------------------------------------------------
def _norm64(x, g, b, rms):
    if rms:
        return x / torch.sqrt(x.square().mean(-1, keepdim=True) + 1e-5) * g
    mu = x.mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt((x - mu).square().mean(-1, keepdim=True) + 1e-5) * g + b


def _rotate64(x, cos, sin):
    a, b = x.chunk(2, -1)
    return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)


def _attend64(q, k, v, causal):
    """[B, H, S, e] each; the context and the natural logarithm of each row's sum of exponentials."""
    s = (q @ k.transpose(-1, -2)) / math.sqrt(q.shape[-1])
    if causal:
        s = s.masked_fill(torch.ones(s.shape[-2:], dtype=torch.bool, device=s.device).triu(1), float("-inf"))
    return torch.softmax(s, -1) @ v, torch.logsumexp(s, -1)


def _loss64(case, p, tok, lab, adapters=None):
    b, n, d, heads, arch = case["batch"], case["seq"], case["d"], case["heads"], case["arch"]
    rms, enc = arch == 2, arch == 1
    tok = tok.long()
    x = p["tok_emb"][tok]
    if not rms:
        x = x + p["pos_emb"][:n]
    if enc:
        x = _norm64(x, p["lne_g"], p["lne_b"], False)
    table = _rope_table(n, d // heads) if rms else None
    for l in range(case["layers"]):
        w = {k.split(".", 1)[1]: t for k, t in p.items() if k.startswith("l%d." % l)}
        h = x if enc else _norm64(x, w["g1" if rms else "ln1_g"], w.get("ln1_b"), rms)
        qkv = h @ w["wqkv"].T + w.get("bqkv", 0.0)
        q, k, v = qkv.split(d, -1)
        if adapters is not None:
            r = case["rank"]
            a = adapters[l * 4 * r * d:(l + 1) * 4 * r * d]
            aq, av, bq, bv = a[:r * d].view(r, d), a[r * d:2 * r * d].view(r, d), a[2 * r * d:3 * r * d].view(d, r), a[3 * r * d:].view(d, r)
            q, v = q + 2.0 * (h @ aq.T) @ bq.T, v + 2.0 * (h @ av.T) @ bv.T
        q, k, v = (t.view(b, n, heads, d // heads).transpose(1, 2) for t in (q, k, v))
        if rms:
            q, k = _rotate64(q, *table), _rotate64(k, *table)
        ctx = _attend64(q, k, v, not enc)[0].transpose(1, 2).reshape(b, n, d)
        x = x + ctx @ w["wo"].T + w.get("bo", 0.0)
        if enc:
            x = _norm64(x, w["ln1_g"], w["ln1_b"], False)
        h = x if enc else _norm64(x, w["g2" if rms else "ln2_g"], w.get("ln2_b"), rms)
        if rms:
            gate, up = (h @ w["wgu"].T).chunk(2, -1)
            x = x + (torch.nn.functional.silu(gate) * up) @ w["wd"].T
        else:
            x = x + torch.nn.functional.gelu(h @ w["w1"].T + w["b1"]) @ w["w2"].T + w["b2"]
        if enc:
            x = _norm64(x, w["ln2_g"], w["ln2_b"], False)
    if enc:
        return torch.nn.functional.cross_entropy(x[:, 0] @ p["wc"].T + p["bc"], lab.long())
    x = _norm64(x, p["gf" if rms else "lnf_g"], p.get("lnf_b"), rms)
    return torch.nn.functional.cross_entropy((x @ p["whead"].T).flatten(0, 1), lab.long().flatten(), ignore_index=-1)


def _update64(o, t, decay, w, g, s1, s2):
    """One update of w, s1, s2 in place; t counts the tensor's updates from 1."""
    wd = o["weight_decay"] if decay else 0.0
    if o["kind"] == "adamw":
        w.mul_(1.0 - o["lr"] * wd)
        s1.mul_(o["beta1"]).add_(g, alpha=1.0 - o["beta1"])
        s2.mul_(o["beta2"]).addcmul_(g, g, value=1.0 - o["beta2"])
        w.sub_(o["lr"] * (s1 / (1.0 - o["beta1"] ** t)) / ((s2 / (1.0 - o["beta2"] ** t)).sqrt_() + o["eps"]))
        return
    g = g + wd * w
    if o["kind"] == "adagrad":
        s1.addcmul_(g, g)
        w.sub_(o["lr"] * g / (s1.sqrt() + o["eps"]))
    else:
        s1.mul_(0.0 if t == 1 else o["momentum"]).add_(g)
        w.sub_(o["lr"] * s1)


def _forward_values(case, w):
    return w.float().to(torch.bfloat16).double() if case["dtype"] == "bf16" else w.float().double()


def exact(case, seed):
    g, kind = _gen(seed), case["kind"]
    if kind in ("sweep", "lora"):
        cfg, o = _config(case), _opt(case)
        tensors, _n = H.tensor_list(cfg)
        flat = torch.cat(_weights(case, tensors, g)).double()
        spans = {name: (off, math.prod(shape), shape, tkind, unit) for name, shape, tkind, unit, off in tensors}
        losses = []

        def view(x):
            return {name: x[off:off + n].view(shape) for name, (off, n, shape, _k, _u) in spans.items()}

        if kind == "lora":
            # the adapters pass through the host in 32 bits, as they do in prepare()
            a = _adapters(case, g).double()
            m, v = torch.zeros_like(a), torch.zeros_like(a)
            p = view(flat)
            for t, (tok, lab) in enumerate(_batches(case, g, case["steps"]), 1):
                leaf = _forward_values(case, a).requires_grad_()
                loss = _loss64(case, p, tok, lab, leaf)
                losses.append(float(loss))
                _update64(o, t, True, a, torch.autograd.grad(loss, leaf)[0], m, v)
            out = {"adapters": a, "moment": m}
        else:
            s1 = torch.zeros_like(flat)
            s2 = torch.zeros_like(flat) if case["opt"] == "adamw" else None
            groups = _groups(case)
            order = H.group_order(len(groups), case["strategy"], 0)
            half = _forward_values(case, flat)
            for gid, (tok, lab) in zip(order, _batches(case, g, len(groups))):
                mine = [name for name, sp in spans.items() if sp[4] in groups[gid]]
                p = view(half)
                for name in mine:
                    p[name] = p[name].clone().requires_grad_()
                loss = _loss64(case, p, tok, lab)
                losses.append(float(loss))
                grads = torch.autograd.grad(loss, [p[name] for name in mine], allow_unused=True)
                for name, gr in zip(mine, grads):
                    off, n, _shape, tkind, _unit = spans[name]
                    at = slice(off, off + n)
                    gr = torch.zeros(n, device="cuda", dtype=torch.float64) if gr is None else gr.reshape(-1)
                    _update64(o, 1, tkind == 0, flat[at], gr, s1[at], None if s2 is None else s2[at])
                    half[at] = _forward_values(case, flat[at])
            out = {"weights": flat}
            if not case["parked"]:
                out["moment"] = s1
        if case["losses"]:
            out["losses"] = torch.tensor(losses, dtype=torch.float64) if kind == "sweep" else losses
        return out
    s = prepare(case, seed)
    if kind == "attention":
        b, h, n, e = case["batch"], case["heads"], case["seq"], case["head_dim"]
        qkv = s["qkv"].double().requires_grad_()
        q, k, v = (t.reshape(b, n, h, e).transpose(1, 2) for t in qkv.split(h * e, -1))
        ctx, lse = _attend64(q, k, v, case["causal"])
        ctx = ctx.transpose(1, 2).reshape(b * n, h * e)
        d = torch.autograd.grad(ctx, qkv, s["dctx"].double())[0]
        if case["rope"]:  # q and k count as rotated; their gradients are turned back
            cos, sin = (t[None, :, None, :] for t in _rope_table(n, e))
            d = d.view(b, n, 3, h, e).clone()
            for j in range(2):
                d[:, :, j] = _rotate64(d[:, :, j], cos, -sin)
            d = d.view(b * n, 3 * h * e)
        return {"ctx": ctx.detach(), "lse": lse.detach() / math.log(2.0), "dqkv": d}
    if kind == "linear":
        x, w, dy = (s[k].double() for k in ("x", "w", "dy"))
        y = x @ w.T
        if s["bias"] is not None:
            y += s["bias"].double()
        if s["res"] is not None:
            y += s["res"].double()
        return {"y": y, "dx": dy @ w, "dw": dy.T @ x}
    if kind == "cross_entropy":
        lab = s["labels"].long()
        on = lab >= 0
        z = s["logits"].double()
        n = max(1, int(on.sum()))
        lse = torch.logsumexp(z, -1, keepdim=True)
        at = lab.clamp(min=0)[:, None]
        loss = ((lse - z.gather(1, at))[:, 0] * on).sum() / n
        z = torch.exp(z - lse)
        z.scatter_add_(1, at, torch.full_like(at, -1, dtype=torch.float64))
        return {"loss": loss.reshape(1), "dlogits": z * (on[:, None] / n)}
    if kind == "optimizer":
        w, gr, s1 = s["w"].double(), s["g"].double(), s["s1"].double()
        s2 = None if s["s2"] is None else s["s2"].double()
        _update64(_opt(case), 3, case["decay"], w, gr, s1, s2)
        # (the bf16 copy of the new weights is a rounding of them: no value of its own)
        return {k: t for k, t in (("w", w), ("s1", s1), ("s2", s2)) if t is not None}
    x = s["x"].double()
    mu = x.mean(-1) if not case["rms"] else torch.zeros(case["rows"], device="cuda", dtype=torch.float64)
    rstd = 1.0 / torch.sqrt((x - mu[:, None]).square().mean(-1) + 1e-5)
    y = (x - mu[:, None]) * rstd[:, None] * s["g"].double()
    return {"y": y if case["rms"] else y + s["b"].double(), "stats": torch.stack([mu, rstd], -1)}
