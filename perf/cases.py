"""The workloads whose speed is measured, as calls of the public API on synthetic data.

One case is one piece of the work a fast worker, or the process that drives all workers, does in a communication round:
the whole pass of a worker (score, select, train, aggregate), its parts at the sizes where they are run alone, and the
epoch's sampling.  Networks and sizes are those of synth.WORKLOADS and bench.py; random-init weights of those
architectures, images normalised to unit scale with class means, token sequences with a Zipf law.
"""
import math

import torch

import paper_2508_08540_amd as bls

# 8 fast workers with 32 local steps and 2 slow ones with 16 per round
TAU_WORKERS = (32,) * 8 + (16,) * 2

_context = []


def _ctx():
    """The one context of a program: current device, current stream."""
    if not _context:
        _context.append(bls.Context(0))
    return _context[0]


def listed():
    return [
        # The smallest call: the MLP, a pool of 256, four steps of 64.  Every launch is latency.
        dict(name="mlp_pass", kind="pass", net="mlp", hidden=128, act="f32", classes=10, pool=256, k=64, batch=64, tau=4, replicas=4,
             lr=0.1, mu=0.0, wd=0.0),
        # The headline workload: a fast worker's whole pass on ResNet20 in fp32.
        dict(name="resnet20_f32_pass", kind="pass", net="resnet", blocks=3, act="f32", classes=10, pool=512, k=128, batch=128, tau=20,
             replicas=10, lr=0.001, mu=0.9, wd=0.0),
        # Mixed precision: one walk through 1024 selected samples.
        dict(name="resnet20_bf16_train", kind="train", net="resnet", blocks=3, act="bf16", classes=10, k=1024, batch=128, tau=8, lr=0.01,
             mu=0.9, wd=0.0),
        # One communication round of eight fast and two slow workers with the batch size and weight decay of the ResNet20
        # runs; ragged shares of the pool.
        dict(name="resnet20_round", kind="round", net="resnet", blocks=3, act="f32", classes=10, pool=9999, workers=10, tau=16,
             tau_slow=8, batch=32, lr=0.001, mu=0.9, wd=1e-4),
        # The wide network: inference over a pool that is no multiple of anything, and training.
        dict(name="wrn_bf16_score", kind="score", net="wrn", blocks=2, act="bf16", classes=100, pool=2001),
        dict(name="wrn_bf16_train", kind="train", net="wrn", blocks=2, act="bf16", classes=100, k=512, batch=128, tau=4, lr=0.05, mu=0.9,
             wd=0.0),
        # The language model: inference (no gradient, logits never leave the chip) and training in mixed precision.
        dict(name="encoder_bf16_score", kind="score", net="encoder", layers=6, seq=128, vocab=32000, act="bf16", pool=1024),
        dict(name="encoder_bf16_train", kind="train", net="encoder", layers=6, seq=128, vocab=32000, act="bf16", k=256, batch=64, tau=4,
             lr=0.001, mu=0.9, wd=0.0),
        # The same in fp32, an odd batch of sequences that are no multiple of a tile.
        dict(name="encoder_f32_train", kind="train", net="encoder", layers=6, seq=100, vocab=32000, act="f32", k=62, batch=31, tau=2,
             lr=0.001, mu=0.9, wd=0.0),
        # The sampler at the top of an epoch of 50 000 samples, half of the fast allocation by loss.
        dict(name="sample_epoch_50k", kind="sample", n=50000, tau_f=32, p_f=8, tau_s=1, p_s=2, lam=0.5, scheme="separated"),
        # Selection from a very large pool.
        dict(name="topk_16m", kind="topk", n=16000001, k=4000000, values="halfnormal"),
        # The aggregation of ten replicas of the wide network.
        dict(name="aggregate_wrn", kind="aggregate", d=11007540, replicas=10, broadcast=False),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("mlp_pass", "resnet_pass", "resnet_train", "round", "wrn_score", "wrn_train", "encoder_score", "encoder_train",
                       "encoder_f32_train", "sample", "topk", "aggregate"))
    if kind == "mlp_pass":
        b = _log_int(rng, 8, 256)
        return dict(kind="pass", net="mlp", hidden=16 * rng.randint(2, 16), act="f32", classes=rng.randint(2, 64),
                    pool=max(b, _log_int(rng, 64, 1024)), k=b, batch=b, tau=rng.randint(1, 8), replicas=rng.randint(2, 10), lr=0.1, mu=0.9,
                    wd=0.0)
    if kind == "resnet_pass":
        b = _log_int(rng, 16, 160)
        return dict(kind="pass", net="resnet", blocks=rng.randint(1, 3), act="f32", classes=10, pool=max(b, _log_int(rng, 100, 1024)), k=b,
                    batch=b, tau=rng.randint(1, 12), replicas=rng.randint(2, 10), lr=0.001, mu=0.9, wd=1e-4)
    if kind == "resnet_train":
        return dict(kind="train", net="resnet", blocks=rng.randint(1, 3), act="bf16", classes=10, k=_log_int(rng, 64, 1024),
                    batch=_log_int(rng, 16, 160), tau=rng.randint(1, 8), lr=0.01, mu=0.9, wd=1e-4)
    if kind == "round":
        w = rng.randint(2, 10)
        return dict(kind="round", net="resnet", blocks=rng.randint(1, 3), act="f32", classes=10, pool=_log_int(rng, 1000, 9999), workers=w,
                    tau=rng.randint(2, 16), tau_slow=rng.randint(1, 8), batch=_log_int(rng, 8, 32), lr=0.001, mu=0.9, wd=1e-4)
    if kind == "wrn_score":
        return dict(kind="score", net="wrn", blocks=rng.randint(1, 2), act="bf16", classes=rng.randint(10, 100), pool=_log_int(rng, 50, 2000))
    if kind == "wrn_train":
        return dict(kind="train", net="wrn", blocks=rng.randint(1, 2), act="bf16", classes=rng.randint(10, 100), k=_log_int(rng, 64, 512),
                    batch=_log_int(rng, 16, 128), tau=rng.randint(1, 4), lr=0.05, mu=0.9, wd=1e-4)
    if kind == "encoder_score":
        return dict(kind="score", net="encoder", layers=rng.randint(1, 6), seq=rng.randint(32, 128), vocab=_log_int(rng, 2000, 32000),
                    act="bf16", pool=_log_int(rng, 16, 1024))
    if kind in ("encoder_train", "encoder_f32_train"):
        f32 = kind == "encoder_f32_train"
        return dict(kind="train", net="encoder", layers=rng.randint(1, 6), seq=rng.randint(32, 100 if f32 else 128),
                    vocab=_log_int(rng, 2000, 32000), act="f32" if f32 else "bf16", k=_log_int(rng, 32, 256),
                    batch=_log_int(rng, 4, 31 if f32 else 64), tau=rng.randint(1, 2 if f32 else 4), lr=0.001, mu=0.9, wd=0.0)
    if kind == "sample":
        return dict(kind="sample", n=_log_int(rng, 2000, 1 << 20), tau_f=rng.randint(4, 64), p_f=rng.randint(1, 8), tau_s=rng.randint(1, 4),
                    p_s=rng.randint(1, 4), lam=round(rng.uniform(0.1, 1.0), 3), scheme=rng.choice(("separated", "unified")))
    if kind == "topk":
        n = _log_int(rng, 512, 16000001)
        return dict(kind="topk", n=n, k=max(1, int(n * rng.uniform(0.02, 1.0) ** 2)), values=rng.choice(("halfnormal", "ties")))
    return dict(kind="aggregate", d=_log_int(rng, 20000, 11007540), replicas=rng.randint(2, 10), broadcast=rng.random() < 0.3)


# ---- what a program has in hand before the call ----------------------------------------------------------------------


def _model(case):
    if case["net"] == "mlp":
        return bls.Model.mlp(hidden=case["hidden"], classes=case["classes"])
    if case["net"] == "resnet":
        return bls.Model.resnet_cifar(blocks=case["blocks"], classes=case["classes"], act_dtype=case["act"])
    if case["net"] == "wrn":
        return bls.Model.wide_resnet(blocks=case["blocks"], classes=case["classes"], act_dtype=case["act"])
    return bls.Model.transformer(vocab=case["vocab"], seq_len=case["seq"], layers=case["layers"], act_dtype=case["act"])


def _init(model, gen):
    """(parameters, buffers): He-normal convolutions, uniform +-1/sqrt(fan_in) linear layers, normalisation scales around 1."""
    p = torch.zeros(model.num_params, device="cuda")
    b = torch.zeros(max(model.num_buffers, 1), device="cuda")
    for t in model.tensors:
        shape, name = t["shape"], t["name"]
        n = math.prod(shape)
        if t["is_buffer"]:
            u = torch.rand(n, device="cuda", generator=gen)
            b[t["offset"]:t["offset"] + n] = 1.0 + 0.2 * u if name.endswith("var") else 0.2 * u - 0.1
            continue
        if len(shape) == 4:
            v = torch.randn(n, device="cuda", generator=gen) * math.sqrt(2.0 / (shape[0] * shape[1] * shape[2]))
        elif name.endswith("emb.weight"):
            v = 0.02 * torch.randn(n, device="cuda", generator=gen)
        elif len(shape) == 2:
            v = (2.0 * torch.rand(n, device="cuda", generator=gen) - 1.0) / math.sqrt(shape[1])
        else:
            v = 0.1 * (2.0 * torch.rand(n, device="cuda", generator=gen) - 1.0)
            if name.endswith(".weight"):
                v = v + 1.0
        p[t["offset"]:t["offset"] + n] = v
    return p, b


def _pool(case, n, gen):
    if case["net"] == "encoder":
        ranks = torch.arange(1, case["vocab"] + 1, device="cuda", dtype=torch.float64)
        cdf = torch.cumsum(ranks ** -1.1, 0)
        u = torch.rand(n, case["seq"] + 1, device="cuda", generator=gen, dtype=torch.float64) * cdf[-1]
        ids = torch.searchsorted(cdf, u).clamp_(max=case["vocab"] - 1).to(torch.int32)
        return ids[:, :-1].contiguous(), ids[:, 1:].contiguous()
    y = torch.randint(case["classes"], (n,), device="cuda", generator=gen)
    mean = 0.5 * torch.randn(case["classes"], 32, 32, 3, device="cuda", generator=gen)
    x = torch.randn(n, 32, 32, 3, device="cuda", generator=gen)
    for i in range(0, n, 4096):
        x[i:i + 4096] += mean[y[i:i + 4096]]
    return x, y.to(torch.int32)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)
    kind = case["kind"]
    s = dict(case=case, ctx=_ctx())
    if kind == "topk":
        v = torch.randn(case["n"], device="cuda", generator=gen).abs_() + math.log(10.0)
        s["losses"] = torch.round(v * 64.0) / 64.0 if case["values"] == "ties" else v
        s["idx"] = torch.empty(case["k"], dtype=torch.int32, device="cuda")
        s["val"] = torch.empty(case["k"], device="cuda")
    elif kind == "sample":
        n_f, _, n_s = bls.epoch_allocation(case["n"], case["tau_f"], case["p_f"], case["tau_s"], case["p_s"], case["lam"])
        s["losses"] = torch.randn(case["n"], device="cuda", generator=gen).abs_() + math.log(10.0)
        s["u_fast"] = torch.rand(case["n"], device="cuda", generator=gen)
        s["u_slow"] = torch.rand(case["n"], device="cuda", generator=gen)
        s["fast"] = torch.empty(n_f, dtype=torch.int32, device="cuda")
        s["slow"] = torch.empty(n_s, dtype=torch.int32, device="cuda")
    elif kind == "aggregate":
        base = torch.randn(case["d"], device="cuda", generator=gen)
        s["replicas"] = [base + 0.01 * torch.randn(case["d"], device="cuda", generator=gen) for _ in range(case["replicas"])]
        s["weights"] = bls.weights_from_tau(TAU_WORKERS[-case["replicas"]:])
        s["out"] = torch.empty_like(base)
    else:
        m = s["model"] = _model(case)
        s["p0"], s["b0"] = _init(m, gen)
        s["b"] = torch.empty_like(s["b0"]) if m.num_buffers else None
        n = case["pool"] if "pool" in case else 2 * case["k"]
        s["x"], s["y"] = _pool(case, n, gen)
        if kind in ("pass", "score"):
            s["losses"] = torch.empty(n, device="cuda")
        if kind in ("pass", "train"):
            s["p"], s["m"] = torch.empty_like(s["p0"]), torch.empty_like(s["p0"])
            s["step_losses"] = torch.empty(case["tau"] * case["batch"], device="cuda")
        if kind == "train":
            s["idx"] = torch.randperm(n, device="cuda", generator=gen)[:case["k"]].to(torch.int32)
        if kind == "pass":
            s["idx"] = torch.empty(case["k"], dtype=torch.int32, device="cuda")
            s["others"] = [s["p0"] + 0.01 * torch.randn(m.num_params, device="cuda", generator=gen) for _ in range(case["replicas"] - 1)]
            s["weights"] = bls.weights_from_tau(TAU_WORKERS[-case["replicas"]:])
            s["out"] = torch.empty_like(s["p0"])
        if kind == "round":
            w = case["workers"]
            order = torch.randperm(n, device="cuda", generator=gen).to(torch.int32)
            s["gp"], s["gb"] = torch.empty_like(s["p0"]), torch.empty_like(s["b0"])
            s["wp"], s["wb"], s["wm"] = (torch.empty(w, t.numel(), device="cuda") for t in (s["p0"], s["b0"], s["p0"]))
            s["table0"] = torch.rand(n, device="cuda", generator=gen)
            s["table"] = torch.empty(n, device="cuda")
            s["workers"] = []
            for i in range(w):
                off, cnt = bls.worker_share(n, w, i)
                s["workers"].append(dict(tau=case["tau"] if 5 * i < 4 * w else case["tau_slow"], idx=order[off:off + cnt].clone(),
                                         params=s["wp"][i], buffers=s["wb"][i], momentum=s["wm"][i]))
    return s


def run(s):
    case, ctx, kind = s["case"], s["ctx"], s["case"]["kind"]
    if kind == "topk":
        bls.topk_by_loss(ctx, s["losses"], case["k"], s["idx"], s["val"])
        return s["idx"], s["val"]
    if kind == "sample":
        if case["scheme"] == "separated":
            bls.sample_epoch(ctx, s["losses"], s["u_fast"], s["u_slow"], case["tau_f"], case["p_f"], case["tau_s"], case["p_s"], case["lam"],
                             s["fast"], s["slow"])
        else:
            bls.sample_epoch(ctx, s["losses"], s["u_fast"], s["u_slow"], case["tau_f"], case["p_f"], case["tau_s"], case["p_s"], case["lam"],
                             s["fast"], s["slow"], scheme=case["scheme"], high_loss_to="fast")
        return s["fast"], s["slow"]
    if kind == "aggregate":
        bls.weighted_aggregate(ctx, s["replicas"], s["weights"], s["out"], bls.AGG_BROADCAST if case["broadcast"] else 0)
        return s["out"]
    model, x, y = s["model"], s["x"], s["y"]
    if kind == "score":
        return bls.score_losses(ctx, model, s["p0"], s["b0"] if model.num_buffers else None, x, y, s["losses"])
    # a round starts from the global model
    if kind == "round":
        s["gp"].copy_(s["p0"])
        s["gb"].copy_(s["b0"])
        s["wm"].zero_()
        s["table"].copy_(s["table0"])
        bls.communication_round(ctx, model, s["gp"], s["gb"], s["workers"], x, y, case["batch"], case["lr"], case["mu"], case["wd"], s["table"])
        return s["gp"], s["gb"], s["wp"], s["wb"], s["wm"], s["table"]
    s["p"].copy_(s["p0"])
    s["m"].zero_()
    if model.num_buffers:
        s["b"].copy_(s["b0"])
    if kind == "pass":
        bls.score_losses(ctx, model, s["p"], s["b"], x, y, s["losses"])
        bls.topk_by_loss(ctx, s["losses"], case["k"], s["idx"])
    bls.local_step(ctx, model, s["p"], s["b"], s["m"], x, y, s["idx"], case["batch"], case["tau"], case["lr"], case["mu"], case["wd"],
                   s["step_losses"])
    # The gradients of a bf16 convolution network are as sensitive to single roundings as they are large (momentum moves by
    # 10-30 % when the parameters move by one unit in the last place): its updated weights are the result, without momentum.
    trained = (s["step_losses"], s["p"])
    if case["net"] in ("mlp", "encoder") or case["act"] == "f32":
        trained += (s["m"],)
    if model.num_buffers:
        trained += (s["b"],)
    if kind == "train":
        return trained
    bls.weighted_aggregate(ctx, [s["p"]] + s["others"], s["weights"], s["out"])
    return (s["losses"], s["idx"]) + trained + (s["out"],)


# ---- what one pass cannot do without -----------------------------------------------------------------------------------


def _network(case):
    """(parameters, forward flops of a sample, flops of a sample's backward pass, bytes of a sample)."""
    if case["net"] == "mlp":
        fwd = 2 * (3072 * case["hidden"] + case["hidden"] * case["classes"])
        return 3072 * case["hidden"] + case["hidden"] * case["classes"], fwd, fwd + 2 * case["hidden"] * case["classes"], 4 * 3072 + 4
    if case["net"] == "encoder":
        d, f, t = 512, 2048, case["seq"]
        lin = case["layers"] * (4 * d * d + 2 * d * f) + case["vocab"] * d
        att = 4 * t * d * case["layers"]
        return lin + case["vocab"] * d, t * (2 * lin + att), t * (4 * lin + 2 * att), 8 * t
    if case["net"] == "resnet":
        widths, stem, shortcut = (16, 32, 64), 16, False
    else:
        widths, stem, shortcut = (128, 256, 512), 16, True
    h, c = 32, stem
    first = 2 * 9 * 3 * stem * h * h
    params, fwd = 27 * stem, first
    for i, w in enumerate(widths):
        for b in range(case["blocks"]):
            h = h // 2 if b == 0 and i > 0 else h
            macs = 9 * c * w + 9 * w * w + (c * w if shortcut and b == 0 else 0)
            params += macs
            fwd += 2 * macs * h * h
            c = w
    return params + c * case["classes"], fwd, 2 * fwd - first, 4 * 3072 + 4


def work(case):
    kind = case["kind"]
    if kind == "topk":
        return {"bytes": 4 * case["n"] + 8 * case["k"], "flops": 0}
    if kind == "sample":
        n_f, _, n_s = bls.epoch_allocation(case["n"], case["tau_f"], case["p_f"], case["tau_s"], case["p_s"], case["lam"])
        return {"bytes": 12 * case["n"] + 4 * (n_f + n_s), "flops": 0}
    if kind == "aggregate":
        r = case["replicas"]
        return {"bytes": 4 * case["d"] * (r + 1 + (r if case["broadcast"] else 0)), "flops": 2 * r * case["d"]}
    params, fwd, bwd, sample = _network(case)
    if kind == "score":
        return {"bytes": 4 * params + case["pool"] * (sample + 4), "flops": fwd * case["pool"]}
    if kind == "round":
        w = case["workers"]
        fast = sum(1 for i in range(w) if 5 * i < 4 * w)
        seen = (fast * case["tau"] + (w - fast) * case["tau_slow"]) * case["batch"]
        # every worker: replica and momentum out, momentum in; the global model in and out
        return {"bytes": 4 * params * (3 * w + 2) + min(seen, case["pool"]) * sample + 4 * seen, "flops": (fwd + bwd) * seen}
    seen = case["tau"] * case["batch"]
    out = {"bytes": 16 * params + min(seen, case["k"]) * sample + 4 * seen, "flops": (fwd + bwd) * seen}
    if kind == "pass":
        out["bytes"] += case["pool"] * (sample + 4) + 4 * case["k"] + 4 * params * case["replicas"]
        out["flops"] += fwd * case["pool"]
    return out


def tolerance(case):
    """Four times what was measured when the parameters move by one unit in the last place, or the samples of every batch
    are taken in another order.  The step sizes of the residual networks are those late in the schedule (fp32 0.001, bf16
    0.01): at 0.1 from a random start rounding differences grow tenfold every few steps."""
    kind = case["kind"]
    if kind in ("topk", "sample"):
        return "exact"
    if kind == "aggregate":
        return {"rel": 1e-6, "max": 1e-5}
    if case["net"] == "mlp":
        return {"rel": 1e-2, "max": 0.5, "differ": 0.01}   # 1e-7, unless a hidden unit crosses its kink: 2.4e-3
    if case["net"] == "encoder":
        if case["act"] == "f32":
            return {"rel": 4e-6, "max": 5e-4}
        return {"rel": 1e-4, "max": 1e-3} if kind == "score" else {"rel": 9e-4, "max": 0.1}
    if case["net"] == "wrn":
        if kind == "score":
            return {"rel": 1e-3, "max": 5e-3}
        return {"rel": 2e-3, "max": 0.25} if case["batch"] >= 64 else {"rel": 5e-3, "max": 0.6}
    if case["act"] == "bf16":
        return {"rel": 6e-3, "max": 0.1}
    # the momentum, the last gradients above all; a round takes more steps, on smaller batches
    return {"rel": 2.7e-2, "max": 1.0 - 1e-6} if kind == "round" else {"rel": 5e-3, "max": 0.2, "differ": 0.01}
