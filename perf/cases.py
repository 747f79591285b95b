"""The work that users of the elbow-routed MoE layer have it do, as timed cases.

Three kinds of case, each through the binding's public calls:

* ``layer``: one MoE layer call (router, elbow or top-K routing, dispatch, expert SwiGLU MLPs,
  combine): a decode step, a small or ragged prefill batch, a large prefill batch, in bf16 on
  OLMoE-shaped or other dimensions, or in fp32 on small ones;
* ``routing``: routing of given logits and the dispatch built from it, for a program that runs
  its experts itself;
* ``diagnostics``: the elbow angle of given logits and the tail-randomised routing.

Layer inputs follow ``synth``: x ~ N(0, 1), weights ~ N(0, 0.02).  Logits of the other two
kinds are noise with a few planted experts per token, sharp and gradual elbows mixed.
"""
import math

import torch

from paper_2608_04401_amd import binding as B

EPS = 1e-8


def _layer(name, T, d=2048, N=64, m=1024, K=8, dtype="bf16", mode="elbow", renormalize=False,
           residual=False, packed=False):
    return {"name": name, "kind": "layer", "T": T, "d": d, "N": N, "m": m, "K": K,
            "dtype": dtype, "mode": mode, "renormalize": renormalize, "residual": residual,
            "packed": packed}


def _logits(name, kind, T, N=64, K=8, renormalize=False):
    return {"name": name, "kind": kind, "T": T, "N": N, "K": K, "renormalize": renormalize}


def listed():
    return [
        # one sequence generating a token: the smallest call, eight experts' weights at most
        _layer("decode_1", 1, residual=True),
        # a decode step of a serving batch, row-major weights as a checkpoint holds them
        _layer("decode_40", 40, renormalize=True, residual=True),
        # the benchmark's decode layer, with the packed weight copy a server keeps
        _layer("decode_64_packed", 64, packed=True),
        # a chunk of chunked prefill, or a large decode batch: every expert has a few dozen rows
        _layer("chunk_512", 512, residual=True),
        # a ragged prompt batch, fixed top-K routing with renormalised weights
        _layer("ragged_1777_topk", 1777, mode="topk", renormalize=True),
        # the benchmark's prefill layer, and the fixed top-K baseline it is compared with
        _layer("prefill_4096", 4096),
        _layer("prefill_4096_topk", 4096, mode="topk"),
        # one layer of the residual stack at its batch size: the largest call
        _layer("stack_16384", 16384, residual=True),
        # the tiny fp32 layer of the tests, and a small fp32 model's layer with odd sizes
        _layer("f32_tiny_256", 256, d=128, N=8, m=256, dtype="f32"),
        _layer("f32_small_1500", 1500, d=1024, N=16, m=528, K=4, dtype="f32", residual=True),
        # routing and dispatch of a large batch for a program with its own experts
        _logits("routing_65536", "routing", 65536),
        # the analysis of a large batch: elbow angles and the tail-randomised routing
        _logits("diagnostics_65536", "diagnostics", 65536),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    r = rng.random()
    if r < 0.65:  # bf16 layers
        if rng.random() < 0.5:
            d, N, m = 2048, 64, 1024
        else:
            d, m = 64 * rng.randint(8, 40), 64 * rng.randint(4, 24)
            N = rng.choice([8, 16, 32, 48, 60, 64])
        K = rng.choice([1, 2, 4, 6, 8, 8, 8]) if N > 8 else rng.choice([1, 2, 4])
        top = min(16384, int(16384 * 2048 * 1024 * 8 / (d * m * K)))
        T = min(_log_int(rng, 1, 16384), top)
        c = _layer(None, T, d, N, m, K, mode=rng.choice(["elbow", "elbow", "topk"]),
                   renormalize=rng.random() < 0.5, residual=rng.random() < 0.5,
                   packed=T <= 256 and rng.random() < 0.4)
    elif r < 0.8:  # fp32 layers
        N = rng.choice([8, 16, 32])
        c = _layer(None, _log_int(rng, 1, 2048), 16 * rng.randint(8, 64), N,
                   16 * rng.randint(8, 40), rng.randint(1, min(N, 8)), dtype="f32",
                   mode=rng.choice(["elbow", "topk"]), renormalize=rng.random() < 0.5,
                   residual=rng.random() < 0.5)
    else:
        N = rng.choice([8, 16, 24, 32, 48, 60, 64, 64])
        K = rng.choice([2, 4, 8, 8, N])
        c = _logits(None, "routing" if r < 0.9 else "diagnostics",
                    _log_int(rng, 64, 262144) | rng.randint(0, 1), N, min(K, N),
                    rng.random() < 0.5)
    del c["name"]
    return c


def _normal(gen, shape, std, dtype):
    return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)


def _planted(gen, T, N):
    """N(0, 1) logits with one shared offset of 2 to 6 on 1 to 8 experts per token."""
    noise = torch.randn((T, N), generator=gen, device="cuda")
    count = torch.randint(1, min(8, N - 1) + 1, (T, 1), generator=gen, device="cuda")
    offset = torch.rand((T, 1), generator=gen, device="cuda") * 4 + 2
    rank = torch.rand((T, N), generator=gen, device="cuda").argsort(1).argsort(1)
    return noise + offset * (rank < count)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = {"case": case}
    T, N = case["T"], case["N"]
    if case["kind"] == "layer":
        d, m = case["d"], case["m"]
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        s["x"] = _normal(gen, (T, d), 1.0, dt)
        s["router"] = _normal(gen, (N, d), 0.02, dt)
        s["gate_up"] = _normal(gen, (N, 2 * m, d), 0.02, dt)
        s["down"] = _normal(gen, (N, d, m), 0.02, dt)
        s["residual"] = _normal(gen, (T, d), 1.0, dt) if case["residual"] else None
        s["packed"] = (B.elb_pack_expert_weights(s["gate_up"], s["down"]) if case["packed"]
                       else None)
    else:
        s["logits"] = _planted(gen, T, N)
        if case["kind"] == "diagnostics":
            s["rand"] = torch.rand((T, N), generator=gen, device="cuda")
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "layer":
        return B.elb_moe_forward(
            s["x"], s["router"], s["gate_up"], s["down"], K=c["K"], eps=EPS,
            mode=B.MODE_ELBOW if c["mode"] == "elbow" else B.MODE_TOPK,
            renormalize=c["renormalize"], residual=s["residual"], packed=s["packed"])
    if c["kind"] == "routing":
        k, ids, w = B.elb_route(s["logits"], c["K"], EPS, renormalize=c["renormalize"])
        return (k, ids, w) + tuple(B.elb_dispatch(k, ids, c["N"]))
    e, theta = B.elb_elbow_angle(s["logits"], EPS)
    k, ids, w = B.elb_route_tail_random(s["logits"], s["rand"], c["K"], EPS,
                                        renormalize=c["renormalize"])
    return e, theta, k, ids, w


def _mean_k(c):
    """Experts per token: K, or the mean of min(e + 1, K) over a sample of logits."""
    if c.get("mode") == "topk":
        return float(c["K"])
    gen = torch.Generator()
    gen.manual_seed(0)
    std = 0.02 * math.sqrt(c["d"]) if c["kind"] == "layer" else 1.0
    logits = torch.randn((2048, c["N"]), generator=gen, dtype=torch.float64) * std
    return float(_route64(logits, c["K"], "elbow", False)[0].double().mean())


def work(case):
    T, N, K = case["T"], case["N"], case["K"]
    if case["kind"] == "layer":
        d, m = case["d"], case["m"]
        size = 2 if case["dtype"] == "bf16" else 4
        k = _mean_k(case)
        used = N * (1.0 - (1.0 - k / N) ** T)  # experts with at least one token
        rows = T * d * (3 if case["residual"] else 2)
        return {"bytes": size * (used * 3 * m * d + N * d + rows),
                "flops": T * (6.0 * d * m * k + 2.0 * d * N)}
    if case["kind"] == "routing":  # logits in; k, ids, w, row_token and inv out
        return {"bytes": T * (4 * N + 4 + 16 * K), "flops": T * N * math.log2(N)}
    return {"bytes": T * (8 * N + 8 + 4 + 8 * K), "flops": T * N * math.log2(N)}


def tolerance(case):
    # bf16 layers round the activations and the expert outputs to 8 bits of mantissa (against
    # 64 bits: about 2.5e-3); fp32 layers sum a few thousand products (about 5e-7); routing
    # weights are a softmax in fp32 (about 1e-7), and ids and counts are whole numbers
    if case["kind"] == "layer":
        return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 2e-6}
    return {"rel": 5e-7}


def _elbow64(logits):
    """(sorted probabilities, their expert ids, deviations, elbow index) in 64 bits."""
    p, order = torch.softmax(logits, 1).sort(dim=1, descending=True, stable=True)
    n = p.shape[1]
    x = torch.arange(n, dtype=torch.float64, device=p.device) / (n - 1)
    curve = (p[:, :1] - p) / (p[:, :1] - p[:, -1:] + EPS)
    dev = curve - x
    first = torch.arange(n, device=p.device).expand_as(dev)
    e = torch.where(dev == dev.max(1, keepdim=True).values, first, n).min(1).values
    return p, order, curve, e


def _route64(logits, K, mode, renormalize):
    p, order, _, e = _elbow64(logits)
    k = (e + 1).clamp(max=K) if mode == "elbow" else torch.full_like(e, K)
    used = torch.arange(K, device=p.device) < k[:, None]
    w = torch.where(used, p[:, :K], 0.0)
    if renormalize:
        w = w / w.sum(1, keepdim=True)
    ids = torch.where(used, order[:, :K], -1)
    return k, ids, w


def _exact_layer(c, s):
    x = s["x"].double()
    k, ids, w = _route64(x @ s["router"].double().t(), c["K"], c["mode"], c["renormalize"])
    y = s["residual"].double() if s["residual"] is not None else torch.zeros_like(x)
    m = c["m"]
    for e in range(c["N"]):
        t, j = (ids == e).nonzero(as_tuple=True)
        if t.numel() == 0:
            continue
        h = x[t] @ s["gate_up"][e].double().t()
        h = torch.nn.functional.silu(h[:, :m]) * h[:, m:]
        y.index_add_(0, t, w[t, j, None] * (h @ s["down"][e].double().t()))
    return y


def _exact_dispatch(ids, N):
    T, K = ids.shape
    flat = ids.reshape(-1)
    used = (flat >= 0).nonzero().reshape(-1)
    expert, order = flat[used].sort(stable=True)
    slots = used[order]
    counts = torch.bincount(expert, minlength=N)
    offsets = torch.zeros(N + 1, dtype=counts.dtype, device=ids.device)
    offsets[1:] = counts.cumsum(0)
    row_token = torch.full((T * K,), -1, device=ids.device)
    row_token[:slots.numel()] = slots // K
    inv = torch.full((T * K,), -1, device=ids.device)
    inv[slots] = torch.arange(slots.numel(), device=ids.device)
    return counts, offsets, row_token, inv.reshape(T, K)


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "layer":
        return _exact_layer(case, s)
    logits, K, N = s["logits"].double(), case["K"], case["N"]
    if case["kind"] == "routing":
        k, ids, w = _route64(logits, K, "elbow", case["renormalize"])
        out = (k, ids, w) + _exact_dispatch(ids, N)
    else:
        p, order, curve, e = _elbow64(logits)
        px, py = e.double() / (N - 1), curve.gather(1, e[:, None])[:, 0]
        cross = (px * (1 - py) - py * (1 - px)).abs()
        theta = torch.rad2deg(torch.atan2(cross, -px * (1 - px) - py * (1 - py)))
        theta = torch.where(e == 0, 180.0, theta)
        k = (e + 1).clamp(max=K)
        # the elbow's experts in order, then those with the smallest draws among the others
        rank = torch.empty_like(order).scatter_(1, order, torch.arange(
            N, device=order.device).expand_as(order))
        taken = rank < k[:, None]
        key = torch.where(taken, rank.double() - N, s["rand"].double())
        ids = key.sort(dim=1, stable=True).indices[:, :K]
        w = torch.softmax(logits, 1).gather(1, ids)
        if case["renormalize"]:
            w = w / w.sum(1, keepdim=True)
        out = (e, theta, k, ids, w)
    return tuple(o.int() if o.dtype == torch.int64 else o for o in out)
