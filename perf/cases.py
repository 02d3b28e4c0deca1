"""What the shared-pool MoE layer is timed on: training steps and forward passes through PoolStep / PoolGroups, over
the sizes, data types and options the package is used with.

A case is a dict of plain values:
  kind      "step": all L layers forward, the auxiliary loss, all L layers backward with weight and router gradients;
            "forward": the L layers forward with the dispatch fused into the first GEMM (inference).
  L, E, d, f, k, T   layers sharing the pool, pool size, d_model, d_ff of an expert, experts per token, tokens per layer
  dtype     "bf16" or "f32";  skew "none", "hot" (a fifth of the experts takes about half of the slots) or "zipf"
  router    "norm" or "softmax";  aux "pool" or "layer";  wgrad "pool" or "layer";  recompute, lagged: PoolStep's
  groups    pools the layers are cut into (1: one PoolStep; more: PoolGroups)
"""
import math

import numpy as np
import torch

import paper_2605_06665_amd as U
from paper_2605_06665_amd.pipeline import PoolGroups, PoolStep

DEVICE = "cuda:0"
EPS = 1e-6
ALPHA = 2e-2
WEIGHT_STD = 0.02


def _case(name=None, **kw):
    c = dict(kind="step", L=2, E=8, d=64, f=128, k=2, T=128, dtype="bf16", skew="none", router="norm", aux="pool",
             wgrad="pool", recompute=False, lagged=False, groups=1)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest configuration of the benchmark, the one that is checked to 1e-5: launches and latency
        _case("tiny-f32-step", L=2, E=8, d=64, f=128, k=2, T=128, dtype="f32"),
        # float mode as a debugging or reference run of a reduced model: ragged widths, pool not a multiple of 8
        _case("reduced-f32-step", L=2, E=12, d=252, f=500, k=3, T=1001, dtype="f32"),
        # the benchmark's small, reduced-pool (hot experts, recomputation, one-step-behind statistic), fine-grained
        # and largest training configurations; the largest at 8 of its 24 layers, so that three sets of state fit
        _case("small-step", L=8, E=64, d=768, f=2048, k=2, T=8192),
        _case("reduced-pool-hot-step", L=16, E=96, d=1024, f=2816, k=2, T=16384, skew="hot", recompute=True, lagged=True),
        _case("fine-grained-step", L=16, E=512, d=1024, f=704, k=8, T=16384),
        _case("largest-step", L=8, E=192, d=1536, f=4096, k=2, T=32768),
        # ablation rows: softmax router with the per-layer loss under skewed use of a fine-grained pool
        _case("fine-grained-zipf-softmax-step", L=6, E=512, d=1024, f=704, k=8, T=16384, skew="zipf", router="softmax",
              aux="layer"),
        # the vanilla MoE that is compared against: layer-private experts, top-1, softmax router; ragged token count
        _case("vanilla-step", L=4, groups=4, E=16, d=768, f=2048, k=1, T=3001, router="softmax"),
        # odd sizes: pool not a multiple of 8, d_model not a multiple of 128, odd top-k, gradients layer by layer
        _case("odd-pool-step", L=4, E=90, d=832, f=1472, k=3, T=5999, wgrad="layer"),
        # inference with the largest pool: a prompt of about 4000 tokens, then a few sequences decoding one token each
        _case("prefill", kind="forward", L=8, E=192, d=1536, f=4096, k=2, T=4001),
        _case("decode-few", kind="forward", L=24, E=192, d=1536, f=4096, k=2, T=4),
        # a batch of sequences decoding with the fine-grained pool
        _case("decode-batch-fine-grained", kind="forward", L=16, E=512, d=1024, f=704, k=8, T=48),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _flops(c):
    """Multiply-adds x 2 of the contractions of one pass."""
    S = c["T"] * c["k"]
    ffn, router = 6.0 * S * c["d"] * c["f"], 2.0 * c["T"] * c["d"] * c["E"]
    if c["kind"] == "forward":
        return c["L"] * (ffn + router)
    return c["L"] * (3.0 * ffn + (4.0 * S * c["d"] * c["f"] if c["recompute"] else 0.0) + 3.0 * router)


def _state_bytes(c):
    act = 2 if c["dtype"] == "bf16" else 4
    S, d, f = c["T"] * c["k"], c["d"], c["f"]
    layer = S * (4 * d + 5 * f) + 4 * c["T"] * d
    return act * (c["L"] * layer + 3 * c["groups"] * c["E"] * d * f) + 12 * c["groups"] * c["E"] * d * f


def draw(rng):
    big = _case(L=8, E=192, d=1536, f=4096, k=2, T=32768)
    while True:
        what = rng.choice(["f32", "step", "step", "step", "forward", "forward"])
        if what == "f32":
            c = _case(dtype="f32", L=rng.randint(1, 4), E=rng.randint(3, 32), d=_log_int(rng, 30, 320),
                      f=_log_int(rng, 17, 640), k=rng.randint(1, 3), T=_log_int(rng, 50, 1500),
                      router=rng.choice(["norm", "norm", "softmax"]), wgrad=rng.choice(["pool", "layer"]))
            most = _flops(_case(dtype="f32", L=2, E=12, d=252, f=500, k=3, T=1001)) * 1.5
        else:
            c = _case(L=rng.randint(2, 16), d=64 * _log_int(rng, 4, 24), f=64 * _log_int(rng, 4, 64),
                      k=rng.choice([1, 2, 2, 2, 3, 4, 6, 8]), skew=rng.choice(["none", "none", "hot", "zipf"]))
            c["E"] = rng.choice([8 * _log_int(rng, 1, 64), _log_int(rng, 10, 500)])
            if what == "forward":
                c["kind"] = "forward"
                c["T"] = _log_int(rng, 1, 8192)
            else:
                c["T"] = _log_int(rng, 256, 32768)
                c["router"] = rng.choice(["norm", "norm", "softmax"])
                c["aux"] = rng.choice(["pool", "pool", "layer"])
                c["lagged"] = c["aux"] == "pool" and rng.random() < 0.3
                c["recompute"] = rng.random() < 0.3
                c["wgrad"] = rng.choice(["pool", "pool", "layer"])
                if c["L"] % 2 == 0 and rng.random() < 0.2:
                    c["groups"] = 2
                    c["lagged"] = False
            most = _flops(big)
        if c["k"] <= c["E"] and _flops(c) <= most and _state_bytes(c) <= 0.9 * _state_bytes(big):
            return c


def _normal(shape, gen, dtype, std=1.0):
    return torch.empty(shape, dtype=dtype, device=DEVICE).normal_(0.0, std, generator=gen)


def _calibration(E, k):
    """The NormRouter constant c(E, k): mean of 1 / norm of the k largest components of relu(x / |x|)."""
    x = np.random.default_rng(7).standard_normal((1000, E))
    y = np.maximum(x / np.linalg.norm(x, axis=1, keepdims=True), 0.0)
    top = -np.sort(-y, axis=1)[:, :k]
    n = np.linalg.norm(top, axis=1)
    return float(np.mean(1.0 / n[n > 0]))


def _expert_bias(c, rng):
    """Per-expert logit offsets of one layer, in units of the logits' noise."""
    E = c["E"]
    bias, order = np.zeros(E), rng.permutation(E)
    if c["skew"] == "hot":
        bias[order[: max(1, E // 5)]] = 0.625
    elif c["skew"] == "zipf":
        p = np.arange(1, E + 1, dtype=np.float64) ** -1.1
        bias[order] = 0.5 * np.log(p / p.sum())
    return bias


def prepare(case, seed):
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    L, E, d, f, k, T, G = c["L"], c["E"], c["d"], c["f"], c["k"], c["T"], c["groups"]
    act = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    train = c["kind"] == "step"
    xs = [_normal((T, d), gen, act) for _ in range(L)]
    # the softmax router's rows are scaled as a trained one's would be (logits of about unit size); NormRouter is
    # invariant to the scale
    scale = 1.0 if c["router"] == "norm" else 1.0 / math.sqrt(d)
    w_routers = [_normal((E, d), gen, act, scale) for _ in range(L)]
    if c["skew"] != "none":
        for x, w in zip(xs, w_routers):
            x[:, d - 1] = 1.0
            w[:, d - 1] = torch.from_numpy(scale * math.sqrt(d - 1) * _expert_bias(c, rng)).to(DEVICE, act)
    weights = [(_normal((E, 2 * f, d), gen, act, WEIGHT_STD), _normal((E, d, f), gen, act, WEIGHT_STD)) for _ in range(G)]
    grads = [_normal((T, d), gen, act) for _ in range(L)] if train else None
    sigmas = [float(s) for s in rng.uniform(0.8, 1.2, L)]
    dtype = U.BF16 if c["dtype"] == "bf16" else U.F32
    kw = dict(device=DEVICE, wgrad=c["wgrad"], recompute=c["recompute"], lagged=c["lagged"], aux=c["aux"],
              router=c["router"])
    shape = (T, d, f, E, k, L, dtype, _calibration(E, k), EPS, ALPHA)
    if G > 1:
        driver = PoolGroups(G, *shape, **kw)
        pools = driver.groups
    else:
        driver = PoolStep(*shape, **kw)
        pools = [driver]
    layers = [st for p in pools for st in p.layers]
    # the small per-layer gradients side by side, as an optimizer holds them
    d_w_router = torch.zeros((L, E, d), dtype=torch.float32, device=DEVICE)
    d_sigma = torch.zeros(L, dtype=torch.float32, device=DEVICE)
    for l, st in enumerate(layers):
        st.d_w_router, st.d_sigma = d_w_router[l], d_sigma[l:l + 1]
    return dict(case=c, driver=driver, pools=pools, layers=layers, xs=xs, w_routers=w_routers, sigmas=sigmas,
                weights=weights, grads=grads, d_w_router=d_w_router, d_sigma=d_sigma)


def run(s):
    c, driver, layers = s["case"], s["driver"], s["layers"]
    if c["kind"] == "forward":
        w_gate_up, w_down = s["weights"][0]
        for l in range(c["L"]):
            driver.forward_layer(l, s["xs"][l], s["w_routers"][l], s["sigmas"][l], w_gate_up, w_down, gather=True)
        return {"out": [st.out for st in layers], "topk_idx": [st.topk_idx for st in layers], "counts": driver.counts}
    if c["groups"] > 1:
        driver.step(s["xs"], s["w_routers"], s["sigmas"], [w[0] for w in s["weights"]], [w[1] for w in s["weights"]],
                    s["grads"])
    else:
        driver.step(s["xs"], s["w_routers"], s["sigmas"], *s["weights"][0], s["grads"])
    pools = s["pools"]
    return {
        "out": [st.out for st in layers], "dx": [st.dx for st in layers], "d_w_router": s["d_w_router"],
        "d_sigma": s["d_sigma"], "d_w_gate_up": [p.d_w_gate_up for p in pools], "d_w_down": [p.d_w_down for p in pools],
        "counts": [p.counts for p in pools],
        "loss": [p.loss_layers if p.aux == "layer" else p.loss for p in pools],
    }


def work(case):
    """Every layer reads x and the weights of the experts that its tokens reach (the layers run one after the other
    and the pool does not fit a cache), once forward and once backward; float weight gradients go out once."""
    c = _case(**{k: v for k, v in case.items() if k != "name"})
    L, E, d, f, k, T = (c[n] for n in ("L", "E", "d", "f", "k", "T"))
    act = 2 if c["dtype"] == "bf16" else 4
    reached = E * (1.0 - (1.0 - k / E) ** T)               # under even use
    experts, token = act * 3.0 * d * f * reached, act * float(T) * d
    per_layer = 2 * token + act * E * d + experts           # x in, out out, router matrix, experts
    if c["kind"] == "step":
        # forward again for the backward pass, grad_out in, dx out, router gradient out
        per_layer += experts + token * 3 + (act + 4) * E * d
        return {"bytes": L * per_layer + 12.0 * c["groups"] * E * d * f, "flops": _flops(c)}
    return {"bytes": L * per_layer, "flops": _flops(c)}


def tolerance(case):
    """About four times the distance from float64 seen over all outputs (float32 8e-7 to 1.2e-6, bfloat16 4.2e-3 with
    its own intermediate roundings), the bfloat16 bound no wider than 1e-2.  Selections are a function of the logits:
    only near-ties may fall the other way."""
    if case.get("dtype") == "f32":
        return {"rel": 5e-6, "differ": 1e-3}
    return {"rel": 1e-2, "differ": 1e-3}
