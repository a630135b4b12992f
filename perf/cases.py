"""What a user of this library has it do, as timed cases.

A case is one pass through the public binding: a `predict` call for L layers
of T tokens (bf16 or fp32 storage, with or without activation, biases and
confidence outputs), or the steps that turn a selection into a prefetch list
and accuracy counters (`confidence_select`, `group_by_expert`,
`activation_profile`, `score`).  `listed()` holds named cases from the
smallest call to the largest, `draw()` more of the same ranges.

Inputs are drawn on the GPU from the seed with the statistics of
`paper_2511_10676_amd.datagen`: post-norm hidden states with a few outlier
channels, weights of variance 1/fan-in, expert popularity that follows a power
law.
"""
import math

import torch

from paper_2511_10676_amd import binding as B

# widths of the workload table
DEEPSEEK = dict(d=2048, r=2048, E=64)
QWEN = dict(d=2048, r=2048, E=128)
PHI = dict(d=4096, r=1024, E=16)
STRESS = dict(d=2048, r=4096, E=256)


def _predict(name, shape, L, T, k, dtype="bf16", act="none", bias="none", prob="softmax", extra="none",
             prepared=False):
    """bias: none, b2 (popularity skew on the scores) or both; extra: none, counts (activation counts are
    accumulated) or margin (confidence margin per row); prepared: the call was marshalled once (a decode loop)."""
    c = dict(kind="predict", L=L, T=T, k=k, dtype=dtype, act=act, bias=bias, prob=prob, extra=extra,
             prepared=prepared, **shape)
    return dict(c, name=name) if name else c


def _route(name, L, T, E, k, k_base):
    c = dict(kind="route", L=L, T=T, E=E, k=k, k_base=k_base)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one token at one layer: the predictor runs when the layer's attention begins, latency is all that counts
        _predict("decode_layer", DEEPSEEK, L=1, T=1, k=6, prepared=True),
        # one token, the predictors of all layers of a model at once
        _predict("decode_bank_t1", DEEPSEEK, L=26, T=1, k=6, prepared=True),
        # a small decode batch, over-provisioned width, expert popularity accumulated over the generation
        _predict("decode_bank_t16_counts", QWEN, L=48, T=16, k=12, extra="counts", prepared=True),
        # a large, odd decode batch with the confidence outputs that drive dynamic widths
        _predict("decode_bank_t61_margin", PHI, L=32, T=61, k=3, bias="b2", prob="softmax_topk", extra="margin",
                 prepared=True),
        # one chunk of a chunked prefill at one layer
        _predict("chunk_layer", DEEPSEEK, L=1, T=512, k=6),
        # a short odd prompt through all layers, SiLU between the two maps and both biases, over-provisioned
        _predict("chunk_bank_silu", DEEPSEEK, L=26, T=301, k=10, act="silu", bias="both"),
        # the benchmark's headline call
        _predict("prefill_deepseek", DEEPSEEK, L=26, T=4096, k=6),
        # a long odd prompt, 128 experts, GELU with folded BatchNorm (both biases)
        _predict("prefill_qwen_gelu", QWEN, L=48, T=6011, k=8, act="gelu", bias="both"),
        # wide hidden state, few experts, popularity skew in b2
        _predict("prefill_phi", PHI, L=32, T=8192, k=2, bias="b2"),
        # the largest call of the workload table
        _predict("prefill_stress", STRESS, L=48, T=32768, k=8),
        # a predictor in the precision it was trained in, evaluated before its conversion to bf16
        _predict("f32_layer", DEEPSEEK, L=1, T=512, k=6, dtype="f32"),
        # the selections of an over-provisioned prefill: widths by confidence, prefetch lists, popularity, accuracy
        _route("route_qwen", L=48, T=8192, E=128, k=12, k_base=8),
    ]


_LARGEST = 2.0 * 4096 * (2048 + 256) * 32768 * 48          # flops of prefill_stress


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "f32", "route"])
    L = rng.choice([1, _log_int(rng, 1, 48)])
    E = rng.choice([16, 64, 128, 256, _log_int(rng, 8, 256)])
    if kind == "route":
        T = _log_int(rng, 1, 32768)
        k = rng.randint(2, min(E, 16))
        return _route(None, L, T, E, k, rng.randint(1, k - 1))
    d = rng.choice([2048, 4096, 64 * rng.randint(12, 80)])
    r = rng.choice([1024, 2048, 4096, 128 * rng.randint(4, 32)])
    shape = dict(d=d, r=r, E=E)
    opts = dict(k=rng.randint(1, min(E, 12)), act=rng.choice(["none", "none", "silu", "gelu"]),
                bias=rng.choice(["none", "b2", "both"]), prob=rng.choice(["softmax", "softmax", "softmax_topk", "sigmoid"]))
    if kind == "f32":
        # the toy workload's widths up to a model's, a few layers, so that a pass stays well below two seconds
        small = rng.random() < 0.4
        shape = dict(d=256, r=64, E=16) if small else dict(shape, d=min(d, 4096), r=min(r, 2048))
        T = _log_int(rng, 1, 1024)
        opts["k"] = min(opts["k"], shape["E"])
        return _predict(None, shape, L=rng.randint(1, 4), T=T, dtype="f32", **opts)
    if kind == "decode":
        T = _log_int(rng, 1, 64)
        extra = rng.choice(["none", "none", "margin", "counts" if T <= 16 else "none"])
        return _predict(None, shape, L=L, T=T, extra=extra, prepared=rng.random() < 0.7, **opts)
    T = _log_int(rng, 65, 32768)
    while 2.0 * r * (d + E) * T * L > _LARGEST:
        L = max(1, L // 2)
    return _predict(None, shape, L=L, T=T, extra=rng.choice(["none", "none", "margin"]), **opts)


def _hidden_states(g, L, T, d, dtype):
    """Post-norm states: N(0, 1), a few outlier channels eight times larger, rows divided by their RMS."""
    x = torch.empty((L, T, d), dtype=dtype, device="cuda")
    for l in range(L):
        h = torch.randn((T, d), generator=g, device="cuda")
        h[:, torch.randperm(d, generator=g, device="cuda")[:max(4, d // 512)]] *= 8.0
        x[l] = h * h.square().mean(dim=1, keepdim=True).rsqrt()
    return x


def _weights(g, L, rows, cols, dtype):
    w = torch.empty((L, rows, cols), dtype=dtype, device="cuda")
    for l in range(L):
        w[l] = torch.randn((rows, cols), generator=g, device="cuda") * (cols ** -0.5)
    return w


def _popularity(g, L, E):
    """Score offsets of a power-law expert popularity, another order of experts in every layer."""
    logp = -1.2 * torch.log(torch.arange(1, E + 1, device="cuda", dtype=torch.float32))
    order = torch.argsort(torch.rand((L, E), generator=g, device="cuda"), dim=1)
    return 0.6 * (logp - logp.mean())[order]


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    L, T, E, k = case["L"], case["T"], case["E"], case["k"]
    if case["kind"] == "route":
        idx = torch.empty((L, T, k), dtype=torch.int32, device="cuda")
        ref = torch.empty((L, T, case["k_base"]), dtype=torch.int32, device="cuda")
        probs = torch.empty((L, T, k), device="cuda")
        pop = _popularity(g, L, E)
        for l in range(L):
            z = torch.randn((T, E), generator=g, device="cuda") + pop[l]
            top = torch.topk(torch.softmax(z, dim=1), k, dim=1)
            probs[l], idx[l] = top.values, top.indices
            router = z + 0.1 * torch.randn((T, E), generator=g, device="cuda")
            ref[l] = torch.topk(router, case["k_base"], dim=1).indices
        return dict(case=case, idx=idx, ref=ref, probs=probs)
    d, r = case["d"], case["r"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    x = _hidden_states(g, L, T, d, dtype)
    W1, W2 = _weights(g, L, r, d, dtype), _weights(g, L, E, r, dtype)
    b1 = (0.1 * torch.randn((L, r), generator=g, device="cuda")).to(dtype) if case["bias"] == "both" else None
    b2 = _popularity(g, L, E).to(dtype) if case["bias"] != "none" else None
    args = dict(b1=b1, b2=b2, act=case["act"], prob=case["prob"], want_margin=case["extra"] == "margin")
    if case["extra"] == "counts":
        args["counts"] = torch.zeros((L, E), dtype=torch.int32, device="cuda")
    state = dict(case=case, x=x, W1=W1, W2=W2, args=args)
    if case["prepared"]:
        state["call"] = B.prepare_predict(x, W1, W2, k, **args)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "route":
        E = case["E"]
        wide = B.confidence_select(state["idx"], state["probs"], case["k_base"], 1.25)
        lists = B.group_by_expert(wide.idx, E)
        profile = B.activation_profile(lists.counts)
        counters = B.score(wide.idx, state["ref"], E, k_row=wide.k_row)
        return [*wide, *lists, *profile, counters]
    if "call" in state:
        out = state["call"]()
    else:
        out = B.predict(state["x"], state["W1"], state["W2"], case["k"], **state["args"])
    got = [out.idx, out.probs]
    if case["extra"] == "margin":
        got.append(out.margin)
    if case["extra"] == "counts":
        got.append(state["args"]["counts"])
    return got


def work(case):
    L, T, E, k = case["L"], case["T"], case["E"], case["k"]
    if case["kind"] == "route":
        # in: ids, probabilities, labels; out: narrowed ids, widths, lists, per-expert and per-layer arrays
        per_layer = 4 * T * (3 * k + case["k_base"] + k + 1) + 4 * (4 * E + 4) + 48
        return {"bytes": L * per_layer, "flops": 0}
    s = 4 if case["dtype"] == "f32" else 2
    d, r = case["d"], case["r"]
    per_layer = s * (r * (d + E) + T * d) + 8 * T * k
    if case["bias"] != "none":
        per_layer += s * E + (s * r if case["bias"] == "both" else 0)
    if case["extra"] == "margin":
        per_layer += 4 * T
    if case["extra"] == "counts":
        per_layer += 8 * E
    return {"bytes": L * per_layer, "flops": 2.0 * r * (d + E) * T * L}


def tolerance(case):
    if case["kind"] == "route":
        return {"rel": 1e-12, "max": 1e-12, "differ": 0.0}   # whole numbers, and an entropy in double
    # Four times what was seen between this path and its definition with the sums in another order (f32: torch's
    # products; bf16: double sums, the hidden vector rounded to bf16 as the path does).  f32: 1.3e-6 / 4.3e-6 / 6.5e-4
    # of the ids.  bf16: 3.5e-5 / 1.3e-3 / 2.2e-4; a hidden unit whose sum falls on the other side of a bf16 rounding
    # boundary moves a score by 1e-4 of its scale.  A margin is the difference of two scores: 8e-4 / 1.1e-2.
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 2e-5, "differ": 3e-3}
    if case["extra"] == "margin":
        return {"rel": 3e-3, "max": 4e-2, "differ": 1e-3}
    return {"rel": 1.5e-4, "max": 5e-3, "differ": 1e-3}
