"""The work that users of this library give it, as cases to time: serving calls (prefill and decode, with given logits
and with the router in front, with fixed thresholds and with thresholds chosen per batch), full-precision layers, shapes
off the matrix-core grid, and what a program does around serving: load a layer and calibrate its neuron order.

The layer shapes are the benchmark layers of bench.py / synth: a wide layer of 8 large experts (Mixtral-shaped), one
expert-parallel rank's share of it under skewed popularity, a fine-grained layer of 64 small experts, and a layer with
shared experts.  Weights are random of standard deviation 0.02, activations N(0, 1), router logits N(0, 1), neuron
orders random, as there.
"""
import math

import torch

from paper_2508_18376_amd import DualSparseLayer
from paper_2508_18376_amd.thresholds import dual_thresholds

WIDE = dict(d_model=4096, d_ff=14336, experts=8, top_k=2, parts=4, shared=0)
SHARE = dict(WIDE, resident=2, zipf=1.2)  # experts 0 and 1 of 8 on this GPU; expert 0 is the most popular one
FINE = dict(d_model=2048, d_ff=1024, experts=64, top_k=8, parts=2, shared=0)
SHARED = dict(d_model=2048, d_ff=1408, experts=64, top_k=6, parts=2, shared=2)
TINY = dict(d_model=128, d_ff=256, experts=8, top_k=2, parts=2, shared=0)
ODD = dict(SHARED, parts=8)  # 176 neurons per sub-expert: no multiple of the 32 that the matrix-core path needs

W_STD = 0.02
ZIPF_RANK = (1, 5, 2, 3, 4, 6, 7, 8)  # popularity rank of each expert id, as in the skewed benchmark layer


def _case(shape, op, tokens, drop, dtype="bf16", **more):
    return dict(shape, op=op, tokens=tokens, drop=drop, dtype=dtype, **more)


def listed():
    return [
        # the smallest call: the unit-test-sized fp32 layer, where launches and latency are everything
        _case(TINY, "forward", 64, 0.2, "f32", name="tiny_f32"),
        # one user's decode step on a fine-grained layer: a single token, 8 experts
        _case(FINE, "routed", 1, 0.25, name="fine_decode_1"),
        # a decode step of a server with 64 users on the wide layer: all weights are read once
        _case(WIDE, "routed", 64, 0.25, name="wide_decode_64"),
        # a small odd prompt on the layer with shared experts
        _case(SHARED, "routed", 333, 0.25, name="shared_prompt_333"),
        # prefill of the wide layer, the headline workload
        _case(WIDE, "forward", 4096, 0.25, name="wide_prefill_4096"),
        # prefill of the fine-grained layer with the router in front
        _case(FINE, "routed", 8192, 0.25, name="fine_prefill_8192"),
        # prefill of the layer with shared experts at a ragged size, thresholds taken from the batch for a target rate
        _case(SHARED, "rate", 7001, 1.0 / 3.0, name="shared_rate_7001"),
        # an expert-parallel rank under skewed popularity: load-aware thresholds with a row cap, then the layer
        _case(SHARE, "load", 16384, 0.25, name="share_load_16384"),
        # the full-precision path at an ordinary size
        _case(FINE, "forward", 512, 0.25, "f32", name="fine_f32_512"),
        # a bf16 layer cut into sub-experts whose width is off the matrix-core grid
        _case(ODD, "forward", 777, 0.25, name="odd_parts_777"),
        # loading a layer: weights into the kernels' layout in a given neuron order, and a first small batch through it
        _case(WIDE, "load_weights", 64, 0.25, name="wide_load_weights"),
        # calibration: importance of every neuron over a calibration batch, and the neuron order from it
        _case(FINE, "calibrate", 8192, 0.0, metric=3, name="fine_calibrate_8192"),
    ]


def draw(rng):
    def tokens(lo, hi):  # spread over the logarithm; any size, odd ones among them
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["forward", "forward", "routed", "routed", "routed", "rate", "load", "f32", "odd", "load_weights", "calibrate"])
    drop = rng.choice([0.0, 0.125, 0.25, 0.25, 0.5])
    if op in ("forward", "routed", "rate"):
        shape, most = rng.choice([(WIDE, 4096), (FINE, 8192), (SHARED, 8192)])
        if op == "rate" and drop == 0.0:
            drop = 0.25
        return _case(shape, op, tokens(1, most), drop, y_fp32=rng.random() < 0.2, renorm=rng.random() < 0.3)
    if op == "load":
        return _case(SHARE, op, tokens(512, 16384), 0.25)
    if op == "f32":
        shape, most = rng.choice([(TINY, 4096), (FINE, 512)])
        return _case(shape, rng.choice(["forward", "routed"]), tokens(1, most), drop, "f32")
    if op == "odd":
        return _case(rng.choice([ODD, dict(FINE, d_ff=1000, parts=4), dict(TINY, d_model=100)]), "forward", tokens(1, 777), drop)
    if op == "load_weights":
        return _case(rng.choice([FINE, SHARED, dict(WIDE, resident=2)]), op, tokens(8, 256), drop)
    return _case(rng.choice([FINE, SHARED]), "calibrate", tokens(1024, 8192), 0.0, metric=rng.choice([1, 3]))


def _resident(c):
    return c.get("resident", c["experts"])


def _zipf_bias(c):
    w = torch.tensor([float(r) ** -c["zipf"] for r in ZIPF_RANK[:c["experts"]]], dtype=torch.float64)
    return torch.log(w / w.sum()).float()


def _scores(logits, k):
    """Top-K experts and their scores normalised over the K."""
    s, idx = torch.topk(logits, k, dim=1)
    return torch.softmax(s, dim=1), idx


def _fixed_tau(c, logits):
    """A threshold row for the drop rate, from the scores of `logits`: what a program has from its calibration."""
    if c["drop"] <= 0.0:
        return torch.zeros(c["parts"])
    n = _scores(logits, c["top_k"])[0].flatten().sort().values
    centre = float(n[min(int(c["drop"] * n.numel()), n.numel() - 1)])
    return torch.from_numpy(dual_thresholds(centre, c["parts"]))


def prepare(case, seed):
    c, dev = case, torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    D, F, E, K, P, T, n_sh, R = (c["d_model"], c["d_ff"], c["experts"], c["top_k"], c["parts"], c["tokens"], c["shared"], _resident(c))

    def normal(*shape, std=1.0, dtype=dt):
        t = torch.randn(*shape, generator=gen, device=dev, dtype=dtype)
        return t if std == 1.0 else t.mul_(std)

    s = {"op": c["op"], "rate": c["drop"], "metric": c.get("metric", 3)}
    layer = s["layer"] = DualSparseLayer(
        d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=P, max_tokens=max(256, T), dtype=c["dtype"], n_shared=n_sh,
        d_ff_shared=F if n_sh else 0, expert_lo=0, expert_hi=R, renorm_combine=bool(c.get("renorm")), y_fp32=bool(c.get("y_fp32")))
    s["x"] = normal(T, D)
    w1, w3, w2 = normal(R, D, F, std=W_STD), normal(R, D, F, std=W_STD), normal(R, F, D, std=W_STD)
    sh = {}
    if n_sh:
        sh = dict(sh_w1=normal(n_sh, D, F, std=W_STD), sh_w3=normal(n_sh, D, F, std=W_STD), sh_w2=normal(n_sh, F, D, std=W_STD))
    perm = torch.rand(R, F, generator=gen, device=dev).argsort(dim=1).to(torch.int32)
    wg = normal(D, E, std=1.0 / math.sqrt(D))
    bias = _zipf_bias(c).to(dev) if c.get("zipf") else 0.0
    s["logits"] = normal(T, E, dtype=torch.float32) + bias
    calibration = normal(4096, E, dtype=torch.float32).cpu()  # another batch's logits: what fixed thresholds come from
    row = _fixed_tau(c, calibration).to(dev)
    s["tau"] = row.repeat(E, 1).contiguous()
    if c["op"] == "load":
        s["tau_max"], s["row_cap"] = row.contiguous(), max(1, int(1.25 * T * K / E))
    if c["op"] == "load_weights":
        s["weights"] = dict(w1=w1, w3=w3, w2=w2, perm=perm, **sh)
    else:  # calibration runs on the original neuron order
        layer.partition_weights(w1, w3, w2, perm=None if c["op"] == "calibrate" else perm, **sh)
    if c["op"] == "routed":
        layer.pack_router(wg)
    return s


def run(state):
    s, layer = state, state["layer"]
    op = s["op"]
    if op == "forward":
        return {"y": layer.forward(s["x"], s["logits"], s["tau"])}
    if op == "routed":
        return {"y": layer.forward_routed(s["x"], s["tau"])}
    if op == "rate":
        tau, stats = layer.thresholds_for_drop_rate(s["logits"], s["rate"])
        return {"y": layer.forward(s["x"], s["logits"], tau), "tau": tau, "stats": stats}
    if op == "load":
        tau, pairs = layer.select_thresholds(s["logits"], s["tau_max"], group_size=1, row_cap=s["row_cap"])
        return {"y": layer.forward(s["x"], s["logits"], tau), "tau": tau, "pairs": pairs}
    if op == "load_weights":
        layer.partition_weights(**s["weights"])
        return {"y": layer.forward(s["x"], s["logits"], s["tau"])}
    importance = layer.profile_importance(s["x"], s["logits"], s["metric"])
    return {"importance": importance, "perm": layer.importance_to_perm(importance)}


def _expected(c):
    """Kept units per token of every (resident expert, partition), from a sample of the case's score distribution."""
    gen = torch.Generator().manual_seed(1)
    logits = torch.randn(4096, c["experts"], generator=gen)
    row = _fixed_tau(c, logits)
    if c.get("zipf"):
        logits = logits + _zipf_bias(c)
    n, idx = _scores(logits, c["top_k"])
    kept = torch.zeros(_resident(c), c["parts"], dtype=torch.float64)
    for e in range(_resident(c)):
        mine = n[idx == e]
        for p in range(c["parts"]):
            kept[e, p] = (mine >= row[p]).sum().item() / 4096.0
        if c["op"] == "load":  # the row cap of the load-aware thresholds
            kept[e] = kept[e].clamp(max=1.25 * c["top_k"] / c["experts"])
    return kept


def work(case):
    c = case
    elem = 2 if c["dtype"] == "bf16" else 4
    D, F, T, R, Fp = c["d_model"], c["d_ff"], c["tokens"], _resident(c), c["d_ff"] // c["parts"]
    routed, shared = R * 3 * D * F * elem, c["shared"] * 3 * D * F * elem  # bytes of all weights
    gating = T * c["experts"] * 4 if c["op"] != "routed" else c["experts"] * D * elem
    kept = _expected(c)
    units = T * float(kept.sum())
    touched = float((1.0 - (1.0 - kept.clamp(max=1.0)) ** T).sum()) / (R * c["parts"])  # share of the sub-experts that any token keeps
    if c["op"] == "calibrate":
        return {"bytes": routed * 2 / 3 + T * D * elem + gating + R * F * 8, "flops": 4 * D * Fp * units}
    y_bytes = T * D * (4 if c.get("y_fp32") else elem)
    flops = 6 * D * Fp * units + 6 * D * F * c["shared"] * T + (2 * D * c["experts"] * T if c["op"] == "routed" else 0)
    moved = routed * touched + shared + T * D * elem + y_bytes + gating
    if c["op"] == "load_weights":  # read, and written in the kernels' layout, which the first batch then reads
        moved += 2 * (routed + shared) + R * F * 4
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # about four times the distance from the same path evaluated in 64 bits (measured; bf16 results against the rounded 64-bit ones)
    if case["dtype"] == "f32":
        return {"rel": 6e-6, "max": 5e-5}
    if case["op"] == "calibrate":  # fp32 sums; neurons whose sums are closer than their rounding may change places in the order
        return {"rel": 1e-6, "max": 5e-6, "differ": 2e-3}
    return {"rel": 4.5e-3, "max": 0.04}
