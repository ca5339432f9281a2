"""GPU: large batches on layers of many experts in the full-precision path: bf16 layers take tiles of two weight images there (tiles with one
image, pieces of one image, one to four blocks of 32 rows, K splits), fp32 layers keep fp32 products (sums of one sign and of one term); infinities.
"""
import numpy as np
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev, to_host64
from test_gpu_forward import spec_of, resolve_tau, oracle_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,T,D,F,P,tau_kind", [
    ("f32", 2000, 256, 128, 1, 0.0),
    ("f32", 4300, 260, 176, 1, "rate0.25"),
    ("f32", 2600, 140, 384, 4, "ragged"),
    ("bf16", 4300, 260, 176, 1, "rate0.25"),
    ("bf16", 4300, 257, 136, 1, 0.0),
])
def test_two_images_to_a_tile(oracle, dtype, T, D, F, P, tau_kind):
    import torch
    spec = spec_of(T=T, D=D, F=F, E=512, K=8, P=P, dtype=dtype, seed=160, x_std=1.0, w_std=0.05)
    t = make_layer(spec)
    t["logits"][: T // 3, 7] += 4.0  # an expert of many row tiles, and some beyond 64 rows
    t["logits"][:130, 11] += 6.0
    tau = resolve_tau(oracle, spec, t, tau_kind)
    layer, dev = make_gpu_layer(spec, t, y_fp32=True)
    assert not layer.uses_mfma
    print(dtype, T, D, F, P, flush=True)
    y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
    torch.cuda.synchronize()
    images = 512 * P * ((F // P + 63) // 64)
    # at least one tile per expert and partition: not of single images
    assert dtype == "f32" or tau_kind != 0.0 or layer.plan(T)["counters"][0] < images
    layer.close()
    # the fp32 bar, 1e-5 x RMS, token by token: rounding scales with a token's own output, and the tokens of the two favoured experts have
    # outputs some ten times those of the others (whose softmax spreads over 512 experts)
    ref = oracle_forward(oracle, spec, t, tau)
    rms = np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True))
    assert (np.abs(to_host64(y, "f32") - ref) <= 1e-5 * rms).all()


def _positive_layer(T, D, F, E, K, dtype="f32"):
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    def rand(*s):
        return torch.rand(*s, generator=gen, device="cuda:0")
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=1, max_tokens=T, dtype=dtype, y_fp32=True)
    assert not layer.uses_mfma
    w1, w3, w2 = (rand(E, *s).mul_(0.01).to(dt) for s in ((D, F), (D, F), (F, D)))
    layer.partition_weights(w1, w3, w2)
    return layer, w1, w3, w2, rand(T, D).to(dt), torch.randn(T, E, generator=gen, device="cuda:0")


def _reference64(w1, w3, w2, x, logits, K):
    import torch
    s, idx = torch.softmax(logits.double(), 1), torch.topk(logits, K, dim=1).indices
    ref = torch.zeros(x.shape, dtype=torch.float64, device="cuda:0")
    for e in range(w1.shape[0]):
        t = (idx == e).any(1).nonzero().flatten()
        g = x[t].double() @ w1[e].double()
        h = g * torch.sigmoid(g) * (x[t].double() @ w3[e].double())
        ref.index_add_(0, t, s[t, e].unsqueeze(1) * (h @ w2[e].double()))
    return ref


def test_split_items_of_two_images():
    """bf16: the items of GEMM-2's last round are cut along K; their extra ranges go to partial-output tiles of 256 columns, written by items of both
    images, by halves of the list's last items and, the last column tile, by single images."""
    import torch
    layer, w1, w3, w2, x, logits = _positive_layer(850, 1400, 600, 104, 8, "bf16")
    x = x.float().sub_(0.5).bfloat16()
    y = layer.forward(x, logits, torch.zeros(104, 1, device="cuda:0"))
    torch.cuda.synchronize()
    counters = layer.plan(850)["counters"].cpu().numpy()
    layer.close()
    assert counters[3] == 3 and counters[1] == 512 + 3 * 112
    ref = _reference64(w1, w3, w2, x, logits, 8)
    assert ((y - ref).abs() <= 1e-5 * ref.square().mean(1, keepdim=True).sqrt()).all()  # the fp32 bar, see above


def test_sums_of_one_sign():
    """fp32 sums round every addition to nearest, so sums of up to 2048 terms of one sign are right on average (measured: mean -1e-9 .. 1e-9,
    largest 1.1e-6).  An instruction that cuts its sums off towards zero leaves them 6e-6 short (bf16 parts), and
    where it drops the smallest products of the parts 1.2e-7: the mean tells both from rounding, whose errors' mean over the 524288
    outputs of three such products is below 3 * 2^-24 / sqrt(256), one token's outputs being the only ones that share roundings."""
    import torch
    T, D, F, E, K = 256, 2048, 1024, 64, 8
    layer, w1, w3, w2, x, logits = _positive_layer(T, D, F, E, K)
    y = layer.forward(x, logits, torch.zeros(E, 1, device="cuda:0")).double()
    ref = _reference64(w1, w3, w2, x, logits, K)
    layer.close()
    err = (y - ref) / ref
    assert err.abs().max().item() <= 3e-6
    assert abs(err.mean().item()) <= 3 * 2.0 ** -24 / 16


@pytest.mark.parametrize("sx,s3,s2", [(1.0, 1.0, 1.0), (2.0 ** -115, 2.0 ** 115, 2.0 ** 100)], ids=["ordinary", "tiny_operands"])
def test_sums_of_one_term_do_not_depend_on_the_batch(sx, s3, s2):
    """Every sum of both products has one term that is not zero, so it is that term rounded once, in whatever order and pieces K is
    taken: the first tokens come out bit for bit as in a batch of their own, also where an operand is close to the end of the range."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    T, D, F, E, K = 2100, 256, 128, 512, 8
    gen = torch.Generator(device="cuda:0").manual_seed(10)
    def normal(*s):
        return torch.randn(*s, generator=gen, device="cuda:0")
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=1, max_tokens=T, dtype="f32")
    w2 = torch.zeros(E, F, D, device="cuda:0")
    d = torch.arange(D, device="cuda:0")
    w2[:, d % F, d] = normal(E, D) * s2
    layer.partition_weights(normal(E, D, F), normal(E, D, F) * s3, w2)
    x = torch.zeros(T, D, device="cuda:0")
    x[torch.arange(T, device="cuda:0"), torch.randint(D, (T,), generator=gen, device="cuda:0")] = normal(T) * sx
    logits, tau = normal(T, E), torch.zeros(E, 1, device="cuda:0")
    y = layer.forward(x, logits, tau)
    few = layer.forward(x[:64], logits[:64], tau)
    torch.cuda.synchronize()
    layer.close()
    assert torch.isfinite(y).all() and (y != 0).all()
    assert torch.equal(y[:64], few)


@pytest.mark.parametrize("dtype,T,D,F", [("f32", 2100, 256, 128), ("bf16", 4300, 260, 176), ("bf16", 4300, 256, 136)])
def test_infinite_tokens(dtype, T, D, F):
    """A token with an infinite value has infinite outputs (all weights are positive), the others what they have without it."""
    import torch
    E, K = 512, 8
    layer, w1, w3, w2, x, logits = _positive_layer(T, D, F, E, K, dtype)
    tau = torch.zeros(E, 1, device="cuda:0")
    clean = layer.forward(x, logits, tau)
    x[5::400, 3] = float("inf")
    y = layer.forward(x, logits, tau)
    torch.cuda.synchronize()
    layer.close()
    hot = torch.zeros(T, dtype=torch.bool, device="cuda:0")
    hot[5::400] = True
    assert torch.isposinf(y[hot]).all()
    assert torch.allclose(y[~hot], clean[~hot], rtol=1e-5, atol=0.0)


@pytest.mark.parametrize("hot_tokens", [False, True])
def test_infinite_weights_in_both_images(hot_tokens):
    """bf16, W2 with infinities and NaN in some experts, in a column of each of a tile's two images and of a tile of one image: where one neuron is
    active, whose activation has one part that is not zero (1024 -> 2^20) or three (3), these columns are infinite or NaN for the tokens of those
    experts, and everything else is bit for bit as with finite weights.  A token with an infinite value is infinite or NaN as a whole."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    T, D, F, E, K, inf = 4300, 260, 176, 512, 8, float("inf")
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=1, max_tokens=T, dtype="bf16", y_fp32=True)
    assert not layer.uses_mfma
    w1 = torch.zeros(E, D, F, dtype=torch.bfloat16, device="cuda:0")
    w1[:, 0, 1] = 1.0
    w2 = torch.rand(E, F, D, generator=gen, device="cuda:0").add_(0.1).bfloat16()
    x = torch.zeros(T, D, dtype=torch.bfloat16, device="cuda:0")
    x[:, 0] = 1024.0
    x[1::2, 0] = 3.0
    logits, tau = torch.randn(T, E, generator=gen, device="cuda:0"), torch.zeros(E, 1, device="cuda:0")
    layer.partition_weights(w1, w1, w2)
    clean = layer.forward(x, logits, tau).clone()
    assert torch.isfinite(clean).all()
    w2[::9, 1, 3], w2[::9, 1, 130], w2[::9, 1, 258] = inf, -inf, float("nan")
    layer.partition_weights(w1, w1, w2)
    if hot_tokens:
        x[7::500, 0] = inf
    y = layer.forward(x, logits, tau)
    torch.cuda.synchronize()
    layer.close()
    struck = (torch.topk(logits, K, dim=1).indices % 9 == 0).any(1)
    hot = torch.isinf(x[:, 0])
    assert struck.any() and not struck.all()
    cold = struck & ~hot
    assert torch.isposinf(y[cold, 3]).all() and torch.isneginf(y[cold, 130]).all() and torch.isnan(y[cold, 258]).all()
    others = [d for d in range(D) if d not in (3, 130, 258)]
    assert torch.equal(y[~hot][:, others], clean[~hot][:, others]) and torch.equal(y[~struck & ~hot], clean[~struck & ~hot])
    assert not torch.isfinite(y[hot]).any()
