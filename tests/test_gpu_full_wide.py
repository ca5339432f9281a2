"""GPU: the full-precision path's tiles of two weight images (large batches on layers of many experts): tiles with one image, pieces of
one image, one to four blocks of 32 rows, K splits, sums of one sign, and infinities.
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
    assert tau_kind != 0.0 or layer.plan(T)["counters"][0] < images  # at least one tile per expert and partition: not of single images
    layer.close()
    # the fp32 bar, 1e-5 x RMS, token by token: rounding scales with a token's own output, and the tokens of the two favoured experts have
    # outputs some ten times those of the others (whose softmax spreads over 512 experts)
    ref = oracle_forward(oracle, spec, t, tau)
    rms = np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True))
    assert (np.abs(to_host64(y, "f32") - ref) <= 1e-5 * rms).all()


def _positive_layer(T, D, F, E, K):
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    def rand(*s):
        return torch.rand(*s, generator=gen, device="cuda:0")
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=1, max_tokens=T, dtype="f32")
    w1, w3, w2 = rand(E, D, F).mul_(0.01), rand(E, D, F).mul_(0.01), rand(E, F, D).mul_(0.01)
    layer.partition_weights(w1, w3, w2)
    return layer, w1, w3, w2, rand(T, D), torch.randn(T, E, generator=gen, device="cuda:0")


def test_sums_of_one_sign():
    """The matrix instruction cuts its sums off: without rounded additions in between, 2048 terms of one sign come out 1e-5 short.
    Each of the three products may be off by half a unit for each of its at most 64 rounded additions (64 * 2^-25) and a unit for each of
    the twelve products summed before (12 * 2^-24), 2.6e-6, and the product of the first two sums by twice that."""
    import torch
    T, D, F, E, K = 256, 2048, 1024, 64, 8
    layer, w1, w3, w2, x, logits = _positive_layer(T, D, F, E, K)
    y = layer.forward(x, logits, torch.zeros(E, 1, device="cuda:0")).double()
    s = torch.softmax(logits.double(), 1)
    idx = torch.topk(logits, K, dim=1).indices
    ref = torch.zeros(T, D, dtype=torch.float64, device="cuda:0")
    for e in range(E):
        t = (idx == e).any(1).nonzero().flatten()
        g = x[t].double() @ w1[e].double()
        h = g * torch.sigmoid(g) * (x[t].double() @ w3[e].double())
        ref.index_add_(0, t, s[t, e].unsqueeze(1) * (h @ w2[e].double()))
    torch.cuda.synchronize()
    layer.close()
    assert ((y - ref).abs() / ref).max().item() <= 3 * 2.6e-6


def test_infinite_tokens():
    """A token with an infinite value has infinite outputs (all weights are positive), the others what they have without it."""
    import torch
    T, D, F, E, K = 2100, 256, 128, 512, 8
    layer, w1, w3, w2, x, logits = _positive_layer(T, D, F, E, K)
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
