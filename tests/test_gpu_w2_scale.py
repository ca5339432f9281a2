"""The power of two that moe_partition_weights gives the packed W2 comes from a sample of it (every fifth run of 2048 values at this
size): weights that only the rest of W2 has, and permutations that are none, on the matrix-core path.

Bar: W2 is exact in half precision from 2^-29 of the scale's binade up, so the outputs differ from float64 by the rounding of H and of
the partial outputs (2^-11 of the value each) and the fp32 sums: below 2e-3 of the output's RMS where many terms of like size are
added, as for any other layer, and up to 2^-10 of the value itself where one term (an outlier weight) carries the sum.
"""
import math

import pytest

pytestmark = pytest.mark.gpu

E, F, D, T = 2, 8192, 2048, 16  # E * F * D = 2^25: every fifth run is sampled
RUN = 2048


def _layer():
    from paper_2508_18376_amd import DualSparseLayer
    return DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=E, n_part=2, max_tokens=T, dtype="bf16", y_fp32=True)


def _reference(x, g, w):
    """Sum over the experts of g[:, e] f_e(x), in 64 bits."""
    import torch
    y = torch.zeros(x.shape[0], w[2].shape[2], dtype=torch.float64)
    xd = x.double().cpu()
    for e in range(w[0].shape[0]):
        a = xd @ w[0][e].double().cpu()
        y += g[:, e:e + 1] * ((a * torch.sigmoid(a) * (xd @ w[1][e].double().cpu())) @ w[2][e].double().cpu())
    return y


@pytest.mark.parametrize("kind", ["even", "within_a_binade", "outlier", "outlier_and_infinity", "sample_of_zeros", "all_zero", "last_run", "sample_of_subnormals"])
def test_w2_values_that_the_sample_misses(kind):
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(5)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda:0").mul_(0.02).bfloat16()

    w1, w3, w2 = normal(E, D, F), normal(E, D, F), normal(E, F, D)
    runs = w2.view(-1, RUN)
    if kind == "within_a_binade":
        runs[1, 7] = 2.0 * float(w2.abs().max())
    elif kind in ("outlier", "outlier_and_infinity"):
        runs[1, 7] = 40.0
    elif kind == "sample_of_zeros":
        runs[0::5] = 0
    elif kind == "sample_of_subnormals":
        w2.mul_(5e-5)  # the rest: 1e-6
        runs[0::5] = 1e-39
    elif kind == "all_zero":
        w2.zero_()
    elif kind == "last_run":  # 16384 runs: the last one is not in the sample
        runs[-1] *= 256.0
    if kind == "outlier_and_infinity":
        runs[4, 9] = float("inf")
    x = torch.randn(T, D, generator=gen, device="cuda:0").bfloat16()
    logits = torch.randn(T, E, generator=gen, device="cuda:0")
    layer = _layer()
    layer.partition_weights(w1, w3, w2)
    y = layer.forward(x, logits, torch.zeros(E, 2, device="cuda:0")).double().cpu()
    ref = _reference(x, torch.softmax(logits.double().cpu(), dim=1), (w1, w3, w2))
    good = torch.isfinite(ref)
    if kind == "outlier_and_infinity":  # the one column of the infinite weight (half-precision partial outputs saturate)
        good = torch.ones_like(good)
        good[:, 9] = False
    assert torch.isfinite(y[good]).all()
    rms = ref[good].square().mean().sqrt()
    assert ((y - ref).abs() <= 2e-3 * rms + 2.0 ** -10 * ref.abs())[good].all()
    layer.close()


@pytest.mark.parametrize("D_,F_", [(128, 256), (96, 120)])  # matrix-core and full-precision path
@pytest.mark.parametrize("kind", ["twice", "beyond", "negative", "other_expert"])
def test_bad_permutation_of_a_bf16_layer_is_rejected(D_, F_, kind):
    import torch
    from paper_2508_18376_amd import DsmoeError, DualSparseLayer
    layer = DualSparseLayer(d_model=D_, d_ff=F_, n_experts=3, top_k=1, n_part=2, max_tokens=8, dtype="bf16")
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    w1, w3, w2 = (torch.randn(s, generator=gen, device="cuda:0").bfloat16() for s in ((3, D_, F_), (3, D_, F_), (3, F_, D_)))
    good = torch.rand(3, F_, generator=gen, device="cuda:0").argsort(dim=1).to(torch.int32)
    x, logits, tau = torch.randn(8, D_, generator=gen, device="cuda:0").bfloat16(), torch.randn(8, 3, generator=gen, device="cuda:0"), torch.zeros(3, 2, device="cuda:0")
    layer.partition_weights(w1, w3, w2, perm=good)
    y = layer.forward(x, logits, tau).clone()
    bad = good.clone()
    if kind == "twice":
        bad[2, F_ - 1] = bad[2, 0]
    elif kind == "beyond":
        bad[0, 5] = F_
    elif kind == "negative":
        bad[1, 0] = -1
    else:
        bad[1] += F_
    with pytest.raises(DsmoeError) as ei:
        layer.partition_weights(w1, w3, w2, perm=bad)
    assert ei.value.status == -2
    layer.partition_weights(w1, w3, w2, perm=good)
    assert torch.equal(layer.forward(x, logits, tau), y)
    layer.close()


def test_headroom_of_partial_outputs_when_the_sample_misses_the_top_binade():
    # One weight of the next binade, which the sample does not meet.  Partial outputs are scaled by the largest weight of all: sums that
    # reach 47800 of half precision's 65504 so, and would saturate at twice that by the sample's.
    import torch
    layer = _layer()
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    x, logits, tau = torch.ones(T, D, device="cuda:0").bfloat16(), torch.randn(T, E, generator=gen, device="cuda:0"), torch.zeros(E, 2, device="cuda:0")
    w1 = torch.full((E, D, F), 1 / 256, device="cuda:0").bfloat16()
    w2 = torch.full((E, F, D), 255 / 128, device="cuda:0").bfloat16()
    w2.view(-1, RUN)[1, 7] = 2.0
    ranges = 1
    for _ in range(2):  # how many K ranges a sum is in is the plan's affair: known after a call
        gate, up = D / 256, 3000.0 * ranges / F / 8.0
        w3 = torch.full((E, D, F), up / D, device="cuda:0").bfloat16()
        layer.partition_weights(w1, w3, w2)
        y = layer.forward(x, logits, tau).double().cpu()
        ranges = int(layer.plan(T)["counters"][3])
    h = gate / (1 + math.exp(-gate)) * D * float(w3[0, 0, 0])
    ref = h * w2.double().sum(1).cpu()  # [E][D]
    ref = torch.softmax(logits.double().cpu(), dim=1) @ ref
    assert 2.9e3 < h * F / ranges < 3.1e3
    assert ((y - ref).abs() <= 2e-3 * ref).all()
    layer.close()


@pytest.mark.parametrize("where,h_scale", [("routed", 0), ("routed", 6), ("shared", -4)])
def test_a_weight_beyond_the_sample_rescales_its_column_tile_alone(where, h_scale):
    # Weights 2^-41 of the outlier's size, in another column tile: nothing is left of them at the outlier's scale (half precision reaches
    # down to 2^-39 of the largest), and they are exact at the sample's.  Partial outputs in fp32: those in half precision share one scale.
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(6)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda:0").mul_(0.02).bfloat16()

    sh = dict(n_shared=1, d_ff_shared=F) if where == "shared" else {}
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=E, n_part=2, max_tokens=T, dtype="bf16", y_fp32=True, partial_fp32=True,
                            h_scale_log2=h_scale, **sh)
    w = [normal(E, D, F), normal(E, D, F), normal(E, F, D)]
    shared = [normal(1, D, F), normal(1, D, F), normal(1, F, D)] if sh else None
    for m in (w, shared):
        if m:
            m[2][:, :, 512:768] *= 2.0 ** -20
    perm = torch.rand(E, F, generator=gen, device="cuda:0").argsort(dim=1).to(torch.int32)
    (shared or w)[2].view(-1, RUN)[1, 7] = 3e4  # neuron 1 of the first expert, column 7
    x, logits = torch.randn(T, D, generator=gen, device="cuda:0").bfloat16(), torch.randn(T, E, generator=gen, device="cuda:0")
    layer.partition_weights(*w, perm=perm, **(dict(zip(("sh_w1", "sh_w3", "sh_w2"), shared)) if shared else {}))
    y = layer.forward(x, logits, torch.zeros(E, 2, device="cuda:0")).double().cpu()
    layer.close()
    g = torch.softmax(logits.double().cpu(), dim=1)
    ref = _reference(x, g, w) + (_reference(x, torch.ones(T, 1, dtype=torch.float64), shared) if shared else 0.0)
    for cols in (slice(0, 256), slice(256, 512), slice(512, 768), slice(768, D)):
        r = ref[:, cols]
        assert ((y[:, cols] - r).abs() <= 2e-3 * r.square().mean().sqrt() + 2.0 ** -10 * r.abs()).all(), cols


@pytest.mark.parametrize("tokens", [16, 300])  # streaming kernels; full, tall and ragged row tiles
@pytest.mark.parametrize("partial_fp32", [False, True])
def test_column_tiles_of_several_scales(tokens, partial_fp32):
    # outliers of several binades in some column tiles of routed and shared experts, one in the last tile of 32 columns and two in one tile,
    # where each decides its own scale; the outputs of all tiles add up
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    D_, F_ = 2080, 4096
    gen = torch.Generator(device="cuda:0").manual_seed(8)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda:0").mul_(0.02).bfloat16()

    layer = DualSparseLayer(d_model=D_, d_ff=F_, n_experts=3, top_k=3, n_part=2, n_shared=2, d_ff_shared=1024, max_tokens=tokens, dtype="bf16",
                            y_fp32=True, partial_fp32=partial_fp32)
    w = [normal(3, D_, F_), normal(3, D_, F_), normal(3, F_, D_)]
    shared = [normal(2, D_, 1024), normal(2, D_, 1024), normal(2, 1024, D_)]
    for e, neuron, col, v in ((0, 1, 5, 0.6), (0, 2, 300, 1.5), (0, 4093, 301, -5.0), (2, 3, 2079, 3.0)):
        assert ((e * F_ + neuron) * D_ + col) // RUN % 3  # (every third run is sampled)
        w[2][e, neuron, col] = v
    perm = torch.rand(3, F_, generator=gen, device="cuda:0").argsort(dim=1).to(torch.int32)
    x, logits = torch.randn(tokens, D_, generator=gen, device="cuda:0").bfloat16(), torch.randn(tokens, 3, generator=gen, device="cuda:0")
    for sh_outlier in (0.02, -6.0):  # (the shared experts' W2 is sampled whole: with the second nothing is beyond the sample)
        shared[2][1, 7, 2050] = sh_outlier
        layer.partition_weights(*w, perm=perm, sh_w1=shared[0], sh_w3=shared[1], sh_w2=shared[2])
        y = layer.forward(x, logits, torch.zeros(3, 2, device="cuda:0")).double().cpu()
        ref = _reference(x, torch.softmax(logits.double().cpu(), dim=1), w) + _reference(x, torch.ones(tokens, 2, dtype=torch.float64), shared)
        assert ((y - ref).abs() <= 2e-3 * ref.square().mean().sqrt() + 2.0 ** -10 * ref.abs()).all()
    layer.close()
