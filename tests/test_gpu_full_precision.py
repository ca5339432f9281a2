"""GPU: the full-precision path (fp32 layers, bf16 layers off the matrix-core grid) at the edges of its tiles: row counts
around 32, 64 and 128 (blocks, tiles, a short last tile taken along), widths that need padding of every K dimension,
activations that need a padded copy, K splits, and a batch of the static entry point that leaves no room for them.

Both types keep fp32 intermediates and accumulate in fp32, bf16 products are exact: with the output stored as fp32 the
fp32 bar (1e-5 x RMS of the oracle's output) holds for both.
"""
import numpy as np
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev, to_host64, tau_table, rel_err
from test_gpu_forward import spec_of, resolve_tau

pytestmark = pytest.mark.gpu

SHAPES = [
    ("rows_1", dict(T=1, D=128, F=176, E=1, K=1, P=1), 0.0),
    ("rows_32", dict(T=32, D=128, F=176, E=1, K=1, P=1), 0.0),
    ("rows_33", dict(T=33, D=128, F=176, E=1, K=1, P=1), 0.0),
    ("rows_65", dict(T=65, D=128, F=176, E=1, K=1, P=1), 0.0),
    ("rows_97", dict(T=97, D=128, F=176, E=1, K=1, P=1), 0.0),
    ("rows_128", dict(T=128, D=128, F=176, E=1, K=1, P=1), 0.0),
    ("rows_129", dict(T=129, D=128, F=176, E=1, K=1, P=1), 0.0),
    ("rows_200_two_column_tiles", dict(T=200, D=260, F=176, E=1, K=1, P=1), 0.0),
    ("padded_everywhere", dict(T=150, D=73, F=99, E=3, K=2, P=3), "rate0.3"),
    ("odd_shared", dict(T=100, D=130, F=72, E=4, K=2, P=2, n_shared=2, F_sh=27), "rate0.3"),
    ("general_masks", dict(T=230, D=96, F=104, E=4, K=3, P=4), "ragged"),
    ("split_k", dict(T=9, D=200, F=1056, E=4, K=2, P=2), 0.0),
    ("split_k_under_drop", dict(T=70, D=136, F=2080, E=4, K=2, P=4), "rate0.25"),
    ("split_k_odd_width", dict(T=80, D=131, F=1056, E=2, K=2, P=1), 0.0),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name,shape,tau_kind", SHAPES, ids=[s[0] for s in SHAPES])
def test_full_precision_tiles(oracle, name, shape, tau_kind, dtype):
    import torch
    spec = spec_of(dtype=dtype, seed=90, x_std=1.0, w_std=0.05, **shape)
    t = make_layer(spec)
    tau = resolve_tau(oracle, spec, t, tau_kind)
    layer, dev = make_gpu_layer(spec, t, y_fp32=True)
    if layer.uses_mfma:
        pytest.skip("the shape is on the matrix-core grid")
    print("%s %s" % (name, dtype), flush=True)
    y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
    # the same activations from an address that is no multiple of 16 bytes
    buf = torch.empty(spec.T * spec.D + 1, dtype=dev["x"].dtype, device="cuda:0")
    shifted = buf[1:].view(spec.T, spec.D)
    shifted.copy_(dev["x"])
    y2 = layer.forward(shifted, dev["logits"], to_dev(tau))
    torch.cuda.synchronize()
    ref = oracle.forward(t["x"], t["logits"], t["w1"], t["w3"], t["w2"], tau, spec.K, spec.P, perm=t["perm"],
                         sh_w1=t.get("sh_w1"), sh_w3=t.get("sh_w3"), sh_w2=t.get("sh_w2"))
    assert rel_err(to_host64(y, "f32"), ref) <= 1e-5
    assert torch.equal(y, y2)
    layer.close()


def test_infinite_activations_stay_infinite_in_the_split_product():
    """A bf16 layer whose intermediate activation overflows fp32 gives infinities (not NaN) where one term is infinite."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    layer = DualSparseLayer(d_model=40, d_ff=8, n_experts=1, top_k=1, n_part=1, max_tokens=4, dtype="bf16", y_fp32=True)
    assert not layer.uses_mfma
    w1 = torch.zeros(1, 40, 8, dtype=torch.bfloat16, device="cuda:0")
    w3, w2 = torch.zeros_like(w1), torch.zeros(1, 8, 40, dtype=torch.bfloat16, device="cuda:0")
    w1[0, 0, 0] = w3[0, 0, 0] = 2.0 ** 40
    w2[0, 0, :] = 0.5
    layer.partition_weights(w1, w3, w2)
    x = torch.zeros(2, 40, dtype=torch.bfloat16, device="cuda:0")
    x[0, 0], x[1, 0] = 2.0 ** 40, 1.0  # Swish(2^80) * 2^80 overflows; Swish(2^40) * 2^40 does not
    y = layer.forward(x, torch.zeros(2, 1, device="cuda:0"), torch.zeros(1, 1, device="cuda:0"))
    torch.cuda.synchronize()
    assert torch.isposinf(y[0]).all() and (y[1] == 2.0 ** 79).all()
    layer.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [5, 70])
@pytest.mark.parametrize("D,F,P,F_sh", [(64, 40, 5, 0), (73, 99, 3, 27), (100, 88, 2, 24)])
def test_infinite_inputs_stay_out_of_the_padding(D, F, P, F_sh, T, dtype):
    """Every weight is positive, so a token with an infinite value has infinite activations and outputs.  The neurons that pad a
    partition to whole stages have zero weights, and infinity times zero must not get into the sums."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(8)
    n_sh, dt = int(F_sh > 0), torch.float32 if dtype == "f32" else torch.bfloat16
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=2, top_k=1, n_part=P, max_tokens=T, dtype=dtype, n_shared=n_sh, d_ff_shared=F_sh, y_fp32=True)
    assert not layer.uses_mfma
    def weights(*s):
        return torch.rand(*s, generator=gen, device="cuda:0").add_(0.1).to(dt)
    sh = dict(sh_w1=weights(1, D, F_sh), sh_w3=weights(1, D, F_sh), sh_w2=weights(1, F_sh, D)) if n_sh else {}
    layer.partition_weights(weights(2, D, F), weights(2, D, F), weights(2, F, D), **sh)
    x = torch.rand(T, D, generator=gen, device="cuda:0").to(dt)
    x[1::3, 0] = float("inf")
    logits = torch.randn(T, 2, generator=gen, device="cuda:0")
    y = layer.forward(x, logits, torch.zeros(2, P, device="cuda:0"))
    importance = layer.profile_importance(x, logits, 3)
    torch.cuda.synchronize()
    layer.close()
    hot = torch.zeros(T, dtype=torch.bool, device="cuda:0")
    hot[1::3] = True
    assert torch.isposinf(y[hot]).all() and torch.isfinite(y[~hot]).all()
    assert not torch.isnan(importance).any()


@pytest.mark.parametrize("shared", [0, 1])
@pytest.mark.parametrize("T", [2, 40])
def test_infinite_weights_in_the_split_product(T, shared):
    """bf16 layers multiply W2 with three parts of an activation, of which some are zero: an infinite weight still gives an
    infinity with the activation's sign, a NaN weight NaN, and the other columns are as without them."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    D, F, inf = 40, 24, float("inf")
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=1, top_k=1, n_part=1, max_tokens=T, dtype="bf16", y_fp32=True, n_shared=shared, d_ff_shared=F * shared)
    assert not layer.uses_mfma
    def zeros(*s):
        return torch.zeros(*s, dtype=torch.bfloat16, device="cuda:0")
    w1, w3, w2 = zeros(1, D, F), zeros(1, D, F), zeros(1, F, D)
    w1[0, 0, 1] = 1.0
    w3[0, 0, 1] = 1.0
    w2[0, 1, :] = 0.5
    finite = w2.clone()
    w2[0, 1, 3], w2[0, 1, 4], w2[0, 1, 39] = inf, -inf, float("nan")
    sh = dict(sh_w1=w1, sh_w3=w3, sh_w2=w2) if shared else {}
    layer.partition_weights(w1, w3, finite if shared else w2, **sh)
    x = zeros(T, D)
    x[:, 0] = 1024.0  # Swish(1024) * 1024 = 2^20: its second and third part are zero
    x[1::2, 0] = 3.0  # all parts
    y = layer.forward(x, zeros(T, 1).float(), zeros(1, 1).float())
    torch.cuda.synchronize()
    layer.close()
    assert torch.isposinf(y[:, 3]).all() and torch.isneginf(y[:, 4]).all() and torch.isnan(y[:, 39]).all()
    others = [d for d in range(D) if d not in (3, 4, 39)]
    assert (y[::2][:, others] == 2.0 ** 19 * (1 + shared)).all()
    h3 = 9.0 / (1.0 + np.exp(-3.0))
    assert float((y[1::2][:, others] - 0.5 * h3 * (1 + shared)).abs().max()) <= 1e-5 * h3


def test_static_batch_without_room_for_k_splits(oracle):
    import torch
    import paper_2508_18376_amd as ds
    spec = spec_of(dtype="f32", T=8, D=1024, F=512, E=4, K=2, P=2, seed=91, w_std=0.05)
    t = make_layer(spec)
    T = 20000  # ~40 k rows x (512 + 1024) x 4 bytes: the array holds it only without the pool of partial-output tiles
    layer, _ = make_gpu_layer(spec, t, max_tokens=T)
    assert ds.DSMOE_STATIC_SCRATCH_BYTES - (32 << 20) < ds.dsmoe_static_workspace_need(layer.ctx, T) <= ds.DSMOE_STATIC_SCRATCH_BYTES
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    x = torch.randn(T, spec.D, generator=gen, device="cuda:0")
    logits = torch.randn(T, spec.E, generator=gen, device="cuda:0")
    tau = to_dev(tau_table(spec, np.zeros(spec.P, np.float32)))
    y = torch.empty(T, spec.D, device="cuda:0")
    ds.moe_dualsparse_forward_static(layer.ctx, layer.packed, x, logits, tau, T, y, torch.cuda.current_stream())
    ref = layer.forward(x, logits, tau)
    torch.cuda.synchronize()
    assert float((y - ref).abs().max()) <= 1e-5 * float(ref.square().mean().sqrt())
    layer.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,F,P,E,K,F_sh,T", [(1024, 264, 8, 32, 4, 0, 12287), (99, 24, 8, 8, 2, 5, 150001), (1800, 40, 8, 512, 16, 0, 135)],
                         ids=["parts_of_33", "odd_width_shared", "a_tile_of_every_expert_is_too_much"])
def test_static_batch_in_pieces(D, F, P, E, K, F_sh, T, dtype):
    """Batches that fit the static array only without the padding of the intermediate arrays: same results as with a workspace.
    (Odd widths: the later pieces of x start at any address.)"""
    import torch
    import paper_2508_18376_amd as ds
    gen = torch.Generator(device="cuda:0").manual_seed(12)
    n_sh, dt = int(F_sh > 0), torch.float32 if dtype == "f32" else torch.bfloat16
    layer = ds.DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=P, max_tokens=T, dtype=dtype, n_shared=n_sh, d_ff_shared=F_sh, y_fp32=True)
    assert not layer.uses_mfma
    def normal(*s, std=0.05):
        return (torch.randn(*s, generator=gen, device="cuda:0") * std).to(dt)
    sh = dict(sh_w1=normal(1, D, F_sh), sh_w3=normal(1, D, F_sh), sh_w2=normal(1, F_sh, D)) if n_sh else {}
    layer.partition_weights(normal(E, D, F), normal(E, D, F), normal(E, F, D), **sh)
    x, logits = normal(T, D, std=1.0), torch.randn(T, E, generator=gen, device="cuda:0")
    tau = torch.full((E, P), 0.5 / K, device="cuda:0")
    y = torch.full((T, D), float("nan"), device="cuda:0")
    ds.moe_dualsparse_forward_static(layer.ctx, layer.packed, x, logits, tau, T, y, torch.cuda.current_stream())
    ref = layer.forward(x, logits, tau)
    torch.cuda.synchronize()
    layer.close()
    assert float((y - ref).abs().max()) <= 1e-5 * float(ref.square().mean().sqrt())


@pytest.mark.parametrize("D", [4100, 4101], ids=["padded_copy", "and_outputs_one_by_one"])
def test_more_values_than_a_launch_has_threads(D):
    """A padded copy of x, and outputs whose rows are not whole vectors, of more than 2^32 values: 1048448 tokens, 34 GB in all."""
    import torch
    import paper_2508_18376_amd as ds
    gen = torch.Generator(device="cuda:0").manual_seed(14)
    F, n, times = 4, 8191, 128
    layer = ds.DualSparseLayer(d_model=D, d_ff=F, n_experts=1, top_k=1, n_part=1, max_tokens=n * times, dtype="bf16")
    assert not layer.uses_mfma and n * times * 4128 > 2 ** 32 and (D % 4 == 0 or n * times * D > 2 ** 32)
    w = [torch.randn(1, *s, generator=gen, device="cuda:0").mul_(0.05).bfloat16() for s in ((D, F), (D, F), (F, D))]
    layer.partition_weights(*w)
    x = torch.randn(n, D, generator=gen, device="cuda:0").bfloat16()
    tau = torch.zeros(1, 1, device="cuda:0")
    ref = layer.forward(x, torch.zeros(n, 1, device="cuda:0"), tau).float()
    y = layer.forward(x.repeat(times, 1), torch.zeros(n * times, 1, device="cuda:0"), tau)
    torch.cuda.synchronize()
    layer.close()
    bound = 2.0 ** -7 * ref.abs() + 1e-5 * ref.square().mean().sqrt()  # two roundings to bf16 of sums that differ by 1e-5 x RMS
    for part in (0, 1, times // 2, times - 1):
        assert bool(((y[part * n:(part + 1) * n].float() - ref).abs() <= bound).all())
