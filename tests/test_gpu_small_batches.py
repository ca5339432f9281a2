"""GPU: batches for which the kernels take their small-batch forms, at the edges of those forms, against the oracle.

Row counts around one row tile (an expert with one row tile is the only reader of its weight tiles, which are then loaded
with the non-temporal hint; with two, or with a short last tile taken along, they are not), around the blocks of 32 rows, and
around the 64 tokens up to which a batch takes the streaming kernels.
"""
import numpy as np
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev, to_host64, assert_output_close
from test_gpu_forward import spec_of, resolve_tau, oracle_forward

pytestmark = pytest.mark.gpu


def _check(oracle, spec, tau_kind, to_expert_0=0, **layer_args):
    import torch
    t = make_layer(spec)
    t["logits"][:to_expert_0, 0] += 4.0  # these tokens' first choice
    tau = resolve_tau(oracle, spec, t, tau_kind)
    layer, dev = make_gpu_layer(spec, t, y_fp32=True, **layer_args)
    y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
    torch.cuda.synchronize()
    layer.close()
    ref = oracle.forward(t["x"], t["logits"], t["w1"], t["w3"], t["w2"], tau, spec.K, spec.P, perm=t["perm"],
                         sh_w1=t.get("sh_w1"), sh_w3=t.get("sh_w3"), sh_w2=t.get("sh_w2"))
    assert_output_close(to_host64(y, "f32"), ref, spec.dtype, y_fp32=True)


@pytest.mark.parametrize("tall", [0, 1])
@pytest.mark.parametrize("T", [1, 32, 33, 129, 255, 256, 257, 320, 321, 513])
def test_rows_around_one_row_tile(oracle, T, tall):
    # one routed expert (all T rows) and one shared pseudo-expert (T rows too)
    _check(oracle, spec_of(T=T, D=128, F=384, E=1, K=1, P=1, n_shared=1, F_sh=256, seed=100 + T), 0.0, tall_items=tall)


@pytest.mark.parametrize("T", [40, 300, 700])
def test_one_tile_experts_beside_larger_ones(oracle, T):
    _check(oracle, spec_of(T=T, D=128, F=512, E=6, K=2, P=2, seed=130), "rate0.25")


@pytest.mark.parametrize("rows", [1, 31, 33, 64, 65, 97, 128, 129, 160, 255, 256, 257])
@pytest.mark.parametrize("D,Fp", [(96, 32), (160, 160), (320, 192)], ids=["no_second_halves", "short_last_tiles", "two_column_tiles"])
def test_streaming_rows_of_one_expert(oracle, rows, D, Fp):
    # `rows` pairs (about) on one expert, up to 64 of them in the streaming kernels; halves of weight tiles that do not exist; a general mask
    # leaves row tiles whose later rows keep nothing of a partition
    _check(oracle, spec_of(T=rows, D=D, F=2 * Fp, E=8, K=1, P=2, seed=140 + rows), 0.0, to_expert_0=rows)
    if rows > 100:
        _check(oracle, spec_of(T=rows, D=D, F=4 * Fp, E=8, K=2, P=4, seed=141 + rows), "ragged", to_expert_0=rows)


@pytest.mark.parametrize("T", [1, 2, 15, 16, 17])
@pytest.mark.parametrize("D,Fp", [(32, 32), (160, 96), (1056, 160), (2208, 288)], ids=["one_stage", "five_stages", "stages_33", "stages_69"])
def test_few_rows(oracle, T, D, Fp):
    # a few tokens: K of 1, 5, 33 and 69 stages; last neuron tiles of 32 to 96 neurons; whole items and halves (up to 128 items the list is
    # cut); rows that keep nothing of a partition
    _check(oracle, spec_of(T=T, D=D, F=2 * Fp, E=8, K=2, P=2, n_shared=1, F_sh=Fp, seed=170 + T), "ragged", to_expert_0=T)
    _check(oracle, spec_of(T=T, D=D, F=4 * Fp, E=24, K=16, P=4, seed=171 + T), "rate0.25")


@pytest.mark.parametrize("T", [64, 65, 300, 511])
def test_hot_expert_in_a_batch_of_few_rows_on_average(oracle, T):
    """All first choices on one of 32 experts: from 257 of its rows on tall items take its short last tile along, and a weight
    tile that is marked as read once has one item of at most a row tile."""
    import torch
    spec = spec_of(T=T, D=96, F=256, E=32, K=2, P=2, seed=145)
    t = make_layer(spec)
    t["logits"][:, 0] += 8.0
    tau = resolve_tau(oracle, spec, t, 0.0)
    layer, dev = make_gpu_layer(spec, t, y_fp32=True, tall_items=1)
    y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
    torch.cuda.synchronize()
    plan = layer.plan(T)
    layer.close()
    ref = oracle.forward(t["x"], t["logits"], t["w1"], t["w3"], t["w2"], tau, spec.K, spec.P, perm=t["perm"])
    assert_output_close(to_host64(y, "f32"), ref, spec.dtype, y_fp32=True)
    rows = int(plan["expert_nrows"][0])
    tallest = rows if rows <= 256 + 64 else 256
    assert rows == T and int(plan["items2"][:, 1].max()) == tallest and int(plan["items1"][:, 1].max()) == tallest


@pytest.mark.parametrize("T", [60, 300])  # (60: every expert has rows, in the streaming kernels)
@pytest.mark.parametrize("E,F", [(40, 512), (64, 512), (66, 512), (64, 768)], ids=["items_160_480", "items_512", "items_528", "items_768"])
def test_streaming_with_whole_and_half_weight_tiles(oracle, E, F, T):
    # the numbers of items around which whole weight tiles or halves are taken (2 x 2 .. 2 x 3 neuron tiles, 2 column tiles an expert)
    _check(oracle, spec_of(T=T, D=512, F=F, E=E, K=4, P=2, seed=150, n_shared=1, F_sh=96), "rate0.25")


@pytest.mark.parametrize("dtype,D", [("bf16", 96), ("bf16", 320), ("f32", 72), ("f32", 260)])
@pytest.mark.parametrize("K,n_shared", [(1, 0), (2, 1), (16, 0), (16, 1)])
def test_combine_with_one_thread_per_slot(oracle, dtype, D, K, n_shared):
    # one slot to seventeen, column groups that do not fill a workgroup, partial outputs of split K ranges (few row tiles)
    spec = spec_of(T=3, D=D, F=1024, E=max(K, 2), K=K, P=2, dtype=dtype, n_shared=n_shared, F_sh=256, seed=160, w_std=0.05)
    _check(oracle, spec, "rate0.25" if K > 1 else 0.0)


def test_combine_on_both_sides_of_the_small_batch_line():
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    D, F, E, T = 512, 128, 4, 513  # 64 column groups: 512 tokens still take the small-batch kernel
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=2, n_part=1, max_tokens=T)
    w = [torch.randn(E, *s, generator=gen, device="cuda:0", dtype=torch.bfloat16) * 0.05 for s in ((D, F), (D, F), (F, D))]
    layer.partition_weights(*w)
    x = torch.randn(T, D, generator=gen, device="cuda:0", dtype=torch.bfloat16)
    logits, tau = torch.randn(T, E, generator=gen, device="cuda:0"), torch.zeros(E, 1, device="cuda:0")
    y = layer.forward(x, logits, tau)
    assert torch.equal(layer.forward(x[:512].contiguous(), logits[:512].contiguous(), tau), y[:512])  # the same sums in the same order
    layer.close()


@pytest.mark.parametrize("n_shared", [0, 1])
@pytest.mark.parametrize("dtype,T", [("bf16", 512), ("f32", 256)])
def test_tokens_without_a_kept_pair_on_both_sides_of_the_small_batch_line(dtype, T, n_shared):
    """Tokens whose scores are NaN (all logits -inf, as for masked padding; a logit of +inf; a NaN one, with a lane per token)
    or all below the thresholds keep nothing: their output is the shared experts' alone, exact zeros without any, from
    both combine kernels (512 columns: 64 groups of 8 bf16, 128 of 4 fp32 values, up to 32768 in the small-batch kernel)."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    D, F, E, dt = 512, 128, 4, torch.bfloat16 if dtype == "bf16" else torch.float32
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=2, n_part=1, max_tokens=T + 1, dtype=dtype, n_shared=n_shared,
                            d_ff_shared=64 * n_shared, y_fp32=True)
    def normal(*s, std=1.0):
        return (torch.randn(*s, generator=gen, device="cuda:0") * std).to(dt)
    sh = dict(sh_w1=normal(1, D, 64, std=0.05), sh_w3=normal(1, D, 64, std=0.05), sh_w2=normal(1, 64, D, std=0.05)) if n_shared else {}
    layer.partition_weights(normal(E, D, F, std=0.05), normal(E, D, F, std=0.05), normal(E, F, D, std=0.05), **sh)
    x, logits = normal(T + 1, D), torch.randn(T + 1, E, generator=gen, device="cuda:0")
    tau = torch.full((E, 1), 0.4, device="cuda:0")  # one pair of most tokens is dropped, the other kept
    shared_only = layer.forward(x, logits, torch.full((E, 1), 2.0, device="cuda:0"))
    if not n_shared:
        assert torch.equal(shared_only, torch.zeros_like(shared_only))
    nan = float("nan")
    for i, row in enumerate(([-float("inf")] * 4, [float("inf"), 0.0, 0.0, 0.0], [nan, 0.0, 0.0, 0.0], [nan] * 4)):
        logits[i::16] = torch.tensor(row, device="cuda:0")
    small = layer.forward(x[:T].contiguous(), logits[:T].contiguous(), tau)
    large = layer.forward(x, logits, tau)
    torch.cuda.synchronize()
    layer.close()
    assert bool(torch.isfinite(small).all()) and bool(torch.isfinite(large).all())
    rms = float(large.square().mean().sqrt())
    tol = (2e-2 if dtype == "bf16" else 1e-5) * rms
    for i in range(4):
        assert float((small[i::16] - shared_only[:T][i::16]).abs().max()) <= (tol if n_shared else 0.0)
        assert float((large[i::16] - shared_only[i::16]).abs().max()) <= (tol if n_shared else 0.0)
    assert float((small - large[:T]).abs().max()) <= tol


@pytest.mark.parametrize("T", [1, 15, 17, 4096, 4097])
@pytest.mark.parametrize("D,E", [(64, 3), (320, 40), (2112, 64), (128, 130)])
def test_router_token_blocks(T, D, E):
    """Workgroups of 16 and of 32 tokens, tiles of 16 experts, steps of 64 that do not fill every wavefront.  Products of bf16
    values are exact, the sum of D of them in fp32 errs by at most (D + 16) x 2^-24 of the sum of their magnitudes."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(T + D)
    layer = DualSparseLayer(d_model=D, d_ff=32, n_experts=E, top_k=2, n_part=1, max_tokens=T)
    wg = torch.randn(D, E, generator=gen, device="cuda:0", dtype=torch.bfloat16)
    x = torch.randn(T, D, generator=gen, device="cuda:0", dtype=torch.bfloat16)
    layer.pack_router(wg)
    got = layer.router_logits(x).cpu().double()
    ref, mag = x.cpu().double() @ wg.cpu().double(), x.cpu().double().abs() @ wg.cpu().double().abs()
    assert bool(((got - ref).abs() <= (D + 16) * 2.0 ** -24 * mag).all())
    layer.close()


@pytest.mark.parametrize("T", [1, 63, 64, 65])
@pytest.mark.parametrize("E,K,P,n_shared,window", [(8, 2, 4, 0, None), (9, 3, 8, 1, (2, 7)), (32, 8, 2, 0, None), (33, 16, 5, 0, (30, 33)),
                                                   (64, 8, 2, 1, None), (65, 4, 2, 0, None)])
def test_lists_of_batches_planned_in_one_launch(oracle, T, E, K, P, n_shared, window):
    # both sides of 64 tokens and of 64 experts, the three ways a workgroup routes (up to 8, 32 and 64 experts)
    import torch
    from plan_cover import check_cover
    spec = spec_of(T=T, D=64, F=64 * P, E=E, K=K, P=P, n_shared=n_shared, F_sh=64, resident=window, seed=170)
    t = make_layer(spec)
    tau = resolve_tau(oracle, spec, t, "ragged")
    r = oracle.route(t["logits"], K, P, tau, spec.lo, spec.hi)
    layer, dev = make_gpu_layer(spec, t)
    layer.forward(dev["x"], dev["logits"], to_dev(tau))
    torch.cuda.synchronize()
    plan = {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in layer.plan(T).items()}
    layer.close()
    np.testing.assert_array_equal(plan["topk_idx"], r.idx)
    np.testing.assert_array_equal(plan["keep_bits"], r.keep_bits)
    assert np.array_equal(plan["pair_row"] < 0, r.keep_bits == 0)
    at = plan["pair_row"][r.keep_bits != 0]
    assert len(np.unique(at)) == len(at)
    np.testing.assert_array_equal(plan["row_token"][at], np.nonzero(r.keep_bits)[0])
    np.testing.assert_array_equal(plan["row_bits"][at], r.keep_bits[r.keep_bits != 0])
    experts = r.idx[r.keep_bits != 0] - spec.lo
    row0, n = plan["expert_row0"][experts], plan["expert_nrows"][experts]
    assert np.all((at >= row0) & (at < row0 + n)) and plan["expert_nrows"].sum() == len(at)
    check_cover(plan, name="small", T=T, D=spec.D, F=spec.F, P=P, E_res=spec.hi - spec.lo, n_shared=n_shared, F_sh=spec.F_sh)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,E", [(1, 1), (16, 1), (17, 1), (33, 8), (70, 8), (100, 8), (128, 8), (129, 8)])
def test_full_precision_halves_of_weight_tiles(oracle, rows, E, dtype):
    # both sides of 16 pairs per expert on average; one to four blocks of 32 rows under half a weight tile; the last neuron tile
    # of a partition (44 of 64 neurons, 12 of 64) and the last column tile (136 of 2 x 128) end inside one of the halves
    for F in (88, 152):
        _check(oracle, spec_of(T=rows, D=136, F=F, E=E, K=1, P=2, dtype=dtype, n_shared=1, F_sh=40, seed=180 + rows, w_std=0.05), 0.0,
               to_expert_0=rows if E > 1 else 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [4, 5, 64, 65])
def test_full_precision_halves_of_weight_tiles_on_a_resident_window(oracle, T, dtype):
    # 16 pairs per expert of the whole layer (64 tokens) and of the window alone (4 tokens), one step on either side of both
    spec = spec_of(T=T, D=136, F=88, E=16, K=4, P=2, dtype=dtype, resident=(3, 4), n_shared=1, F_sh=40, seed=190 + T, w_std=0.05)
    t = make_layer(spec)
    tau = resolve_tau(oracle, spec, t, 0.0)
    layer, dev = make_gpu_layer(spec, t, y_fp32=True)
    y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
    layer.close()
    ref = oracle_forward(oracle, spec, t, tau)
    assert_output_close(to_host64(y, "f32"), ref, spec.dtype, y_fp32=True)


@pytest.mark.parametrize("E,F,D,where", [(1, 32, 32, 0), (1, 32, 32, -1), (2, 96, 160, 9), (8, 1024, 2048, 2048 * 256 * 8 - 1), (8, 1024, 2048, -1),
                                         (9, 1024, 2048, -8), (33, 1024, 2048, 4 * 2048 * 256 * 8 - 8), (33, 1024, 2048, -1)])
@pytest.mark.parametrize("offset", [0, 1])
def test_scale_of_the_largest_w2(E, F, D, where, offset):
    """W2 is scaled by a power of two that its largest value decides, wherever that sits: in the four loads at a time, the single ones
    behind them, or a tensor at any address.  Were it missed, it would overflow half precision."""
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    gen = torch.Generator(device="cuda:0").manual_seed(20)
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=1, n_part=1, max_tokens=E, y_fp32=True)
    assert layer.uses_mfma
    w1 = torch.randn(E, D, F, generator=gen, device="cuda:0").mul_(D ** -0.5).bfloat16()
    w2 = torch.zeros(E * F * D + offset, dtype=torch.bfloat16, device="cuda:0")[offset:]
    w2[::7] = 1e-3
    w2[where] = 4096.0
    layer.partition_weights(w1, w1, w2.view(E, F, D))
    x = torch.randn(E, D, generator=gen, device="cuda:0").bfloat16()
    y = layer.forward(x, 10.0 * torch.eye(E, device="cuda:0"), torch.zeros(E, 1, device="cuda:0"))
    torch.cuda.synchronize()
    layer.close()
    e, f, d = np.unravel_index(where % (E * F * D), (E, F, D))
    gate = (x[e].double() @ w1[e, :, f].double()).item()
    g = 1.0 / (1.0 + (E - 1) * np.exp(-10.0))
    want = g * gate * gate / (1.0 + np.exp(-gate)) * 4096.0
    assert abs(float(y[e, d]) - want) <= 2e-2 * max(abs(want), 4096.0)
