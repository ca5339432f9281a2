"""GPU: the order in which the work lists are handed out, where it changes: lists of about one round of workgroups, and of so
many that the last pieces are handed out one by one, and layers whose shared experts have one row tile or several.
"""
import numpy as np
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev, to_host64, assert_output_close
from plan_cover import check_cover
from test_gpu_forward import spec_of, resolve_tau, oracle_forward

pytestmark = pytest.mark.gpu


def _check(oracle, spec, tau_kind, cover=True, by_token=False):
    import torch
    t = make_layer(spec)
    tau = resolve_tau(oracle, spec, t, tau_kind)
    layer, dev = make_gpu_layer(spec, t, y_fp32=True)
    y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
    y2 = layer.forward(dev["x"], dev["logits"], to_dev(tau))  # the counts of pieces handed out start again
    torch.cuda.synchronize()
    plan = {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in layer.plan(spec.T).items()}
    if cover:
        check_cover(plan, name="order", T=spec.T, D=spec.D, F=spec.F, P=spec.P, E_res=spec.hi - spec.lo, n_shared=spec.n_shared, F_sh=spec.F_sh)
    layer.close()
    assert torch.equal(y, y2)
    ref = oracle_forward(oracle, spec, t, tau)
    if by_token:  # the fp32 bar on each token's own RMS: of many tokens with 32 neurons some have outputs of 30 x the RMS of all, and rounding as large
        assert (np.abs(to_host64(y, "f32") - ref) <= 1e-5 * np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True))).all()
    else:
        assert_output_close(to_host64(y, "f32"), ref, spec.dtype, y_fp32=True)
    return plan


EDGES = (255, 256, 257, 263, 511, 900, 1023, 1024, 1151, 1152, 1300)


@pytest.mark.parametrize("dtype,n", [("bf16", n) for n in EDGES] + [("f32", n) for n in EDGES])
def test_pieces_of_a_list_of_n_items(oracle, dtype, n):
    # one expert, one row tile, n neuron tiles
    rows, neurons = (130, 128) if dtype == "bf16" else (64, 64)
    plan = _check(oracle, spec_of(T=rows, D=32, F=neurons * n, E=1, K=1, P=1, dtype=dtype, seed=150), 0.0)
    assert plan["counters"][0] == n


@pytest.mark.parametrize("dtype,tiles,columns", [("bf16", 1, n) for n in (1024, 1100, 1152, 1300)] + [("f32", 128, 8), ("f32", 220, 5), ("f32", 144, 8), ("f32", 260, 5)])
def test_pieces_of_a_second_list_of_n_items(oracle, dtype, tiles, columns):
    # one expert, row tiles x column tiles; its few K stages are never worth a split.  (fp32 in many row tiles: the columns are also the first
    # product's K, and the rounding of its sums grows with the root of that.)
    rows, width = (70, 256) if dtype == "bf16" else (64 * tiles + 64, 128)  # (64 rows go with the tile before)
    plan = _check(oracle, spec_of(T=rows, D=width * columns, F=32, E=1, K=1, P=1, dtype=dtype, seed=153), 0.0, by_token=dtype == "f32")
    assert plan["counters"][1] == tiles * columns and plan["counters"][3] == 1


@pytest.mark.parametrize("T", [200, 256, 257, 330, 700])
def test_shared_experts_of_one_or_several_row_tiles(oracle, T):
    _check(oracle, spec_of(T=T, D=96, F=640, E=16, K=2, P=2, n_shared=2, F_sh=192, seed=151), "rate0.25")


def test_shared_experts_among_very_many_row_tiles(oracle):
    # more row tiles than the plan kernel keeps in LDS
    _check(oracle, spec_of(T=190000, D=32, F=64, E=4, K=2, P=2, n_shared=1, F_sh=32, seed=152), 0.0, cover=False)
