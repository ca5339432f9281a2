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


def _check(oracle, spec, tau_kind, cover=True):
    import torch
    t = make_layer(spec)
    tau = resolve_tau(oracle, spec, t, tau_kind)
    layer, dev = make_gpu_layer(spec, t, y_fp32=True)
    y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
    y2 = layer.forward(dev["x"], dev["logits"], to_dev(tau))  # the counts of pieces handed out start again
    torch.cuda.synchronize()
    plan = {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in layer.plan(spec.T).items()}
    if cover and layer.uses_mfma:
        check_cover(plan, name="order", T=spec.T, D=spec.D, F=spec.F, P=spec.P, E_res=spec.hi - spec.lo, n_shared=spec.n_shared, F_sh=spec.F_sh)
    layer.close()
    assert torch.equal(y, y2)
    assert_output_close(to_host64(y, "f32"), oracle_forward(oracle, spec, t, tau), spec.dtype, y_fp32=True)
    return plan


@pytest.mark.parametrize("dtype,n", [("bf16", n) for n in (255, 256, 257, 263, 511, 900, 1023, 1024, 1151, 1152, 1300)] + [("f32", n) for n in (256, 259, 1027, 1400)])
def test_pieces_of_a_list_of_n_items(oracle, dtype, n):
    # one expert, one row tile of 130 rows (fp32: three), n neuron tiles
    rows, tiles = (130, 1) if dtype == "bf16" else (160, 3)
    plan = _check(oracle, spec_of(T=rows, D=32, F=128 * (n // tiles), E=1, K=1, P=1, dtype=dtype, seed=150), 0.0)
    if dtype == "bf16":
        assert plan["counters"][0] == n


@pytest.mark.parametrize("T", [200, 256, 257, 330, 700])
def test_shared_experts_of_one_or_several_row_tiles(oracle, T):
    _check(oracle, spec_of(T=T, D=96, F=640, E=16, K=2, P=2, n_shared=2, F_sh=192, seed=151), "rate0.25")


def test_shared_experts_among_very_many_row_tiles(oracle):
    # more row tiles than the plan kernel keeps in LDS
    _check(oracle, spec_of(T=190000, D=32, F=64, E=4, K=2, P=2, n_shared=1, F_sh=32, seed=152), 0.0, cover=False)
