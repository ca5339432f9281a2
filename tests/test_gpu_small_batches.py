"""GPU: batches for which the kernels take their small-batch forms, at the edges of those forms, against the oracle.

Row counts around one row tile (an expert with one row tile is the only reader of its weight tiles, which are then loaded
with the non-temporal hint; with two, or with a short last tile taken along, they are not) and around the blocks of 32 rows.
"""
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev, to_host64, assert_output_close
from test_gpu_forward import spec_of, resolve_tau

pytestmark = pytest.mark.gpu


def _check(oracle, spec, tau_kind, **layer_args):
    import torch
    t = make_layer(spec)
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
