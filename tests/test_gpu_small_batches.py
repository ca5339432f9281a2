"""GPU: batches for which the kernels take their small-batch forms, at the edges of those forms, against the oracle.

Row counts around one row tile (an expert with one row tile is the only reader of its weight tiles, which are then loaded
with the non-temporal hint; with two, or with a short last tile taken along, they are not), around the blocks of 32 rows, and
around the 128 rows that a workgroup of the streaming kernels takes (batches of at most 64 pairs per expert on average).
"""
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev, to_host64, assert_output_close
from test_gpu_forward import spec_of, resolve_tau

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
    # 8 x 64 pairs at most: `rows` of them (about) on one expert; halves of weight tiles that do not exist; a general mask
    # leaves row tiles whose later rows keep nothing of a partition
    _check(oracle, spec_of(T=rows, D=D, F=2 * Fp, E=8, K=1, P=2, seed=140 + rows), 0.0, to_expert_0=rows)
    if rows > 100:
        _check(oracle, spec_of(T=rows, D=D, F=4 * Fp, E=8, K=2, P=4, seed=141 + rows), "ragged", to_expert_0=rows)


@pytest.mark.parametrize("E,F", [(40, 512), (64, 512), (66, 512), (64, 768)], ids=["items_160_480", "items_512", "items_528", "items_768"])
def test_streaming_with_whole_and_half_weight_tiles(oracle, E, F):
    # the numbers of items around which whole weight tiles or halves are taken (2 x 2 .. 2 x 3 neuron tiles, 2 column tiles an expert)
    _check(oracle, spec_of(T=300, D=512, F=F, E=E, K=4, P=2, seed=150, n_shared=1, F_sh=96), "rate0.25")
