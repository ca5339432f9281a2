"""GPU, fp32 layers: blocks of 16 pair rows, under whole weight tiles and halves of them (up to 16 pairs per expert of the whole router all items are cut,
from 32 on the last ones of the list, in between none), against the oracle.  One to eight blocks, the last one with 1, 15 or 16 rows.
"""
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev, to_host64, assert_output_close
from test_gpu_forward import spec_of, resolve_tau, oracle_forward

pytestmark = pytest.mark.gpu

ROWS = (1, 15, 16, 17, 32, 33, 47, 49, 64, 65, 80, 81, 96, 97, 112, 113, 127, 128)


@pytest.mark.parametrize("rows", ROWS)
@pytest.mark.parametrize("E,T", [(64, 128), (5, 128), (2, 130)], ids=["all_halves", "whole", "last_ones_halved"])
def test_blocks_of_rows(oracle, E, T, rows):
    import torch
    for D, Fp, window, tau_kind in ((136, 88, None, 0.0), (128, 64, (0, 2), "ragged")):
        spec = spec_of(T=T, D=D, F=2 * Fp, E=E, K=1, P=2, dtype="f32", resident=window, n_shared=1, F_sh=40, seed=400 + rows, w_std=0.05)
        t = make_layer(spec)
        t["logits"][:rows, 0] += 40.0
        t["logits"][rows:, 0] -= 40.0
        tau = resolve_tau(oracle, spec, t, tau_kind)
        layer, dev = make_gpu_layer(spec, t)
        y = layer.forward(dev["x"], dev["logits"], to_dev(tau))
        torch.cuda.synchronize()
        if tau_kind == 0.0:
            assert int(layer.plan(T)["expert_nrows"][0]) == rows
        layer.close()
        assert_output_close(to_host64(y, "f32"), oracle_forward(oracle, spec, t, tau), "f32")


def test_a_long_list_ends_in_halves(oracle):
    # more items than the 256 that are cut; what is whole and what is cut depends on the place in the list, the sums do not
    import torch
    spec = spec_of(T=2560, D=128, F=256, E=64, K=1, P=8, dtype="f32", seed=450, w_std=0.05)  # (one K stage a partition: no K splits, which would follow the list)
    t = make_layer(spec)
    layer, dev = make_gpu_layer(spec, t, renorm=True)  # (weights of one: a softmax's last bits follow the experts' order)
    tau = to_dev(resolve_tau(oracle, spec, t, 0.0))
    y = layer.forward(dev["x"], dev["logits"], tau)
    assert int(layer.plan(spec.T)["counters"][0]) > 256
    swap = torch.arange(spec.E, device="cuda:0").flip(0)  # the same experts in the opposite order
    layer.partition_weights(*(dev[k][swap].contiguous() for k in ("w1", "w3", "w2")), perm=dev["perm"][swap].contiguous())
    z = layer.forward(dev["x"], dev["logits"][:, swap].contiguous(), tau)
    torch.cuda.synchronize()
    assert int(layer.plan(spec.T)["counters"][3]) == 1
    layer.close()
    assert torch.equal(y, z)
    assert_output_close(to_host64(y, "f32"), oracle_forward(oracle, spec, t, to_host64(tau, "f32").astype("float32"), renorm=True), "f32")
