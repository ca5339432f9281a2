"""GPU: the row lists and the two work lists on both sides of the lines between the ways in which they are made: a batch routed and planned
in one launch (a lane per token up to 32 experts, up to 1024 tokens and 2048 pairs), row lists written by workgroups of the plan launch,
and by the scatter kernel where the histograms are too large for that (E x sort bins x route blocks > 65536 counts).
"""
import numpy as np
import pytest

from synth import make_layer
from gpu_util import make_gpu_layer, to_dev
from plan_cover import check_cover
from test_gpu_forward import spec_of, resolve_tau

pytestmark = pytest.mark.gpu

CASES = [
    # tokens, experts, top_k, parts, shared, resident window, thresholds
    (1, 8, 2, 4, 0, None, "ragged"), (1000, 8, 2, 4, 1, None, "ragged"), (1024, 8, 2, 2, 0, (2, 7), "rate0.25"), (1025, 8, 2, 2, 0, None, "rate0.25"),
    (256, 8, 8, 3, 0, None, "ragged"), (257, 8, 8, 3, 1, None, "ragged"), (128, 32, 16, 1, 0, None, "rate0.25"), (129, 20, 16, 5, 0, (3, 20), "ragged"),
    (1024, 64, 2, 4, 1, None, "ragged"), (1025, 64, 2, 4, 0, None, "ragged"), (65, 40, 3, 1, 0, None, "rate0.25"), (2049, 33, 16, 2, 0, (0, 1), "ragged"),
    (4500, 3, 2, 8, 1, None, "ragged"), (2300, 512, 1, 1, 0, None, "rate0.25"),
    # histograms summed a bin per thread: 8192 bins (7 rows), 66 bins (no multiple of four)
    (100, 512, 16, 8, 1, None, "ragged"), (1100, 33, 3, 1, 0, None, "rate0.25"),
    # more (row tile, partition) pairs than are kept in LDS, experts of several tiles: up to 64 experts, more, and an odd number with two bins each
    (4500, 64, 8, 8, 1, None, "ragged"), (4500, 70, 8, 8, 1, (3, 70), "ragged"), (3001, 65, 4, 1, 1, None, "rate0.25"), (1000, 512, 8, 8, 0, (0, 511), "rate0.25"),
]


@pytest.mark.parametrize("T,E,K,P,n_shared,window,tau_kind", CASES)
def test_rows_and_lists(oracle, T, E, K, P, n_shared, window, tau_kind):
    import torch
    spec = spec_of(T=T, D=64, F=32 * P, E=E, K=K, P=P, n_shared=n_shared, F_sh=32, resident=window, seed=300 + T, w_std=0.05)
    t = make_layer(spec)
    tau = resolve_tau(oracle, spec, t, tau_kind)
    layer, dev = make_gpu_layer(spec, t)
    layer.forward(dev["x"], dev["logits"], to_dev(tau))
    torch.cuda.synchronize()
    plan = {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in layer.plan(T).items()}
    _, _, keep, _ = layer.route_and_mask(dev["logits"], to_dev(tau))
    keep = keep.cpu().numpy()
    layer.close()
    assert np.array_equal(plan["keep_bits"], keep)
    row, e = plan["pair_row"], plan["topk_idx"] - spec.lo
    kept = keep != 0
    assert np.array_equal(row >= 0, kept)
    assert len(np.unique(row[kept])) == kept.sum()
    tokens = np.broadcast_to(np.arange(T)[:, None], row.shape)
    assert np.array_equal(plan["row_token"][row[kept]], tokens[kept]) and np.array_equal(plan["row_bits"][row[kept]], keep[kept])
    first, rows = plan["expert_row0"][e[kept]], plan["expert_nrows"][e[kept]]
    assert np.all(row[kept] >= first) and np.all(row[kept] < first + rows) and plan["expert_nrows"].sum() == kept.sum()
    if n_shared:
        assert np.array_equal(plan["row_token"][:T], np.arange(T)) and np.all(plan["row_bits"][:T] == 1)
    check_cover(plan, name="rows", T=T, D=spec.D, F=spec.F, P=P, E_res=spec.hi - spec.lo, n_shared=n_shared, F_sh=spec.F_sh)
