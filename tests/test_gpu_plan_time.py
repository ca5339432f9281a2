"""GPU: the plan adds the histograms of the route blocks up many at a time, whatever their number of bins: its time for bins that are no multiple
of four, and for more than 4096 of them.  Bars: twice what it takes and more, half of what one load after the other takes.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,P,us", [(257, 1, 55.0), (512, 8, 300.0)])  # 26 and 121 us; one load after the other: 85 and 603
def test_plan_time_of_many_histograms(E, P, us):
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    from paper_2508_18376_amd.binding import dsmoe_profile_begin, dsmoe_profile_end
    D, F, K, T = 64, 32 * P, 8, 16384
    gen = torch.Generator(device="cuda:0").manual_seed(4)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda:0").bfloat16()

    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=P, max_tokens=T, dtype="bf16")
    layer.partition_weights(normal(E, D, F), normal(E, D, F), normal(E, F, D))
    x, logits = normal(T, D), torch.randn(T, E, generator=gen, device="cuda:0")
    tau = (torch.rand(E, P, generator=gen, device="cuda:0").cumsum(1) * (0.8 / (K * P))).contiguous()
    layer.forward(x, logits, tau)
    best = float("inf")
    for _ in range(3):
        dsmoe_profile_begin(layer.ctx, 2, 10)
        for _ in range(10):
            layer.forward(x, logits, tau)
        best = min(best, dsmoe_profile_end(layer.ctx)[0]["plan"] * 1e3)
    layer.close()
    assert best < us
