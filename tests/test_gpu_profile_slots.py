"""GPU: the per-kernel times of a profiled call name the kernels that ran: a step that another kernel does reads 0, every other one more."""
import pytest

pytestmark = pytest.mark.gpu

ALWAYS = {"plan", "gemm1", "gemm2", "combine"}


@pytest.mark.parametrize("E,K,P,T,routed,more", [
    (8, 2, 2, 64, False, set()), (8, 2, 2, 64, True, {"router"}),                                       # routed in the plan's launch
    (64, 4, 2, 300, False, {"route_mask"}), (64, 4, 2, 300, True, {"router"}),                          # ... in the router's
    (129, 4, 2, 300, True, {"router", "route_mask"}), (8, 2, 2, 2049, True, {"router", "route_mask"}),  # ... in its own
    (512, 2, 4, 300, False, {"route_mask", "scatter"}),                                                 # 19 histograms of 8192 bins
])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_slots_of_the_kernels_that_ran(E, K, P, T, routed, more, dtype):
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    from paper_2508_18376_amd.binding import dsmoe_profile_begin, dsmoe_profile_end
    D, F = 64, 32 * P
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    if dtype == "f32" and routed and E == 64:
        more = {"router", "route_mask"}  # (the router of fp32 layers does not route)
    gen = torch.Generator(device="cuda:0").manual_seed(3)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda:0").to(dt)

    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=P, max_tokens=T, dtype=dtype)
    layer.partition_weights(normal(E, D, F), normal(E, D, F), normal(E, F, D))
    layer.pack_router(normal(D, E))
    x, tau = normal(T, D), torch.zeros(E, P, device="cuda:0")
    logits = layer.router_logits(x)
    for _ in range(2):
        dsmoe_profile_begin(layer.ctx, 2, 3)
        for _ in range(4):  # (the last one is not recorded)
            layer.forward_routed(x, tau) if routed else layer.forward(x, logits, tau)
        ms, calls = dsmoe_profile_end(layer.ctx)
        assert calls == 3
        assert {k for k, v in ms.items() if v > 0.0} == ALWAYS | more, ms
    layer.close()
