"""The router product and the routing of its batch in one launch (33 to 128 experts, up to 2048 tokens) against the two launches: the same
arithmetic on the same logits, so the plan's arrays and the outputs are equal bit for bit.  Sizes at the edges of the rule (experts, tokens),
of the workgroups of 16 tokens, of the chunks of 64 experts, and of the launches that route in the plan (up to 64 tokens).
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,K,P,window", [(33, 3, 2, None), (62, 6, 2, (5, 40)), (64, 8, 4, None), (65, 8, 5, None), (96, 5, 1, (0, 96)),
                                          (128, 16, 2, (100, 128)), (129, 4, 2, None), (32, 4, 2, None)])
@pytest.mark.parametrize("T", [1, 15, 17, 64, 65, 333, 2048, 2049])
def test_routed_in_one_launch_as_in_two(E, K, P, window, T):
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    D, F = 192, 32 * P
    lo, hi = window or (0, E)
    gen = torch.Generator(device="cuda:0").manual_seed(E * 10007 + T)

    def normal(*shape, std=1.0):
        return torch.randn(*shape, generator=gen, device="cuda:0").mul_(std).bfloat16()

    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=E, top_k=K, n_part=P, max_tokens=2049, dtype="bf16", expert_lo=lo, expert_hi=hi)
    layer.partition_weights(normal(hi - lo, D, F, std=0.05), normal(hi - lo, D, F, std=0.05), normal(hi - lo, F, D, std=0.05))
    layer.pack_router(normal(D, E, std=0.1))
    x = normal(T, D)
    # thresholds that differ by expert and rise with the partition, around 1 / K
    tau = (torch.rand(E, P, generator=gen, device="cuda:0").cumsum(1) * (1.2 / (K * P))).contiguous()
    y, logits = layer.forward_routed(x, tau, want_logits=True)
    one = layer.plan(T)
    ref = layer.forward(x, layer.router_logits(x), tau)
    two = layer.plan(T)
    assert torch.equal(logits, layer.router_logits(x))
    for name in ("topk_idx", "topk_w", "keep_bits", "expert_nrows"):
        assert torch.equal(one[name], two[name]), name
    assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
    assert torch.equal(layer.forward_routed(x, tau).view(torch.int16), ref.view(torch.int16))
    layer.close()
