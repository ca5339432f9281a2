"""GPU: experts of so many neurons (2^22) that two row tiles of the intermediate activation are 4 GiB, beyond what one buffer descriptor of
32-bit offsets reaches: an expert's short last row tile then has items of its own.  Routed and shared experts, against 64-bit sums.

Bar: a sum is up to 8 partial outputs, each rounded to 2^-11 of itself, of like size and either sign: together at most 2^-11 of the value plus
2^-11 of about three times the RMS; the rounding of the activations averages out over 2^22 terms.  2^-10 of the value + 2e-3 of the RMS.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["routed", "shared"])
def test_two_row_tiles_of_4_gib(where):
    import torch
    from paper_2508_18376_amd import DualSparseLayer
    D, T, big, small = 32, 300, 1 << 22, 128
    F, F_sh = (big, small) if where == "routed" else (small, big)
    gen = torch.Generator(device="cuda:0").manual_seed(2)

    def normal(*shape, std):
        return torch.randn(*shape, generator=gen, device="cuda:0").mul_(std).bfloat16()

    w, sh = ([normal(1, D, f, std=0.1), normal(1, D, f, std=0.1), normal(1, f, D, std=0.02)] for f in (F, F_sh))
    x = normal(T, D, std=1.0)
    layer = DualSparseLayer(d_model=D, d_ff=F, n_experts=1, top_k=1, n_part=1, max_tokens=T, dtype="bf16", n_shared=1, d_ff_shared=F_sh, y_fp32=True)
    assert layer.uses_mfma
    layer.partition_weights(*w, sh_w1=sh[0], sh_w3=sh[1], sh_w2=sh[2])
    y = layer.forward(x, torch.zeros(T, 1, device="cuda:0"), torch.zeros(1, 1, device="cuda:0")).double()
    layer.close()
    ref = torch.zeros(T, D, dtype=torch.float64, device="cuda:0")
    xd = x.double()
    for w1, w3, w2 in (w, sh):
        for n in range(0, w1.shape[2], 1 << 17):
            a = xd @ w1[0, :, n:n + (1 << 17)].double()
            ref += (a * torch.sigmoid(a) * (xd @ w3[0, :, n:n + (1 << 17)].double())) @ w2[0, n:n + (1 << 17)].double()
    assert ((y - ref).abs() <= 2.0 ** -10 * ref.abs() + 2e-3 * ref.square().mean().sqrt()).all()
