"""The single launch where the second key block ends early (128 < N <= 224): 32-key tiles and waves without keys and rows are left
out there.  Against the launches over a workspace and the 8-wave form, bit for bit."""
import pytest
import torch

from paper_2603_09582_amd import binding as ba

pytestmark = pytest.mark.gpu


# both sides of every tile's edge; two heads take 8 waves each, 260 four (d <= 96); 520 heads, d = 64, three workgroups per compute unit with
# the last heads split by row blocks, 768 whole ones
@pytest.mark.parametrize("N", [100, 129, 160, 161, 192, 193, 224, 225, 256])
@pytest.mark.parametrize("heads,d", [(2, 32), (2, 64), (2, 72), (2, 128), (260, 32), (260, 64), (260, 96), (520, 64), (768, 64)])
@pytest.mark.parametrize("bias", ["none", "bf16", "fp32", "masked"])
def test_single_launch_with_an_early_end(N, heads, d, bias):
    g = torch.Generator(device="cuda").manual_seed(N * 7 + heads + d)
    q, k, v = (torch.randn(heads // 2, 2, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    b = None
    if bias != "none":
        b = torch.randn(2, N, N, generator=g, device="cuda").to(torch.float32 if bias == "fp32" else torch.bfloat16)
    if bias == "masked":  # rows that see the second block alone, and rows that do not see it
        edge = 128 if N > 128 else 64
        b[:, : N // 2, :edge] = float("-inf")
        b[:, N // 2:, edge:] = float("-inf")
    scale = d ** -0.5
    mu = [torch.empty(heads // 2, 2, device="cuda") for _ in range(2)]
    got = ba.forward_fused(q, k, v, b, scale, mu_q=mu[0], mu_k=mu[1])
    wide = ba.forward_fused(q, k, v, b, scale, flags=ba.FLAG_WIDE8 | ba.FLAG_NO_MU)
    some = ba.forward_fused(q, k, v, b, scale, flags=ba.FLAG_NO_MU)
    qb, kb, mq, mk = ba.pack_qk(q, k)
    ref = ba.forward(qb, kb, mu[0], mu[1], v, b, scale)  # the same abs-means
    assert torch.isfinite(got.float()).all()
    # a tile that is left out would have had weights of 0 and codes of -128: the same bits
    assert torch.equal(got, ref)
    assert torch.equal(some, wide)
    for m, n in ((mu[0], mq), (mu[1], mk)):  # fp32 sums of N d terms in two orders
        assert torch.allclose(m, n, rtol=1e-5, atol=0)
