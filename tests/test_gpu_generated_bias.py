"""The biases generated from tables at the edges of the token grid: the staged rows and windows reach past the grid's last row and
past the tables' ends, and nothing of what lies there may show."""
import pytest
import torch

from paper_2603_09582_amd import binding as ba

pytestmark = pytest.mark.gpu


def inside_nan(t, pad=1100):
    """The same values in the middle of a buffer of NaN."""
    buf = torch.full((t.numel() + 2 * pad,), float("nan"), dtype=t.dtype, device=t.device)
    v = buf[pad:pad + t.numel()].view(t.shape)
    v.copy_(t)
    return v


# grids whose last key block and last query rows end inside the grid, on its edge, and before the first whole block
@pytest.mark.parametrize("Gy,Gx", [(17, 16), (24, 16), (9, 32), (40, 32), (5, 64), (7, 64), (3, 128), (3, 256), (5, 256)])
@pytest.mark.parametrize("d", [32, 64, 72, 128])
def test_generated_bias_equals_the_dense_one_and_ignores_what_surrounds_the_tables(Gy, Gx, d):
    B, H, N = 1, 2, Gy * Gx
    g = torch.Generator().manual_seed(Gy * 1000 + Gx + d)
    q, k, v = (torch.randn(B, H, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    table = torch.randn(H, 2 * Gy - 1, 2 * Gx - 1, generator=g).cuda()
    by, bx = torch.randn(H, 2 * Gy - 1, generator=g).cuda(), torch.randn(H, 2 * Gx - 1, generator=g).cuda()
    i = torch.arange(N, device="cuda")
    dy = (i // Gx)[:, None] - (i // Gx)[None, :] + Gy - 1
    dx = (i % Gx)[:, None] - (i % Gx)[None, :] + Gx - 1
    scale = d ** -0.5
    qb, kb, mq, mk = ba.pack_qk(q, k)
    dense = ba.forward(qb, kb, mq, mk, v, table[:, dy, dx].contiguous(), scale)
    got = ba.forward_relpos(qb, kb, mq, mk, v, inside_nan(table), scale)
    # (both add the fp32 entry divided by the multiplier to the exact logit: the same bits)
    assert torch.equal(got, dense)
    dense = ba.forward(qb, kb, mq, mk, v, (by[:, dy] + bx[:, dx]).contiguous(), scale)
    got = ba.forward_axial(qb, kb, mq, mk, v, inside_nan(by), inside_nan(bx), scale)
    # the two terms are divided, rounded and added apart: a code of P falls to the other side of a half-integer here and there, and one
    # code moves an output by at most max |v| / 255 (under 5 / 255); bf16 rounds to 2^-8 on either side
    diff = (got.float() - dense.float()).abs()
    assert torch.isfinite(got.float()).all() and (diff <= 2e-2 + 2e-2 * dense.float().abs()).all()
