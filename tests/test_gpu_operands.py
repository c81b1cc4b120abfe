"""The operand preparation at the values where its arithmetic could go wrong: every pair of bf16
significands in the V quantiser (exact ties included), scales at the ends of the range, and the signs of
NaN, infinities and zeros on the paths that make the FP4 operands without sign words."""
import numpy as np
import pytest
import torch

from oracle import binattn_oracle as orc
from paper_2603_09582_amd import binding as ba
from tests.helpers import bf16_bits

pytestmark = pytest.mark.gpu


# absmax of channel c: significand 128 + c; the last two groups take the division inside the quantiser
@pytest.mark.parametrize("exponent", [0, -1, 30, -101, 101, -126, -130])
def test_v_codes_for_every_pair_of_significands(exponent):
    A = torch.arange(128, 256, dtype=torch.float64)
    V = torch.arange(128, 256, dtype=torch.float64)
    e = torch.arange(0, 10, dtype=torch.float64)
    v = (V[None, :] * 2.0 ** -e[:, None]).reshape(-1, 1).repeat(1, 128)  # [10 * 128, 128]
    v[v > A[None, :]] = 0.0
    v = torch.cat([A[None, :], v, -v]) * 2.0 ** (exponent - 7)
    v = v.to(torch.float32).to(torch.bfloat16)[None, None]
    vq, delta = ba.quant_v_debug(v.cuda())
    ref_q, ref_d = orc.quant_v(bf16_bits(v[0, 0]))
    assert np.array_equal(delta[0, 0].cpu().numpy(), ref_d)
    assert np.array_equal(vq[0, 0].cpu().numpy(), ref_q)


@pytest.mark.parametrize("N,d", [(100, 64), (250, 72), (300, 40), (333, 128)])
def test_signs_of_special_values_without_sign_words(N, d):
    g = torch.Generator().manual_seed(N)
    q, k, v = (torch.randn(1, 2, N, d, generator=g).to(torch.bfloat16) for _ in range(3))
    special = torch.tensor([float("nan"), -0.0, 0.0, float("inf"), -float("inf")], dtype=torch.bfloat16)
    neg_nan = torch.tensor([-64], dtype=torch.int16).view(torch.bfloat16)  # 0xFFC0
    special = torch.cat([special, neg_nan])
    for t in (q, k):
        at = torch.randint(0, N * d, (60,), generator=g)
        t[0, 0].view(-1)[at] = special.repeat(10)  # head 1 stays ordinary
    q, k, v = q.cuda(), k.cuda(), v.cuda()
    qb, kb, _, _ = ba.pack_qk(q, k)
    want = ba.forward(qb, kb, None, None, v, None, d ** -0.5, flags=ba.FLAG_NO_MU)
    got = ba.attention(q, k, v, None, d ** -0.5, flags=ba.FLAG_NO_MU)
    # the same signs, the same scale: the same logits, so the same codes on both paths
    assert torch.equal(want, got)


@pytest.mark.parametrize("N,d", [(1, 64), (63, 64), (129, 32), (197, 64), (256, 72), (200, 96)])
def test_both_single_launch_forms_give_the_same_bits(N, d):
    """The 4-wave form adds the magnitudes in the 8-wave form's order: abs-means and outputs agree exactly."""
    B, H = 2, 130
    g = torch.Generator(device="cuda")
    g.manual_seed(N + d)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    bias = torch.randn(H, N, N, generator=g, device="cuda").to(torch.bfloat16)
    res = []
    for flags in (0, ba.FLAG_WIDE8):
        mq, mk = torch.zeros(B, H, device="cuda"), torch.zeros(B, H, device="cuda")
        res.append((ba.forward_fused(q, k, v, bias, d ** -0.5, mu_q=mq, mu_k=mk, flags=flags), mq, mk))
    torch.cuda.synchronize()
    for a, b in zip(*res):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,H,N,d,flags", [(1, 2, 300, 72, 0), (2, 2, 577, 40, 0), (1, 1, 391, 104, 0), (1, 2, 257, 8, 0),
                                           (1, 2, 300, 72, ba.FLAG_LUT), (2, 1, 1030, 48, 0)])
@pytest.mark.parametrize("with_bias", [False, True])
def test_what_the_workspace_held_before_does_not_matter(B, H, N, d, flags, with_bias):
    """Places of the operand images that no key or channel fills keep the workspace's old bytes."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + d)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    bias = torch.randn(H, N, N, generator=g, device="cuda").to(torch.bfloat16) if with_bias else None
    ws = ba.alloc_workspace(B, H, N, d)
    res = []
    for fill in (0x00, 0xFF, 0x7F, 0x80):
        ws.fill_(fill)
        one = ba.attention(q, k, v, bias, d ** -0.5, workspace=ws, flags=flags)
        ws.fill_(fill)
        qb, kb, mq, mk = ba.pack_qk(q, k)
        res.append((one, ba.forward(qb, kb, mq, mk, v, bias, d ** -0.5, workspace=ws, flags=flags)))
    torch.cuda.synchronize()
    for one, packed in res[1:]:
        assert torch.equal(one, res[0][0]) and torch.equal(packed, res[0][1])
        assert torch.isfinite(one).all()
