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


@pytest.mark.parametrize("N,d", [(100, 64), (128, 72), (300, 40)])
def test_an_infinity_in_v_gives_code_zero_and_stays_in_its_channel(N, d):
    """Outside what the calls promise (V is finite), but no number may come out of an infinite scale."""
    g = torch.Generator().manual_seed(N)
    q, k, v = (torch.randn(1, 2, N, d, generator=g).to(torch.bfloat16) for _ in range(3))
    clean = v.clone()
    v[0, 0, 5, 3], v[0, 0, 7, d - 1], v[0, 0, 9, d - 1] = float("inf"), float("-inf"), float("inf")
    hit = [3, d - 1]
    vq, delta = ba.quant_v_debug(v.cuda())
    assert (vq[0, 0][:, hit] == 0).all() and torch.isinf(delta[0, 0, hit]).all()
    q, k = q.cuda(), k.cuda()
    qb, kb, mq, mk = ba.pack_qk(q, k)

    def outs(v):
        return [ba.attention(q, k, v.cuda(), None, d ** -0.5), ba.forward(qb, kb, mq, mk, v.cuda(), None, d ** -0.5)]

    for got, want in zip(outs(v), outs(clean)):
        keep = torch.ones(2, d, dtype=torch.bool)
        keep[0, hit] = False
        assert torch.equal(got.cpu().transpose(2, 3)[0][keep], want.cpu().transpose(2, 3)[0][keep])
        if N <= 128:  # one key block: the codes' zero times the scale
            assert torch.isnan(got[0, 0][:, hit]).all()


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


def ordered_abs_mean(x, waves, keys):
    """Mean of |x| (fp32 [N, d]) in the order a workgroup of the single-launch forms adds it: every lane the
    chunks of 8 channels it owns, in turn; a tree over the 64 lanes; the waves one after the other."""
    N, d = x.shape
    DK, C16 = -(-d // 32), d // 8
    lane, wave = np.arange(64)[None, :], np.arange(waves)[:, None]
    s = np.zeros((waves, 64), np.float32)
    ax = np.abs(np.concatenate([x, np.zeros((1, d), np.float32)]))  # row N stands for "no row"

    def add(row, c0, live):
        nonlocal s
        row, c0 = np.where(live, row, N), np.where(live, c0, 0)
        for i in range(0, 8, 2):
            s = np.where(live, s + (ax[row, c0 + i] + ax[row, c0 + i + 1]), s)

    if keys:
        for kk in range(-(-(256 * 4 * DK) // (64 * waves))):
            i = 64 * waves * kk + 64 * wave + lane
            ic, c8 = i // C16, i % C16
            m, t = ic % 32, ic % 128 // 32
            key = ic // 128 * 128 + 64 * (m // 4 % 2) + 16 * t + 4 * (m // 8) + m % 4
            add(key, 8 * c8, (ic < 256) & (key < N))
    else:
        for row0 in range(0, 256, 32 * waves):
            row = row0 + 32 * wave + lane % 32
            for sI in range((DK + 1) // 2):
                for j in range(4):
                    c0 = 64 * sI + 32 * (lane // 32) + 8 * j + 0 * wave
                    add(row, c0, (row < N) & (c0 < d))
    for off in (32, 16, 8, 4, 2, 1):
        s[:, :64 - off] = s[:, :64 - off] + s[:, off:]
    total = np.float32(0.0)
    for w in range(waves):
        total = total + s[w, 0]
    return total * (np.float32(1.0) / (np.float32(N) * np.float32(d)))


# (kind of bias decides between the forms above 256 heads and 64 channels)
@pytest.mark.parametrize("H,flags,kind", [(6, 0, "rows16"), (260, 0, "rows16"), (260, ba.FLAG_WIDE8, "rows16"), (260, 0, "odd"),
                                          (260, 0, "none"), (260, 0, "table"), (260, 0, "f32")])
@pytest.mark.parametrize("N,d", [(1, 64), (96, 64), (208, 64), (256, 32), (240, 72), (256, 96), (128, 80)])
def test_abs_means_of_the_single_launch_are_added_in_a_fixed_order(N, d, H, flags, kind):
    """The logit multiplier is made of these two numbers: their last bits decide single 8-bit codes of P.  So
    the order of the sums is part of the result, whichever kernel a call is given to."""
    if kind == "table" and N % 16:
        pytest.skip("token grids have rows of 16")
    g = torch.Generator(device="cuda")
    g.manual_seed(N + d)
    q, k, v = (torch.randn(1, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    mq, mk = torch.zeros(1, H, device="cuda"), torch.zeros(1, H, device="cuda")
    if kind == "table":
        table = torch.randn(H, 2 * (N // 16) - 1, 31, generator=g, device="cuda")
        ba.forward_fused_relpos(q, k, v, table, d ** -0.5, mu_q=mq, mu_k=mk, flags=flags)
    else:
        pitch = N + (1 if kind == "odd" else -N % 8)
        dtype = torch.float32 if kind == "f32" else torch.bfloat16
        bias = None if kind == "none" else torch.randn(H, N, pitch, generator=g, device="cuda").to(dtype)[:, :, :N]
        ba.forward_fused(q, k, v, bias, d ** -0.5, mu_q=mq, mu_k=mk, flags=flags)
    torch.cuda.synchronize()
    eight = H <= 256 or flags or (d > 64 and kind in ("odd", "table"))
    for h in range(0, H, 3 if H < 256 else 37):
        for t, mu, keys in ((q, mq, False), (k, mk, True)):
            want = ordered_abs_mean(t[0, h].float().cpu().numpy(), 8 if eight else 4, keys)
            assert mu[0, h].item() == want, (h, "k" if keys else "q")


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
