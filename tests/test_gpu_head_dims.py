"""Head dimensions on both sides of the middle of their last 32 channels, which have kernels of their own, against Algorithm 1 in
64 bits (signs, abs-means, 8-bit V per channel, 8-bit P relative to the running maximum of blocks of 128 keys)."""
import math

import pytest
import torch

from paper_2603_09582_amd import binding as ba

pytestmark = pytest.mark.gpu


def algorithm1(q, k, v, bias, scale):
    q, k, v = q.double(), k.double(), v.double()
    N = q.shape[2]
    alpha = scale * q.abs().mean(dim=(2, 3)) * k.abs().mean(dim=(2, 3))
    one = torch.ones((), dtype=torch.float64, device=q.device)
    S = torch.matmul(torch.where(q >= 0, one, -one), torch.where(k >= 0, one, -one).transpose(2, 3).contiguous()) * alpha[:, :, None, None]
    if bias is not None:
        S = S + bias.double()
    delta = v.abs().amax(dim=2, keepdim=True) / 127
    codes = torch.round(v / delta)
    m = torch.full((*S.shape[:3], 1), -math.inf, dtype=torch.float64, device=q.device)
    l, o = torch.zeros_like(m), torch.zeros_like(q)
    for j in range(0, N, 128):
        s = S[..., j:j + 128]
        mn = torch.maximum(m, s.amax(dim=3, keepdim=True))
        p, r = torch.exp(s - mn), torch.exp(m - mn)
        l = l * r + p.sum(dim=3, keepdim=True)
        o = o * r + torch.matmul(torch.round(255 * p), codes[:, :, j:j + 128].contiguous())
        m = mn
    return o / (255 * l) * delta


@pytest.mark.parametrize("d", [40, 48, 56, 72, 80, 88])
@pytest.mark.parametrize("B,H,N,bias", [(1, 2, 50, "bf16"), (1, 2, 200, "fp32"), (150, 2, 200, "bf16"), (150, 2, 250, "none"), (1, 2, 300, "none"),
                                        (1, 2, 392, "bf16"), (1, 3, 301, "bf16"), (1, 2, 300, "fp32"), (2, 2, 1100, "bf16"), (1, 2, 512, "table")])
def test_head_dimensions(d, B, H, N, bias):
    g = torch.Generator(device="cuda").manual_seed(d * 1000 + N + B)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    scale = d ** -0.5
    if bias == "table":
        Gy, Gx = N // 32, 32
        table = torch.randn(H, 2 * Gy - 1, 2 * Gx - 1, generator=g, device="cuda") * 0.3
        i = torch.arange(N, device="cuda")
        b = table[:, (i // Gx)[:, None] - (i // Gx)[None, :] + Gy - 1, (i % Gx)[:, None] - (i % Gx)[None, :] + Gx - 1]
        got = ba.attention_relpos(q, k, v, table, scale)
    else:
        b = None if bias == "none" else (torch.randn(H, N, N, generator=g, device="cuda") * 0.3).to(torch.bfloat16 if bias == "bf16" else torch.float32)
        got = ba.attention(q, k, v, b, scale)
    ref = algorithm1(q, k, v, b, scale)
    # rows of 50 and more keys: the stated tolerance of the outputs
    assert ((got.double() - ref).abs() <= 1e-2 + 2e-2 * ref.abs()).all()


# (a bias of more than 256 MB is copied past the caches where its rows start on 128-byte lines: here by its pitch)
@pytest.mark.parametrize("d", [24, 40, 48, 64])
def test_two_batch_entries_share_a_streamed_bias(d):
    B, H, N, pitch = 2, 1, 1000, 134_272
    g = torch.Generator(device="cuda").manual_seed(d)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    b = (torch.randn(H, N, N, generator=g, device="cuda") * 0.3).to(torch.bfloat16)
    store = torch.full((N * pitch,), float("nan"), dtype=torch.bfloat16, device="cuda")
    far = store.as_strided((H, N, N), (N * pitch, pitch, 1)).copy_(b)
    scale = d ** -0.5
    got, near, alone = ba.attention(q, k, v, far, scale), ba.attention(q, k, v, b, scale), ba.attention(q[:1], k[:1], v[:1], b, scale)
    # (an even number of key blocks: the accumulator's offset is removed before the same ones in every form)
    assert torch.equal(got, near) and torch.equal(got[:1], alone)
    ref = algorithm1(q, k, v, b, scale)
    assert ((got.double() - ref).abs() <= 1e-2 + 2e-2 * ref.abs()).all()
