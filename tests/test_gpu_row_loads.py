"""Loads and slabs of the operand preparation: rows that lie anywhere (single launch), and the one-pass
quantiser of V at the edges of its blocks per wave, chunks per slab and blocks per workgroup."""
import numpy as np
import pytest
import torch

from oracle import binattn_oracle as orc
from paper_2603_09582_amd import binding as ba
from tests.helpers import bf16_bits
from tests.test_gpu_parity import check_close, gpu_out_f64, relpos_dense, say

pytestmark = pytest.mark.gpu


def at_the_end(x, pitch, other=float("nan")):
    """The same [1, H, N, d] values, heads side by side in rows `pitch` elements apart, as the very end of a buffer
    that holds `other` elsewhere (a row of it would follow the last one)."""
    _, H, N, d = x.shape
    n = (N - 1) * pitch + H * d
    store = torch.full((8 + n,), other, dtype=x.dtype, device="cuda")
    view = store[8:].as_strided((1, H, N, d), (n, d, pitch, 1))
    view.copy_(x)
    return view


# (pitches from 2^22 elements on take 64-bit addresses; more than 256 heads the 4-wave form)
@pytest.mark.parametrize("H,N,d", [(2, 1, 64), (2, 5, 72), (3, 9, 128), (260, 3, 40), (260, 4, 64), (258, 130, 72), (2, 197, 104)])
def test_single_launch_rows_anywhere(H, N, d):
    g = torch.Generator().manual_seed(H + N + d)
    q, k, v = (torch.randn(1, H, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    want = ba.attention(q, k, v, None, d ** -0.5)
    for pitch in (H * d, H * d + 8) + (((1 << 22) - 8, 1 << 22) if N <= 9 else ()):
        say(f"single launch rows H={H} N={N} d={d} pitch={pitch}")
        got = ba.attention(*(at_the_end(t, pitch) for t in (q, k, v)), None, d ** -0.5)
        torch.cuda.synchronize()
        assert torch.equal(got, want), pitch


# (up to d = 24 one pass has threads for more than the 64 token quads; 16 and 24 only in the 8-wave form)
@pytest.mark.parametrize("H,d", [(3, 8), (3, 16), (3, 24), (260, 8), (260, 16), (260, 24)])
def test_single_launch_far_rows_of_small_heads(H, d):
    N = 5
    g = torch.Generator().manual_seed(H + d)
    q, k, v = (torch.randn(1, H, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    want = ba.attention(q, k, v, None, d ** -0.5)
    for pitch in (1 << 20, (1 << 20) + (1 << 18), 5 << 19, (3 << 20) + 8, (1 << 22) - 8, 1 << 22):
        say(f"single launch far rows H={H} d={d} pitch={pitch}")
        got = ba.attention(at_the_end(q, pitch), at_the_end(k, pitch), at_the_end(v, pitch, 1e30), None, d ** -0.5)
        torch.cuda.synchronize()
        assert torch.equal(got, want), pitch


# (a wave per key block up to 4 and 8 blocks, then 2 and 4 of them per wave; above 32 blocks two passes)
@pytest.mark.parametrize("N,d", [(257, 8), (300, 72), (512, 40), (513, 104), (1024, 24), (1025, 72), (2048, 32), (2049, 80),
                                 (4096, 16), (4097, 72), (3000, 128)])
def test_one_pass_quantiser_and_abs_means(N, d):
    say(f"one pass over V N={N} d={d}")
    B, H = 1, 3
    g = torch.Generator().manual_seed(N + d)
    q, k, v = (torch.randn(B, H, N, d, generator=g).to(torch.bfloat16) for _ in range(3))
    v[0, 0, N - 1] *= 9.0  # the maximum of every channel in the last row
    v[0, 1, :, d - 1] = 0.0
    dq, dk, dv = q.cuda(), k.cuda(), v.cuda()
    vq, delta = ba.quant_v_debug(dv)
    mq, mk = (torch.empty(B, H, dtype=torch.float32, device="cuda") for _ in range(2))
    got = ba.attention(dq, dk, dv, None, d ** -0.5, mu_q=mq, mu_k=mk)
    plain = ba.attention(dq, dk, dv, None, d ** -0.5, flags=ba.FLAG_NO_MU)
    qb, kb, _, _ = ba.pack_qk(dq, dk)
    torch.cuda.synchronize()
    for h in range(H):
        codes, scales = orc.quant_v(bf16_bits(v[0, h]))
        assert np.array_equal(vq[0, h].cpu().numpy(), codes) and np.array_equal(delta[0, h].cpu().numpy(), scales)
        for mu, x in ((mq, q), (mk, k)):
            assert float(mu[0, h]) == pytest.approx(orc.abs_mean(bf16_bits(x[0, h])), rel=2e-6)
    # the same signs, codes and scales through the sign words: the same bits
    assert torch.equal(ba.forward(qb, kb, None, None, dv, None, d ** -0.5, flags=ba.FLAG_NO_MU), plain)
    assert torch.equal(ba.forward(qb, kb, mq, mk, dv, None, d ** -0.5), got)


@pytest.mark.parametrize("N,d", [(300, 64), (1500, 72)])
def test_a_nan_in_v_hides_no_other_value(N, d):
    """Outside what the calls promise (V is finite): the scale is the largest magnitude of the channel's numbers."""
    g = torch.Generator().manual_seed(N)
    v = torch.randn(1, 2, N, d, generator=g).to(torch.bfloat16)
    _, want = ba.quant_v_debug(v.cuda())
    bad = v.clone()
    at = torch.randint(0, N, (d,), generator=g)
    keep = v[0, 0].abs().float().argmax(dim=0)  # never the maximum itself
    at = torch.where(at == keep, (at + 1) % N, at)
    bad[0, 0, at, torch.arange(d)] = float("nan")
    _, got = ba.quant_v_debug(bad.cuda())
    assert torch.equal(got, want)


# (heads left for a last round: one, a few that do not fill the eight chiplets, the most that are split, one more; where three workgroups
# share a compute unit also above 768 heads, and as many as fill a round, with one chiplet's share not full)
@pytest.mark.parametrize("B,H,N,d,kind", [(513, 1, 197, 64, "bf16"), (65, 8, 129, 40, "bf16"), (160, 4, 256, 72, "bf16"), (641, 1, 130, 64, "none"),
                                          (75, 7, 200, 96, "fp32"), (215, 3, 256, 24, "none"), (130, 4, 256, 72, "table"), (1025, 1, 256, 64, "none"),
                                          (769, 1, 197, 64, "bf16"), (835, 1, 197, 64, "bf16"), (833, 1, 200, 32, "bf16"), (700, 1, 225, 32, "none"),
                                          (1401, 1, 197, 64, "none"), (1401, 1, 197, 64, "bf16"), (173, 8, 224, 48, "bf16"),
                                          (896, 1, 160, 40, "bf16"), (897, 1, 160, 40, "bf16"), (1024, 1, 224, 64, "bf16"), (150, 8, 160, 56, "bf16")])
def test_heads_of_the_last_round_by_row_blocks(B, H, N, d, kind):
    """The single launch's 4-wave form takes those heads with a workgroup per row block: the bits of a call that takes
    the same heads whole."""
    say(f"last round by row blocks B={B} H={H} N={N} d={d} {kind}")
    g = torch.Generator().manual_seed(B + N + d)
    q, k, v = (torch.randn(B, H, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    table = (torch.randn(H, 31, 31, generator=g) * 0.5).cuda()
    bias = None if kind == "none" else torch.randn(H, N, N, generator=g).to(torch.float32 if kind == "fp32" else torch.bfloat16).cuda()

    def call(b0):
        mu = [torch.full((B - b0, H), float("nan"), device="cuda") for _ in range(2)]
        a = (q[b0:], k[b0:], v[b0:])
        out = (ba.attention_relpos(*a, table, d ** -0.5, mu_q=mu[0], mu_k=mu[1]) if kind == "table" else
               ba.attention(*a, bias, d ** -0.5, mu_q=mu[0], mu_k=mu[1]))
        torch.cuda.synchronize()
        return out, *mu

    b0 = B - 1 - 300 // H  # 301 heads or more, at most 512: no last round of their own
    assert 256 < (B - b0) * H <= 512
    for whole, some in zip(call(0), call(b0)):
        assert torch.equal(whole[b0:], some)


@pytest.mark.parametrize("kind", ["none", "bf16", "odd", "f32", "table"])
@pytest.mark.parametrize("N", [252, 253, 256])
def test_last_token_quad_of_the_widest_rows(N, kind):
    """d = 96 in the 4-wave form: 21 token quads per pass, so that the 64th is a pass of its own.  The last rows hold every
    channel's maximum."""
    if kind == "table" and N % 16:
        pytest.skip("token grids have rows of 16")
    say(f"last quad of d = 96, N={N}, {kind}")
    H, d = 260, 96
    g = torch.Generator().manual_seed(N)
    q, k, v = (torch.randn(1, H, N, d, generator=g).to(torch.bfloat16) for _ in range(3))
    v[:, :, N - 4:] = (torch.where(torch.rand(1, H, 4, d, generator=g) < 0.5, -1.25, 1.25) * v.abs().float().amax(dim=2, keepdim=True)).to(torch.bfloat16)
    table = (torch.randn(H, 31, 31, generator=g) * 0.3).cuda()
    bias, dense = None, None
    if kind == "table":
        dense = relpos_dense(table.cpu(), 16, 16)
    elif kind != "none":
        dense = (torch.randn(H, N, N, generator=g) * 0.3).to(torch.float32 if kind == "f32" else torch.bfloat16)
        store = torch.zeros(H, N, N + (1 if kind == "odd" else -N % 8), dtype=dense.dtype, device="cuda")
        bias = store[:, :, :N].copy_(dense)
    a = (q.cuda(), k.cuda(), v.cuda())

    def call(flags):
        out = (ba.forward_fused_relpos(*a, table, d ** -0.5, flags=flags) if kind == "table" else
               ba.forward_fused(*a, bias, d ** -0.5, flags=flags))
        torch.cuda.synchronize()
        return gpu_out_f64(out)[0]

    got, wide = call(0), call(ba.FLAG_WIDE8)
    # (V is at most 1.25 times what the forms' 2e-3 stands for elsewhere)
    assert np.abs(got - wide).max() <= 2.5e-3
    for h in range(0, H, 37):
        qq, kk, vv = (bf16_bits(t[0, h]) for t in (q, k, v))
        codes, scales = orc.quant_v(vv)
        b = None if dense is None else dense[h].numpy() if dense.dtype == torch.float32 else bf16_bits(dense[h])
        want = orc.attention_rows(qq, kk, vv, b, d ** -0.5, orc.abs_mean(qq), orc.abs_mean(kk), codes, scales, want=("O2",))
        check_close(got[h], want["O2"], f"head {h}")


# (2400 items of a head and row block: more than three in turn for every workgroup of each grid: 512, 768 and 256 pairs)
@pytest.mark.parametrize("d,kind", [(64, "none"), (64, "bf16"), (64, "odd"), (72, "bf16"), (72, "f32"), (96, "none"), (128, "none"), (128, "bf16"), (128, "f32")])
def test_abs_means_of_the_head_after_the_next(d, kind):
    """Heads whose abs-means differ by powers of two, several of them in turn in a workgroup: each with its own logit multiplier."""
    B, H, N = 100, 8, 300
    say(f"abs-means by powers of two d={d} {kind}")
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda") for _ in range(3))
    for t in (q, k):
        t *= torch.exp2(torch.randint(-3, 4, (B, H, 1, 1), generator=g, device="cuda").float())
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    bias = None
    if kind != "none":
        dtype = torch.float32 if kind == "f32" else torch.bfloat16
        bias = torch.randn(H, N, N + (1 if kind == "odd" else -N % 8), generator=g, device="cuda").to(dtype)[:, :, :N]
    mq, mk = (torch.full((B, H), float("nan"), device="cuda") for _ in range(2))
    got = ba.attention(q, k, v, bias, d ** -0.5, mu_q=mq, mu_k=mk)
    qb, kb, _, _ = ba.pack_qk(q, k)
    want = ba.forward(qb, kb, mq, mk, v, bias, d ** -0.5)  # the same abs-means, one number per head
    torch.cuda.synchronize()
    for mu, x in ((mq, q), (mk, k)):  # fp32 sums of 300 d terms in two orders
        assert torch.allclose(mu.double(), x.double().abs().mean(dim=(2, 3)), rtol=1e-5, atol=0)
    assert torch.equal(got, want)


# (heads of a last round by row blocks; whole heads in the 4- and the 8-wave form; more than two key blocks)
@pytest.mark.parametrize("B,H,N,d", [(520, 1, 200, 64), (80, 8, 256, 72), (40, 7, 130, 32), (2, 3, 200, 64), (2, 3, 300, 72), (1, 2, 4200, 64)])
@pytest.mark.parametrize("which", ["q", "k", "v"])
def test_output_on_the_storage_of_an_input(B, H, N, d, which):
    say(f"output on the storage of {which} B={B} H={H} N={N} d={d}")
    g = torch.Generator().manual_seed(N)
    x = {n: torch.randn(B, N, H, d, generator=g).to(torch.bfloat16).cuda().transpose(1, 2) for n in "qkv"}
    bias = torch.randn(H, N, N, generator=g).to(torch.bfloat16).cuda() if N < 1000 else None
    want = ba.attention(x["q"], x["k"], x["v"], bias, d ** -0.5)
    got = ba.attention(x["q"], x["k"], x["v"], bias, d ** -0.5, out=x[which])
    torch.cuda.synchronize()
    assert got.data_ptr() == x[which].data_ptr() and torch.equal(got, want)


# (more than 16 key blocks: two passes up to 16 slabs of 32 channels in the one call - up to 32 in the preparation for d <= 64 and
# d >= 96 - and one pass above; one pass with any number of them from d = 104, or from 72 to 88 in the preparation)
@pytest.mark.parametrize("H,N,d", [(16, 2049, 32), (17, 2049, 32), (33, 2100, 24), (5, 2049, 96), (6, 2500, 72), (16, 2049, 64), (17, 2177, 64), (1, 2049, 104), (11, 2049, 96), (9, 2049, 128)])
def test_one_or_two_passes_over_long_v(H, N, d):
    """The same codes, scales and abs-means on either side of the rule (half the heads, all of them, and alone), and the outputs
    of the one call those of the preparation and the attention stage."""
    say(f"one or two passes H={H} N={N} d={d}")
    g = torch.Generator().manual_seed(N + d)
    q, k, v = (torch.randn(1, H, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    res = {}
    for n in {H, max(1, H // 2), 1}:
        mu = [torch.full((1, n), float("nan"), device="cuda") for _ in range(2)]
        a = [t[:, :n] for t in (q, k, v)]
        qb, kb, _, _ = ba.pack_qk(a[0], a[1])
        one = ba.attention(*a, None, d ** -0.5, mu_q=mu[0], mu_k=mu[1])
        res[n] = (one, *mu, *ba.quant_v_debug(a[2]), ba.forward(qb, kb, *mu, a[2], None, d ** -0.5))
        torch.cuda.synchronize()
        assert torch.equal(res[n][0], res[n][5])
    for n, r in res.items():
        for x, y in zip(res[H][1:5], r[1:5]):  # (an output's last bits depend on where in the grid its head lies)
            assert torch.equal(x[:, :n], y)
    codes, scales = orc.quant_v(bf16_bits(v[0, 0]))
    assert np.array_equal(res[H][3][0, 0].cpu().numpy(), codes) and np.array_equal(res[H][4][0, 0].cpu().numpy(), scales)
    assert float(res[H][1][0, 0]) == pytest.approx(orc.abs_mean(bf16_bits(q[0, 0])), rel=2e-6)


def test_more_heads_than_one_launch_of_the_preparation_takes():
    """2.1 million heads of N = 513, d = 8: the runtime refuses 2^32 threads or more in a launch.  All heads on the same Q, K, V."""
    H, N, d = 2_097_150 + 60, 513, 8
    say(f"preparation in two launches, {H} heads")
    if torch.cuda.mem_get_info()[0] < ba.workspace_bytes(1, H, N, d) + 3 * H * N * d * 2:
        pytest.skip("not enough free memory")
    g = torch.Generator().manual_seed(2)
    x = [torch.randn(1, 1, N, d, generator=g).to(torch.bfloat16).cuda() for _ in range(3)]
    want = ba.attention(*x, None, d ** -0.5)
    got = ba.attention(*(t.expand(1, H, N, d) for t in x), None, d ** -0.5)
    torch.cuda.synchronize()
    # (an output's last bits depend on where in the grid its head lies)
    assert torch.isfinite(got[0, -100:]).all() and (got[0, -100:].float() - want[0].float()).abs().max() <= 2e-3
    worst = max((got[0, h:h + 65536].float() - want[0].float()).abs().amax().item() for h in range(0, H, 65536))
    del got
    torch.cuda.empty_cache()
    assert worst <= 2e-3


# (grids of rows of 64 stay off the single launch: items of one or two key blocks, several of them in turn in a workgroup)
@pytest.mark.parametrize("Gy,d,flags", [(1, 64, 0), (2, 72, 0), (4, 64, 0), (1, 64, ba.FLAG_NO_BIAS), (1, 72, ba.FLAG_NO_BIAS), (3, 72, ba.FLAG_NO_BIAS),
                                        (1, 128, ba.FLAG_NO_BIAS), (1, 32, ba.FLAG_NO_BIAS | ba.FLAG_LUT)])
def test_abs_means_of_the_head_after_the_next_with_short_items(Gy, d, flags):
    B, H, Gx = 350, 8, 64
    N = Gy * Gx
    say(f"abs-means by powers of two, {Gy} x {Gx} grid d={d} flags={flags}")
    g = torch.Generator(device="cuda")
    g.manual_seed(d + Gy)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda") for _ in range(3))
    for t in (q, k):
        t *= torch.exp2(torch.randint(-3, 4, (B, H, 1, 1), generator=g, device="cuda").float())
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    table = torch.randn(H, 2 * Gy - 1, 2 * Gx - 1, generator=g, device="cuda") * 0.3
    mq, mk = (torch.full((B, H), float("nan"), device="cuda") for _ in range(2))
    got = ba.attention_relpos(q, k, v, table, d ** -0.5, mu_q=mq, mu_k=mk, flags=flags)
    qb, kb, _, _ = ba.pack_qk(q, k)
    want = ba.forward_relpos(qb, kb, mq, mk, v, table, d ** -0.5, flags=flags)
    torch.cuda.synchronize()
    for mu, x in ((mq, q), (mk, k)):
        assert torch.allclose(mu.double(), x.double().abs().mean(dim=(2, 3)), rtol=1e-5, atol=0)
    assert torch.equal(got, want)
