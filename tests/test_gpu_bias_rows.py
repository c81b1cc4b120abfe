"""Where the rows of a dense bias lie in memory (alignment of the base, row pitch, what follows the last row)
never changes the result: every layout against the oracle, and bit-identical to the contiguous one."""
import numpy as np
import pytest
import torch

from paper_2603_09582_amd import binding as ba
from tests.test_gpu_parity import check_close, dev, gpu_out_f64, oracle_algorithm1, say, small_inputs

pytestmark = pytest.mark.gpu


def placed(bias, offset, extra):
    """The same [H, N, N] values with the first element at `offset` and rows N + extra apart, as the very end
    of a buffer whose other elements are NaN."""
    H, N, _ = bias.shape
    pitch = N + extra
    n = (H * N - 1) * pitch + N
    store = torch.full((offset + n,), float("nan"), dtype=bias.dtype, device="cuda")
    view = store[offset:].as_strided((H, N, N), (N * pitch, pitch, 1))
    view.copy_(bias)
    return view


# (block edges and remainders of the 8-key copy chunks; d = 64 with an even batch and >= 8 key blocks shares
# its tiles between two batch entries, d = 128 takes 8-wave workgroups)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,H,N,d", [(1, 2, 1, 64), (1, 3, 7, 64), (2, 1, 127, 72), (1, 2, 129, 64), (2, 2, 197, 64),
                                     (1, 2, 255, 104), (130, 2, 131, 64), (1, 1, 257, 72), (1, 2, 391, 128), (2, 2, 642, 80),
                                     (3, 1, 577, 64), (2, 2, 577, 32), (4, 1, 965, 64), (2, 1, 1030, 64),
                                     # multiples of 8: no chunk straddles the end of a row
                                     (1, 2, 8, 64), (2, 1, 200, 72), (1, 2, 264, 32), (3, 1, 520, 96), (2, 2, 384, 64)])
def test_bias_rows_of_any_alignment(B, H, N, d, dtype):
    x = small_inputs(B, H, N, d, 900 + N)
    bias = (x.bias.float() * 40.0).to(dtype)  # strong enough that every entry shows in the output
    q, k, v, db = dev(x.q), dev(x.k), dev(x.v), dev(bias)
    ws = ba.alloc_workspace(B, H, N, d)
    qb, kb, mq, mk = ba.pack_qk(q, k)
    plain = {}
    for offset, extra in [(0, 0), (1, 0), (0, 1), (3, 3), (0, -N % 8), (8, 8)]:
        say(f"bias rows B={B} H={H} N={N} d={d} {dtype} offset={offset} pitch=N+{extra}")
        pb = placed(db, offset, extra)
        for name, out in (("packed", ba.forward(qb, kb, mq, mk, v, pb, x.scale, workspace=ws)),
                          ("one call", ba.attention(q, k, v, pb, x.scale, workspace=ws))):
            torch.cuda.synchronize()
            if name not in plain:
                plain[name] = out
                if B * H * N <= 4096:
                    ref = oracle_algorithm1(x, bias)
                    check_close(gpu_out_f64(out), ref, f"{name}: out vs Alg. 1")
            assert torch.equal(out, plain[name]), (name, offset, extra)


@pytest.mark.parametrize("N,d", [(9, 64), (5, 128)])
def test_bias_rows_further_apart_than_a_copy_offset_reaches(N, d):
    """Row pitches from 2^27 elements on take the register path."""
    x = small_inputs(1, 1, N, d, 77)
    pitch = 1 << 27
    store = torch.empty((N - 1) * pitch + N, dtype=torch.bfloat16, device="cuda")
    view = store.as_strided((1, N, N), (N * pitch, pitch, 1))
    view.copy_(dev(x.bias))
    q, k, v = dev(x.q), dev(x.k), dev(x.v)
    qb, kb, mq, mk = ba.pack_qk(q, k)
    ref = oracle_algorithm1(x, x.bias)
    for out in (ba.forward(qb, kb, mq, mk, v, view, x.scale), ba.attention(q, k, v, view, x.scale)):
        torch.cuda.synchronize()
        check_close(gpu_out_f64(out), ref, "giant pitch: out vs Alg. 1")


@pytest.mark.parametrize("B,H,N,d,kind", [(3, 57, 300, 64, "none"), (1, 256, 257, 40, "none"), (1, 129, 513, 16, "none"),
                                          (2, 65, 512, 64, "table"), (1, 87, 720, 40, "table"), (3, 58, 290, 32, "bf16"), (1, 290, 257, 8, "bf16"), (1, 224, 400, 24, "bf16")])
def test_three_workgroups_per_compute_unit_give_the_same_bits(B, H, N, d, kind):
    """More than 512 work items that leave the last round of 512 part empty take the kernels built for three
    waves per SIMD; a few heads of the same call take the others.  Up to 8 key blocks (the accumulator's offset is
    never removed) a head's bits do not depend on what else is in the call."""
    say(f"three waves B={B} H={H} N={N} d={d} {kind}")
    items = B * H * -(-N // 128)
    assert items > 512 and (kind == "table" or 0 < items % 512 <= 384)
    x = small_inputs(B, H, N, d, 300 + N)
    q, k, v = dev(x.q), dev(x.k), dev(x.v)
    bias = None if kind == "none" else dev(x.bias)
    if kind == "table":  # token grid of 16 columns
        table = torch.randn(H, 2 * (N // 16) - 1, 31, generator=torch.Generator().manual_seed(N)).cuda()

    def run(hs):
        if kind == "table":
            return ba.attention_relpos(q[:, hs], k[:, hs], v[:, hs], table[hs], x.scale)
        return ba.attention(q[:, hs], k[:, hs], v[:, hs], None if bias is None else bias[hs], x.scale)

    out = run(slice(0, H))
    for h0 in (0, H - 3):
        hs = slice(h0, h0 + 3)
        part = run(hs)
        torch.cuda.synchronize()
        assert torch.equal(part, out[:, hs]), h0


def removal_phase(heads, nrb):
    """[heads, nrb]: whether the accumulator's offset leaves a row block before key blocks 9, 17, ... (1) or
    8, 16, ... (0), for an odd number of key blocks and batch 1: item u of a call is dealt out as the v-th, and
    v / 512 items of its workgroup come before it in a grid of 512."""
    per = -(-heads * nrb // 8)
    return (np.arange(heads * nrb) % per * 8 // 512 % 2).reshape(heads, nrb)


@pytest.mark.parametrize("kind,d,H1,H2", [("none", 64, 98, 100), ("none", 48, 98, 100), ("bf16", 32, 98, 100), ("table", 64, 150, 3),
                                          ("table", 32, 150, 140), ("axial", 64, 150, 3), ("axial", 32, 150, 140)])
def test_more_than_eight_key_blocks_give_the_same_bits_in_every_grid(kind, d, H1, H2):
    """The same row blocks in calls of H1 and H2 heads, on grids of three or two workgroups per compute unit: where
    the offset is removed before the same key blocks the bits are the same."""
    N, nrb = 1104, 9  # token grid of 69 x 16
    say(f"same bits {kind} d={d} heads {H1} / {H2}")
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    H = max(H1, H2)
    q, k, v = (torch.randn(1, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    bias = torch.randn(H, N, N, generator=g, device="cuda").to(torch.bfloat16) if kind == "bf16" else None
    table = torch.randn(H, 137, 31, generator=g, device="cuda")

    def run(h):
        if kind == "table":
            return ba.attention_relpos(q[:, :h], k[:, :h], v[:, :h], table[:h], d ** -0.5)
        if kind == "axial":
            qb, kb, mq, mk = ba.pack_qk(q[:, :h], k[:, :h])
            return ba.forward_axial(qb, kb, mq, mk, v[:, :h], table[:h, :, 0].contiguous(), table[:h, 0].contiguous(), d ** -0.5)
        return ba.attention(q[:, :h], k[:, :h], v[:, :h], None if bias is None else bias[:h], d ** -0.5)

    n = min(H1, H2)
    a, b = run(H1), run(H2)
    torch.cuda.synchronize()
    same = removal_phase(H1, nrb)[:n] == removal_phase(H2, nrb)[:n]
    assert same.sum() > 10
    for h, rb in zip(*np.nonzero(same)):
        rows = slice(128 * rb, 128 * rb + 128)
        assert torch.equal(a[0, h, rows], b[0, h, rows]), (h, rb)


@pytest.mark.parametrize("B,H,N,d", [(2, 40, 1101, 64), (2, 40, 1101, 32), (2, 40, 1101, 128), (4, 20, 1149, 104)])
def test_more_than_eight_key_blocks_give_the_same_bits_for_odd_and_even_rows(B, H, N, d):
    """Rows of odd alignment go to 8-wave workgroups (pairs of batch entries, of row blocks), rows on 4-byte words
    to 4-wave ones: more than 512 row blocks of an odd number of key blocks, the same bits."""
    assert B * H * (-(-N // 128)) > 512 and -(-N // 128) % 2 == 1
    say(f"odd and even rows B={B} H={H} N={N} d={d}")
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    bias = torch.randn(H, N, N, generator=g, device="cuda").to(torch.bfloat16)
    odd = ba.attention(q, k, v, placed(bias, 0, 0), d ** -0.5)
    even = ba.attention(q, k, v, placed(bias, 0, 1), d ** -0.5)
    torch.cuda.synchronize()
    assert torch.equal(odd, even)
