"""The attention layers whose speed is followed, each through the library's public entry points.

A case is one attention layer as a vision or diffusion transformer calls it: the bf16 Q, K, V of
the projections come in, the bf16 output (and, where the caller packs the signs itself, the sign
words and abs-means) go out.  `listed` names the layers, `draw` gives others of the same ranges.

A case: entry  "attention"  one call from Q, K, V, dense bias or none (binding.attention)
               "relpos"     one call from Q, K, V, full relative-position table (binding.attention_relpos)
               "packed"     pack_qk, then forward with a dense bias or none
               "packed_axial"   pack_qk, then forward_axial (decomposed relative-position bias)
        B, H, N, d      problem size; N = Gy * Gx for the two grid entries
        bias            "none", "bf16" or "fp32": a dense [H, N, N] shared over the batch
        Gy, Gx          token grid (0 where there is none)
        extra           input recipe of workloads.make_inputs
"""
import math

import torch

from paper_2603_09582_amd import binding as ba
from paper_2603_09582_amd import workloads as wl


def _case(entry, B, H, N, d, bias="none", Gy=0, Gx=0, extra="", name=None):
    c = {"entry": entry, "B": B, "H": H, "N": N, "d": d, "bias": bias, "Gy": Gy, "Gx": Gx, "extra": extra}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # one image through the smallest ViT: three heads, latency and launches count
        _case("attention", 1, 3, 197, 64, "bf16", name="vit_tiny_one_image"),
        # a serving batch of a base-size ViT at 224 px; N = 196 patches + class token, odd bias rows
        _case("attention", 64, 12, 197, 64, "bf16", extra="k_channel_offset", name="vit_base_batch"),
        # one layer of a diffusion transformer at 256 px (16 x 16 latent patches), d = 72
        _case("attention", 32, 16, 256, 72, "bf16", name="dit_256px"),
        # the same at 512 px (32 x 32 latent patches) with the dense bias ...
        _case("attention", 8, 16, 1024, 72, "bf16", name="dit_512px"),
        # ... and with the trainable table of relative positions it is made from
        _case("relpos", 8, 16, 1024, 72, Gy=32, Gx=32, name="dit_512px_table"),
        # fine-tuning resolution (24 x 24 patches + class token), bias parameter kept in fp32
        _case("packed", 16, 12, 577, 64, "fp32", name="vit_base_fp32_bias"),
        # 37 x 37 patches + class token, d = 80: rows that are aligned to nothing
        _case("attention", 4, 16, 1370, 80, "bf16", name="vit_d80_odd_rows"),
        # the long-sequence ViT (128 x 128 patches) with the dense bias: the largest call
        _case("packed", 2, 16, 16384, 64, "bf16", extra="token_outliers", name="vit_hires"),
        # the same layer with the decomposed bias, which needs no [N, N] tensor ...
        _case("packed_axial", 2, 16, 16384, 64, Gy=128, Gx=128, extra="token_outliers", name="vit_hires_axial"),
        # ... and with the full table
        _case("relpos", 2, 16, 16384, 64, Gy=128, Gx=128, extra="token_outliers", name="vit_hires_table"),
        # head dimension 128 without bias (the setting of kernel speed comparisons)
        _case("attention", 4, 16, 4096, 128, name="hd128_no_bias"),
        # and with one
        _case("attention", 8, 16, 2048, 128, "bf16", name="hd128_bias"),
    ]


def draw(rng):
    """Another layer: heads 3 .. 16, head dimensions in use, 50 .. 16384 tokens (odd and even),
    every bias form, and a batch that keeps the call below the largest listed one."""
    entry = rng.choice(["attention", "attention", "packed", "relpos", "packed_axial"])
    H = rng.choice([3, 4, 6, 8, 12, 16])
    d = rng.choice([32, 48, 64, 64, 72, 80, 96, 128])
    extra = rng.choice(["", "", "k_channel_offset", "token_outliers"])
    Gy = Gx = 0
    bias = "none"
    if entry in ("relpos", "packed_axial"):
        Gx = rng.choice([16, 32, 64, 128])
        Gy = min(128, max(4, round(math.exp(rng.uniform(math.log(Gx / 4), math.log(2 * Gx))))))
        N = Gy * Gx
    else:
        N = round(math.exp(rng.uniform(math.log(50), math.log(16384))))
        bias = rng.choice(["none", "bf16", "bf16", "bf16", "fp32"])
        if bias != "none":  # at most 4 GB of bias
            N = min(N, int(math.sqrt(4.0e9 / (H * (2 if bias == "bf16" else 4)))))
    most = max(1.0, min(64.0, 2.0e9 / (H * N * N), 6.0e7 / (H * N * d)))
    B = max(1, round(math.exp(rng.uniform(0.0, math.log(most)))))
    return _case(entry, B, H, N, d, bias, Gy, Gx, extra)


def _inputs(case, seed):
    w = wl.custom_workload(case["B"], case["H"], case["N"], case["d"], int(seed), case["extra"])
    x = wl.make_inputs(w, device="cuda", with_bias=case["bias"] != "none",
                       bias_dtype=torch.float32 if case["bias"] == "fp32" else torch.bfloat16)
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 7919)

    def table(*s):
        return torch.randn(*s, generator=g, device="cuda", dtype=torch.float32) * 0.02

    H, Gy, Gx = case["H"], case["Gy"], case["Gx"]
    t = table(H, 2 * Gy - 1, 2 * Gx - 1) if case["entry"] == "relpos" else None
    by, bx = (table(H, 2 * Gy - 1), table(H, 2 * Gx - 1)) if case["entry"] == "packed_axial" else (None, None)
    return x, t, by, bx


def prepare(case, seed):
    """The tensors of the layer and the workspace such a program keeps for its shape."""
    x, t, by, bx = _inputs(case, seed)
    ws = ba.alloc_workspace(case["B"], case["H"], case["N"], case["d"])
    return {"entry": case["entry"], "q": x.q, "k": x.k, "v": x.v, "bias": x.bias, "scale": x.scale,
            "table": t, "by": by, "bx": bx, "ws": ws}


def run(s):
    if s["entry"] == "attention":
        return {"out": ba.attention(s["q"], s["k"], s["v"], s["bias"], s["scale"], workspace=s["ws"])}
    if s["entry"] == "relpos":
        return {"out": ba.attention_relpos(s["q"], s["k"], s["v"], s["table"], s["scale"], workspace=s["ws"])}
    q_bits, k_bits, mu_q, mu_k = ba.pack_qk(s["q"], s["k"])
    if s["entry"] == "packed":
        out = ba.forward(q_bits, k_bits, mu_q, mu_k, s["v"], s["bias"], s["scale"], workspace=s["ws"])
    else:
        out = ba.forward_axial(q_bits, k_bits, mu_q, mu_k, s["v"], s["by"], s["bx"], s["scale"], workspace=s["ws"])
    return {"out": out, "q_bits": q_bits, "k_bits": k_bits, "mu_q": mu_q, "mu_k": mu_k}


def work(case):
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    n = B * H * N * d
    b = 4 * 2 * n  # bf16 Q, K, V in, the output out
    b += {"none": 0, "bf16": 2, "fp32": 4}[case["bias"]] * H * N * N
    if case["entry"] == "relpos":
        b += 4 * H * (2 * case["Gy"] - 1) * (2 * case["Gx"] - 1)
    if case["entry"] == "packed_axial":
        b += 4 * H * (2 * case["Gy"] + 2 * case["Gx"] - 2)
    if case["entry"].startswith("packed"):  # the sign words and abs-means are results too
        b += 2 * 4 * B * H * (N * ((d + 31) // 32) + 1)
    return {"bytes": b, "flops": 4 * B * H * N * N * d}


def tolerance(case):
    # bf16 outputs (2^-9 of each value) and 8-bit P codes that fall on the other side of a
    # half-integer: about four times the distance to the 64-bit result below.  Sign words are exact.
    return {"rel": 8e-3, "max": 0.1}


def exact(case, seed):
    """The layer in 64 bits: signs, abs-means, 8-bit V per channel, and the online softmax over blocks
    of 128 keys with 8-bit P relative to the running row maximum."""
    x, table, by, bx = _inputs(case, seed)
    B, H, N, d = case["B"], case["H"], case["N"], case["d"]
    Gy, Gx = case["Gy"], case["Gx"]
    out = torch.empty(B, H, N, d, dtype=torch.float64, device="cuda")
    mu_q = torch.empty(B, H, dtype=torch.float64, device="cuda")
    mu_k = torch.empty_like(mu_q)
    rows = torch.arange(N, device="cuda")
    step = max(1, min(H, (1 << 26) // (N * 128)))  # heads at a time
    for b in range(B):
        for h0 in range(0, H, step):
            hs = slice(h0, min(H, h0 + step))
            q, k, v = (t[b, hs].double() for t in (x.q, x.k, x.v))
            mq, mk = q.abs().mean(dim=(1, 2)), k.abs().mean(dim=(1, 2))
            mu_q[b, hs], mu_k[b, hs] = mq, mk
            one = torch.ones((), dtype=torch.float64, device="cuda")
            sq, sk = torch.where(q >= 0, one, -one), torch.where(k >= 0, one, -one)
            delta = v.abs().amax(dim=1, keepdim=True) / 127.0
            delta = torch.where(delta == 0, one, delta)
            codes = torch.round(v / delta)
            alpha = (x.scale * mq * mk)[:, None, None]
            m = torch.full((sq.shape[0], N, 1), -math.inf, dtype=torch.float64, device="cuda")
            l = torch.zeros_like(m)
            o = torch.zeros_like(q)
            for j0 in range(0, N, 128):
                j1 = min(N, j0 + 128)
                S = torch.matmul(sq, sk[:, j0:j1].transpose(1, 2).contiguous()) * alpha
                if x.bias is not None:
                    S += x.bias[hs, :, j0:j1].double()
                if Gx:
                    j = rows[j0:j1]
                    dy = (rows // Gx)[:, None] - (j // Gx)[None, :] + Gy - 1
                    dx = (rows % Gx)[:, None] - (j % Gx)[None, :] + Gx - 1
                    S += (table[hs, dy, dx] if table is not None else by[hs, dy] + bx[hs, dx]).double()
                mn = torch.maximum(m, S.amax(dim=2, keepdim=True))
                p = torch.exp(S - mn)
                r = torch.exp(m - mn)
                l = l * r + p.sum(dim=2, keepdim=True)
                o = o * r + torch.matmul(torch.round(255.0 * p), codes[:, j0:j1].contiguous())
                m = mn
            out[b, hs] = o / (255.0 * l) * delta
    if case["entry"].startswith("packed"):
        return {"out": out, "q_bits": None, "k_bits": None, "mu_q": mu_q, "mu_k": mu_k}
    return {"out": out}
