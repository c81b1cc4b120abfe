"""What the compiler made of the kernels (registers, scratch, LDS), from the resource-usage remarks
the build collects.  A register spill inside the block loop of the fused kernel is not a
correctness problem but a performance cliff (its reload waits on the same counter as the
asynchronous copies of the next key block), and nothing else would notice it: so it is pinned here."""
import re

import pytest

from paper_2603_09582_amd import build

HALF = 16  # added to the form where d ends in the first half of the last 32 channels: d = 40, 48 (DK = 2), 72, 80 (DK = 3)

# fused_kernel<DK, MODE, NB, FORM> variants that are known to spill, and how many bytes: head dimension above 96, the
# single-launch form with a bias that is read straight into registers (row pitches from 2^27 elements on).
KNOWN_SPILLS = {(4, 1, 2, 1): 32}


def fused_variants():
    res = build.kernel_resources()
    if not res:
        pytest.skip("no build in this tree yet (python -m paper_2603_09582_amd.build)")
    out = {}
    for name, r in res.items():
        m = re.match(r"_ZN7binattn12fused_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)EEEv", name)
        if m:
            out[tuple(int(x) for x in m.groups())] = r
    return out


def test_fused_kernels_do_not_spill_and_keep_two_waves_per_simd():
    fv = fused_variants()
    assert len(fv) >= 40
    for key, r in sorted(fv.items()):
        assert r["waves_per_simd"] >= 2, (key, r)
        assert r["lds_bytes"] <= 160 * 1024, (key, r)
        if key in KNOWN_SPILLS:
            assert r["scratch_bytes"] <= KNOWN_SPILLS[key], (key, r)
        else:
            assert r["scratch_bytes"] == 0, (key, r)


def forms(*numbers):
    return {k: r for k, r in fused_variants().items() if k[3] & (HALF - 1) in numbers}


def with_halves(keys):
    return {(dk, mode, nb, form + half) for dk, mode, nb, form in keys for half in ((0, HALF) if dk in (2, 3) else (0,))}


def test_headline_kernels_have_the_expected_shape():
    fv = fused_variants()
    for once in (0, 4, HALF, 4 + HALF):  # 32 < d <= 64, LDS bias tiles shared by two batch entries (long sequences); 4: streamed bias
        pair = fv[(2, 5, 2, once)]
        assert pair["vgprs"] <= 256 and pair["scratch_bytes"] == 0 and 100 * 1024 <= pair["lds_bytes"] <= 128 * 1024
    for mode in (5, 17):                 # 64 < d <= 96, private bias tiles, two workgroups per compute unit; 17: N a multiple of 8
        for half in (0, HALF):           # d = 72 runs the half form
            dit = fv[(3, mode, 1, half)]
            assert dit["scratch_bytes"] == 0 and dit["lds_bytes"] <= 80 * 1024


def fits_three(r):
    return r["waves_per_simd"] >= 3 and r["vgprs"] <= 168 and r["scratch_bytes"] == 0 and 3 * r["lds_bytes"] <= 160 * 1024


def test_three_wave_kernels_fit_three_per_compute_unit():
    """The launcher sizes their grid at three workgroups per compute unit: registers and LDS for that many."""
    three = forms(5)   # WIDE_WAVES3
    assert set(three) == with_halves({(1, 0, 1, 5), (2, 0, 1, 5), (1, 5, 1, 5), (1, 17, 1, 5), (1, 7, 1, 5), (2, 7, 1, 5), (1, 13, 1, 5), (2, 13, 1, 5)})
    for key, r in sorted(three.items()):
        assert fits_three(r), (key, r)


def test_single_launch_kernels_that_are_split_for_rounds_of_768_fit_three_per_compute_unit():
    three = forms(8, 9)   # WIDE_TRI4, WIDE_TRISHORT4
    assert set(three) == with_halves({(2, 0, 1, 8), (2, 0, 1, 9), (2, 5, 1, 9)})
    # up to 32 channels, without a bias and with bf16 tiles, the forms for two do as well (WIDE_ONEHEAD4, WIDE_SHORT4)
    narrow = {k: r for k, r in forms(3, 7).items() if k[0] == 1 and k[1] in (0, 5)}
    assert set(narrow) == {(1, 0, 1, 3), (1, 0, 1, 7), (1, 5, 1, 3), (1, 5, 1, 7)}
    for key, r in sorted({**three, **narrow}.items()):
        assert fits_three(r), (key, r)


def test_four_wave_single_launch_kernels_fit_two_per_compute_unit():
    four = forms(3, 7)   # WIDE_ONEHEAD4, WIDE_SHORT4
    modes = {1: (0, 1, 3, 5, 7, 9, 11, 15), 2: (1, 3, 5, 7, 9, 11, 15), 3: (0, 3, 5, 7, 9, 15)}  # (2, 0: WIDE_TRI4 alone)
    short = {(dk, m, 1, 7) for dk, ms in modes.items() for m in ms if m in (0, 5, 15)}
    assert set(four) == with_halves({(dk, m, 1, 3) for dk, ms in modes.items() for m in ms} | short)
    for key, r in sorted(four.items()):
        assert r["scratch_bytes"] == 0 and r["lds_bytes"] <= 80 * 1024, (key, r)
