"""The bf16 kernels that grids of more than one round of the chip run on, which small test grids do not reach (their waves
share the streamed side in groups): the backward pair at every padded width, with LSE and delta in columns, in the C operand
and mixed, tiles of 32 and 64 tokens, sides that are and are not multiples of 8, 16- and 8-byte pieces, dkv in workgroups of
three, four and eight waves, packed and gated; and the forward of the same calls.  Every element against the oracle,
which computes the two images that the batch repeats; the kernels' names are checked where the chip has 256 compute units.

Bounds: 2e-2 for every element, as in the parity tests, and REL in the 2-norm: roundings to bf16, of at most 2^-8 each, enter a
gradient with Q_aug (through the logits), with P or dS and with the result, which is 2.6 times 2^-8 if none cancel.  (An image
left out of the sums of 72 is 1.4e-2.)"""
import pytest

pytestmark = pytest.mark.gpu

from paper_2603_06738_amd import workloads as wk

REL = 1e-2

CASES = [  # (d, r, M, shift, windows across, heads, images, kind, "columns, tile, XS, XD, aligned, pieces" of dq, dkv's pieces, dkv's threads)
    (16, 14, 24, 12, 2, 2, 24, "", "32, 32, false, false, true, 0", 0, 256),
    (16, 16, 23, 5, 2, 2, 24, "", "32, 32, true, false, false, 0", 0, 256),
    (30, 16, 24, 0, 2, 2, 24, "", "48, 32, false, false, true, 0", 0, 256),
    (30, 18, 24, 12, 2, 2, 24, "packed", "48, 32, true, false, true, 0", 0, 256),
    (30, 18, 23, 22, 2, 2, 24, "", "48, 32, true, false, false, 0", 0, 256),
    (32, 16, 24, 7, 2, 2, 24, "", "48, 32, true, true, true, 0", 0, 256),
    (30, 34, 24, 0, 2, 2, 24, "", "64, 32, true, false, true, 0", 0, 256),
    (32, 32, 24, 3, 2, 2, 24, "packed", "64, 32, true, true, true, 0", 4, 256),
    (24, 34, 23, 1, 2, 2, 24, "", "64, 32, false, false, false, 0", 0, 256),
    (16, 14, 25, 4, 2, 2, 24, "", "32, 64, false, false, false, 0", 0, 256),
    (16, 16, 48, 0, 1, 3, 10, "gated", "32, 64, true, false, true, 0", 0, 256),
    (30, 16, 32, 16, 1, 3, 24, "gated", "48, 64, false, false, true, 0", 0, 256),
    (30, 16, 25, 0, 2, 2, 24, "packed", "48, 64, false, false, false, 0", 0, 256),
    (30, 18, 41, 20, 1, 2, 20, "", "48, 64, true, false, false, 0", 0, 256),
    (30, 18, 40, 9, 1, 2, 20, "", "48, 64, true, false, true, 0", 0, 256),
    (32, 16, 25, 3, 2, 2, 24, "", "48, 64, true, true, false, 0", 0, 256),
    (32, 8, 25, 0, 2, 2, 24, "", "48, 64, false, true, false, 0", 0, 256),
    (32, 8, 32, 8, 1, 3, 24, "", "48, 64, false, true, true, 0", 0, 256),
    (30, 34, 41, 0, 1, 2, 20, "", "64, 64, true, false, false, 0", 0, 256),
    (32, 32, 25, 24, 2, 2, 24, "gated", "64, 64, true, true, false, 0", 0, 256),
    (24, 34, 25, 6, 2, 2, 24, "", "64, 64, false, false, false, 0", 0, 256),
    (30, 34, 32, 0, 1, 3, 24, "packed", "64, 64, true, false, true, 0", 4, 256),
    (32, 32, 40, 11, 1, 2, 20, "", "64, 64, true, true, true, 0", 4, 256),
    (32, 32, 48, 0, 1, 2, 72, "", "64, 64, true, true, true, 0", 4, 512),
    (32, 32, 45, 13, 1, 4, 48, "", "64, 64, true, true, false, 0", 4, 512),
    (16, 14, 23, 0, 2, 2, 24, "", "32, 32, false, false, false, 0", 0, 256),
    (16, 14, 32, 7, 1, 3, 24, "", "32, 64, false, false, true, 0", 0, 256),
    (16, 16, 25, 0, 2, 2, 24, "gated", "32, 64, true, false, false, 0", 0, 256),
    (30, 16, 23, 9, 2, 2, 24, "", "48, 32, false, false, false, 0", 0, 256),
    (32, 8, 23, 0, 2, 2, 24, "", "48, 32, false, true, false, 0", 0, 256),
    (32, 8, 24, 1, 2, 2, 24, "", "48, 32, false, true, true, 0", 0, 256),
    (32, 16, 23, 3, 2, 2, 24, "", "48, 32, true, true, false, 0", 0, 256),
    (32, 16, 32, 0, 1, 3, 24, "", "48, 64, true, true, true, 0", 0, 256),
    (24, 34, 24, 5, 2, 2, 24, "", "64, 32, false, false, true, 0", 0, 256),
    (32, 24, 23, 0, 2, 2, 24, "", "64, 32, false, true, false, 0", 0, 256),
    (32, 24, 24, 23, 2, 2, 24, "", "64, 32, false, true, true, 0", 0, 256),
    (30, 34, 23, 4, 2, 2, 24, "", "64, 32, true, false, false, 0", 0, 256),
    (32, 32, 23, 0, 2, 2, 24, "", "64, 32, true, true, false, 0", 0, 256),
    (24, 34, 32, 0, 1, 3, 24, "", "64, 64, false, false, true, 0", 4, 256),
    (32, 24, 25, 2, 2, 2, 24, "", "64, 64, false, true, false, 0", 0, 256),
    (32, 24, 32, 31, 1, 3, 24, "", "64, 64, false, true, true, 0", 4, 256),
    (24, 34, 31, 0, 1, 4, 64, "", "64, 64, false, false, false, 0", 4, 512),
    (32, 24, 31, 5, 1, 4, 64, "", "64, 64, false, true, false, 0", 4, 512),
    (32, 24, 32, 0, 1, 4, 64, "", "64, 64, false, true, true, 0", 4, 512),
    (30, 34, 31, 8, 1, 4, 64, "packed", "64, 64, true, false, false, 0", 4, 512),
    (6, 4, 24, 2, 2, 2, 24, "", "32, 32, false, false, true, 4", 4, 256),
    (30, 4, 32, 0, 1, 3, 24, "", "48, 64, false, false, true, 4", 4, 256),
    (30, 6, 25, 0, 2, 2, 24, "packed", "48, 64, false, false, false, 4", 4, 256),
    (6, 4, 23, 0, 2, 2, 24, "", "32, 32, false, false, false, 4", 4, 256),
    (6, 4, 32, 3, 1, 3, 24, "", "32, 64, false, false, true, 4", 4, 256),
    (6, 26, 24, 0, 2, 2, 24, "", "32, 32, true, false, true, 4", 4, 256),
    (4, 28, 25, 1, 2, 2, 24, "", "32, 64, true, false, false, 4", 4, 256),
    (30, 4, 23, 0, 2, 2, 24, "", "48, 32, false, false, false, 4", 4, 256),
    (32, 4, 24, 5, 2, 2, 24, "", "48, 32, false, true, true, 4", 4, 256),
    (32, 6, 25, 0, 2, 2, 24, "", "48, 64, false, true, false, 4", 4, 256),
    (4, 44, 24, 0, 2, 2, 24, "", "64, 32, false, false, true, 4", 4, 256),
    (4, 44, 25, 6, 2, 2, 24, "", "64, 64, false, false, false, 4", 4, 256),
    (4, 60, 23, 0, 2, 2, 24, "", "64, 32, true, false, false, 4", 4, 256),
    (6, 58, 32, 9, 1, 3, 24, "", "64, 64, true, false, true, 4", 4, 256),
]


@pytest.mark.parametrize("d,r,M,s,nx,heads,images,kind,dq,pieces,threads", CASES)
def test_backward_pair_of_large_grids(oracle, d, r, M, s, nx, heads, images, kind, dq, pieces, threads):
    import torch
    import gpu_helpers as gh
    wl = wk.custom(f"many-d{d}r{r}m{M}", "bf16", 1, M, nx * M, heads, d, r, M, s, 12000 + 64 * M + d + r)
    got, ref, names = gh.many_images(oracle, wl, images, packed=kind == "packed", gated=kind == "gated")
    if names and torch.cuda.get_device_properties(0).multi_processor_count == 256:
        dkv = dq[:-1] + f"{pieces}, false, {threads}, 1>"
        for kern in (f"dq_kernel<{dq}, false, 256, 1>", f"dkv_kernel<{dkv}"):
            assert any(kern in n for n in names), (kern, names)
    for name, a, b in zip(gh.NAMES + ("dG",), got, ref):
        a = gh.host(a)
        if name[:2] != "dF":
            assert gh.max_abs(a, b) <= gh.TOL["bf16"], name
        assert gh.rel(a, b) <= REL, name


@pytest.mark.parametrize("d,r,M,s,images,kern", [
    (5, 3, 12, 0, 64, "<16, 32>"), (16, 14, 12, 5, 64, "<32, 32>"), (30, 17, 12, 0, 64, "<48, 32>"), (32, 32, 12, 3, 64, "<64, 32>"),
    (9, 4, 16, 0, 64, "<16, 64>"), (14, 18, 16, 8, 64, "<32, 64>"), (30, 8, 22, 0, 32, "<48, 64>"), (31, 30, 16, 1, 64, "<64, 64>"),
], ids=lambda v: v if isinstance(v, str) else None)
def test_fp32_kernels_of_large_grids(oracle, d, r, M, s, images, kern):
    """The fp32 kernels without groups of waves, tiles of 32 and 64 tokens at every padded width."""
    import torch
    import gpu_helpers as gh
    wl = wk.custom(f"many-f32-d{d}r{r}m{M}", "f32", 1, M, 2 * M, 3, d, r, M, s, 13000 + 64 * M + d + r)
    got, ref, names = gh.many_images(oracle, wl, images)
    if names and torch.cuda.get_device_properties(0).multi_processor_count == 256:
        for n in ("dq_kernel", "dkv_kernel"):
            assert any(f"split::{n}{kern}" in k for k in names), names
    for name, a, b in zip(gh.NAMES, got, ref):
        a = gh.host(a)
        if name[:2] != "dF":
            assert gh.max_abs(a, b) <= gh.TOL["f32"], name
        # every product is good to 2.5 * 2^-24, and sums of N terms of fp32 add half a unit at random each: 2^-24 sqrt(N)
        assert gh.rel(a, b) <= 2.0 ** -24 * (2.5 + M), name
