"""GPU tests of the fused contraction's walk: scales that come in rounds of n groups whatever the groups
of a tap, bands of the operand that does not fit an XCD's L2, both passes of its output stage, and sums
that do not depend on the form that runs a layer."""
import pytest
import torch

import test_parity_gpu as parity
from paper_2412_19867_amd import wq as wqmod
from paper_2412_19867_amd import workloads

pytestmark = pytest.mark.gpu

FUSED = ["fused_16x16", "fused_ksplit", "fused_32x16", "fused_32x32"]
SHAPES = [   # N H W Cin Cout m g: groups per tap below, at and above the taps of a round, dividing it or not
    (1, 9, 14, 64, 33, 4, 64), (2, 10, 9, 160, 40, 4, 32), (1, 13, 22, 384, 64, 4, 64), (3, 8, 11, 448, 70, 4, 64),
    (1, 9, 9, 320, 24, 4, 32), (1, 12, 13, 224, 36, 6, 32), (1, 15, 11, 512, 48, 6, 64), (1, 7, 20, 704, 32, 6, 64),
    (1, 7, 9, 192, 40, 2, 64), (1, 6, 11, 320, 17, 2, 64),
    # half of the channels per XCD; one or two blocks of tiles at a time
    (1, 72, 96, 512, 160, 6, 64), (1, 60, 96, 512, 224, 6, 64),
    # more than 512 blocks of F(6,3): half of the columns a pass
    (1, 96, 96, 96, 1080, 6, 32),
]


ALL_TILES = ("fused_16x16", "fused_32x16", "fused_32x32")


def forward_with(shape, variant, x, w, bias):
    plan = wqmod.Plan(*shape).tune(0, variant)
    blob, ws = plan.alloc_blob(), plan.alloc_workspace()
    plan.weight_prepare(w, bias, blob)
    y = torch.full((shape[0], shape[1], shape[2], shape[4]), float("nan"), device="cuda")
    plan.forward(x, blob, ws, y)
    return plan.k2_variant_name, y


def inputs(shape):
    N, H, W, Cin, Cout, m, g = shape
    gen = torch.Generator(device="cuda").manual_seed(5)
    return (torch.randn((N, H, W, Cin), generator=gen, device="cuda"), torch.randn((Cout, Cin, 3, 3), generator=gen, device="cuda"),
            torch.randn(Cout, generator=gen, device="cuda"))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%dx%d_%d-%d_F%d_g%d" % s)
def test_rounds_bands_and_passes(shape):
    N, H, W, Cin, Cout, m, g = shape
    d = workloads.small_layer(77, N, H, W, Cin, Cout, m, g)
    for variant in FUSED:
        if variant == "fused_16x16" or (m != 2 and (variant != "fused_ksplit" or (Cin // g) % 2 == 0)):
            parity.check(wqmod, d, want_P=N * H * W < 1000, variant=variant)   # codes and sums bit for bit, y to 1e-5
        else:
            with pytest.raises(wqmod.WqError):
                wqmod.Plan(*shape).tune(0, variant)


# Layers whose operand that the XCDs do not share out passes in bands, the last one narrower, with one and with four
# blocks per workgroup: which XCDs share out (0: channels, 1: tiles), (band, last band) of each
BANDS = [
    ((1, 192, 228, 128, 1184, 6, 64), 1, (8, 2), (4, 1)), ((1, 124, 124, 256, 928, 4, 64), 1, (7, 2), (3, 2)),
    ((1, 192, 222, 128, 1184, 6, 64), 0, (8, 2), (4, 1)), ((1, 124, 116, 256, 928, 4, 64), 0, (7, 2), (3, 2)),
]


@pytest.mark.parametrize("shape", [b[0] for b in BANDS], ids=lambda s: "%dx%dx%d_%d-%d_F%d_g%d" % s)
def test_bands_with_a_narrower_last_one(shape):
    """Every output, bit for bit, as the LDS form whose order of additions the layer has: the full form's on F(4,3) layers
    of its size, otherwise the tap form's (up to 8 groups in one chain of fp32)."""
    data = inputs(shape)
    want = forward_with(shape, "lds_full_32x32" if shape[5] == 4 else "lds_tap_64x64", *data)[1]
    assert not torch.isnan(want).any()
    for variant in ALL_TILES:
        assert torch.equal(forward_with(shape, variant, *data)[1], want), variant


# (a fused tile the caller picks on a layer of the row form's size sums more precisely than that form above 8 groups:
# there only the plan's own pick has its bits)
@pytest.mark.parametrize("shape,other,forms", [
    ((1, 128, 128, 64, 512, 4, 32), "lds_full_32x32", ALL_TILES), ((1, 126, 127, 192, 512, 4, 64), "lds_full_32x32", ALL_TILES),
    ((1, 128, 126, 288, 256, 4, 32), "lds_row_64x64", ("auto",)), ((1, 125, 128, 512, 256, 4, 64), "lds_row_64x64", ALL_TILES),
    ((2, 64, 62, 128, 96, 4, 32), "lds_tap_64x64", ALL_TILES),
    # F(6,3), whose output transform cancels most: below, at and above the row form's 16 groups of fp32
    ((1, 96, 94, 288, 768, 6, 32), "lds_row_64x64", ("auto",)), ((1, 94, 96, 512, 768, 6, 32), "lds_row_64x64", ("auto",)),
    ((1, 96, 96, 544, 768, 6, 32), "lds_row_64x64", ("auto",) + ALL_TILES),
], ids=lambda v: v if isinstance(v, str) else "-".join(v) if isinstance(v[0], str) else "%dx%dx%d_%d-%d_F%d_g%d" % v)
def test_the_sums_of_a_layer_do_not_depend_on_the_form_that_runs_it(shape, other, forms):
    """Layers that a chain quantizes again: the fused kernel gives the bits of the LDS form of their size."""
    data = inputs(shape)
    want = forward_with(shape, other, *data)[1]
    for form in forms:
        name, y = forward_with(shape, form, *data)
        assert torch.equal(y, want), name


@pytest.mark.parametrize("shape", [(1, 128, 126, 288, 256, 4, 32), (1, 96, 96, 384, 768, 6, 32), (1, 96, 96, 576, 768, 6, 32)],
                         ids=lambda s: "%dx%dx%d_%d-%d_F%d_g%d" % s)
def test_a_fused_form_the_caller_picks_sums_alike_on_layers_of_every_size(shape):
    """The fp64 totals above 8 groups of a wave do not go away where a layer is of the row form's size: the upper
    half of the image, which is not, has the same bits (a tile's codes and sums depend on its own patch alone)."""
    N, H, W, Cin, Cout, m, g = shape
    x, w, bias = inputs(shape)
    half = (N, H // 2, W, Cin, Cout, m, g)
    rows = (H // 2 // m) * m - m      # output rows whose patches lie inside the upper half
    for variant in FUSED:
        try:
            y = forward_with(shape, variant, x, w, bias)[1]
        except wqmod.WqError as e:
            assert variant == "fused_ksplit" and (Cin // g) % 2, e
            continue
        top = forward_with(half, variant, x[:, :H // 2].contiguous(), w, bias)[1]
        assert torch.equal(y[:, :rows], top[:, :rows]), variant


@pytest.mark.parametrize("variant", FUSED)
def test_an_output_that_starts_at_any_float(variant):
    """The output stage stores four channels at a time; y need not start at a multiple of 16 bytes."""
    shape = (2, 13, 11, 128, 40, 4, 64)
    x, w, bias = inputs(shape)
    want = forward_with(shape, variant, x, w, bias)[1]
    plan = wqmod.Plan(*shape).tune(0, variant)
    blob, ws = plan.alloc_blob(), plan.alloc_workspace()
    plan.weight_prepare(w, bias, blob)
    for at in (1, 2, 3):
        store = torch.full((want.numel() + 8,), float("nan"), device="cuda")
        plan.forward(x, blob, ws, store[at:at + want.numel()].view(want.shape))
        assert torch.equal(store[at:at + want.numel()].view(want.shape), want)
        assert torch.isnan(store[:at]).all() and torch.isnan(store[at + want.numel():]).all()
