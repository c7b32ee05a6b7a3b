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
    # bands of output channels (more tiles than channels) and of tiles, the last one narrower
    (1, 72, 96, 512, 160, 6, 64), (1, 60, 96, 512, 224, 6, 64),
    # more than 512 blocks of F(6,3): half of the columns a pass
    (1, 96, 96, 96, 1080, 6, 32),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%dx%d_%d-%d_F%d_g%d" % s)
def test_rounds_bands_and_passes(shape):
    N, H, W, Cin, Cout, m, g = shape
    d = workloads.small_layer(77, N, H, W, Cin, Cout, m, g)
    ran = 0
    for variant in FUSED:
        try:
            parity.check(wqmod, d, want_P=N * H * W < 1000, variant=variant)   # codes and sums bit for bit, y to 1e-5
            ran += 1
        except wqmod.WqError as e:
            assert e.status == 2, e      # the variant does not apply to this shape
    assert ran >= 1


@pytest.mark.parametrize("shape,other", [
    ((1, 128, 128, 64, 512, 4, 32), "lds_full_32x32"), ((1, 126, 127, 192, 512, 4, 64), "lds_full_32x32"),
    ((1, 128, 126, 288, 256, 4, 32), "lds_row_64x64"), ((1, 125, 128, 512, 256, 4, 64), "lds_row_64x64"),
    ((2, 64, 62, 128, 96, 4, 32), "lds_tap_64x64"),
], ids=lambda v: v if isinstance(v, str) else "%dx%dx%d_%d-%d_F%d_g%d" % v)
def test_the_sums_of_a_layer_do_not_depend_on_the_form_that_runs_it(shape, other):
    """Layers that a chain quantizes again: every fused tile gives the bits of the LDS form of their size."""
    N, H, W, Cin, Cout, m, g = shape
    gen = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((N, H, W, Cin), generator=gen, device="cuda")
    plan = wqmod.Plan(*shape)
    blob, ws = plan.alloc_blob(), plan.alloc_workspace()
    plan.weight_prepare(torch.randn((Cout, Cin, 3, 3), generator=gen, device="cuda"),
                        torch.randn(Cout, generator=gen, device="cuda"), blob)
    got = {}
    for variant in (other, "fused_16x16", "fused_32x16", "fused_32x32"):
        plan.tune(0, variant)
        y = torch.full((N, H, W, Cout), float("nan"), device="cuda")
        plan.forward(x, blob, ws, y)
        got[variant] = y
    for variant, y in got.items():
        assert torch.equal(y, got[other]), variant
