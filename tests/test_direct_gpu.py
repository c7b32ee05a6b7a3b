"""GPU parity of the group-wise quantized standard convolution against its oracle, with 8-bit
and with 4-bit weight codes (W8A8, W4A8).

Bit-exact on the int8 codes and the fp32 scales of activations and weights; fp32
output within 1e-5 of the layer's largest output magnitude.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2412_19867_amd import workloads

pytestmark = pytest.mark.gpu

Y_TOL = 1e-5


def run_direct(wq, x, w, bias, g, bits=8):
    N, H, W, Cin = x.shape
    Cout = w.shape[0]
    plan = wq.DirectPlan(N, H, W, Cin, Cout, g, weight_bits=bits)
    L = plan.layout
    blob, ws, y = plan.alloc_blob(), plan.alloc_workspace(), plan.alloc_output()
    y.fill_(float("nan"))
    xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    bd = None if bias is None else torch.from_numpy(bias).cuda()
    plan.weight_prepare(wd, bd, blob)
    plan.forward(xd, blob, ws, y)
    torch.cuda.synchronize()
    Wq, sW, b = plan.blob_views(blob)
    xq, sx = plan.workspace_views(ws)
    return dict(wq=Wq[:, :Cout].cpu().numpy(), sw=sW[:, :, :Cout].cpu().numpy(),
                xq=xq.cpu().numpy(), sx=sx.cpu().numpy(), y=y.cpu().numpy(),
                pad_ok=bool((Wq[:, Cout:] == 0).all() and (sW[:, :, Cout:] == 0).all()
                            and (b[Cout:] == 0).all()))


def check_direct(wq, x, w, bias, g, name, bits=8):
    ref = oracle.direct_pipeline(x, w, bias, g, weight_bits=bits)
    got = run_direct(wq, x, w, bias, g, bits)
    assert got["pad_ok"]
    for key in ("wq", "xq"):
        bad = np.count_nonzero(got[key] != ref[key])
        assert bad == 0, f"{name}: {key} differs in {bad} of {ref[key].size} codes"
    for key in ("sw", "sx"):
        assert np.array_equal(got[key].view(np.uint32), ref[key].view(np.uint32)), f"{name}: {key}"
    assert np.isfinite(got["y"]).all(), f"{name}: y has unwritten or non-finite entries"
    scale = np.abs(ref["y64"]).max()
    err = np.abs(got["y"].astype(np.float64) - ref["y64"]).max()
    assert err <= Y_TOL * scale, f"{name}: y max|err| {err:.3e} > {Y_TOL * scale:.3e}"
    print(f"direct {name}: max|err|/max|y| = {err / max(scale, 1e-300):.2e}")


SMALL = [
    # seed N  H   W  Cin Cout  g
    (1, 1, 8, 8, 32, 16, 32),
    (2, 2, 7, 10, 64, 48, 32),        # pixels not a multiple of 64, Cout padded
    (3, 1, 13, 6, 64, 33, 32),        # odd Cout
    (4, 3, 9, 9, 128, 64, 64),
    (5, 2, 12, 12, 256, 32, 128),
    (6, 1, 6, 20, 512, 16, 256),
    (7, 1, 4, 4, 512, 32, 512),
    (8, 5, 11, 11, 96, 80, 32),       # several pixel tiles across image boundaries
    (9, 1, 1, 1, 32, 1, 32),          # a single pixel
    (10, 2, 3, 70, 64, 8, 64),        # rows longer than a pixel tile
]


@pytest.mark.parametrize("bits", [8, 4], ids=["w8", "w4"])
@pytest.mark.parametrize("case", SMALL, ids=lambda c: "d%d_%dx%dx%d_%d-%d_g%d" % c)
def test_direct_small_layers(wq, case, bits):
    seed, N, H, W, Cin, Cout, g = case
    d = workloads.small_layer(seed, N, H, W, Cin, Cout, 4, g)
    check_direct(wq, d.x, d.w, d.bias, g, "small%d" % seed, bits)


def test_direct_no_bias_and_zero_groups(wq):
    d = workloads.small_layer(31, 2, 9, 7, 64, 32, 4, 32)
    d.x[..., :32] = 0
    d.x[0, 0, 0, 32:] *= np.float32(1e-41)      # a sub-normal group
    check_direct(wq, d.x, d.w, None, 32, "nobias")


def test_direct_config1(wq):
    lay = workloads.CONFIGS[1][0]
    d = workloads.make_layer_data(lay)
    check_direct(wq, d.x, d.w, d.bias, lay.group_size, lay.name)


@pytest.mark.parametrize("cfg,idx", [(2, 3), (3, 1), (4, 4)], ids=lambda v: str(v))
def test_direct_config_layers_full_size(wq, cfg, idx):
    lay = workloads.CONFIGS[cfg][idx]
    d = workloads.make_layer_data(lay)
    check_direct(wq, d.x, d.w, d.bias, lay.group_size, lay.name)
    check_direct(wq, d.x, d.w, d.bias, lay.group_size, lay.name + " W4A8", bits=4)


def _random_cases(count, seed):
    rng = np.random.default_rng(seed)
    cases = []
    for k in range(count):
        g = int(rng.choice([32, 32, 64, 128]))
        cases.append((2000 + k, int(rng.integers(1, 4)), int(rng.integers(1, 20)), int(rng.integers(1, 20)),
                      g * int(rng.integers(1, 5)), int(rng.integers(1, 100)), g))
    return cases


@pytest.mark.parametrize("case", _random_cases(12, 2025), ids=lambda c: "r%d_%dx%dx%d_%d-%d_g%d" % c)
def test_direct_random_small_shapes(wq, case):
    seed, N, H, W, Cin, Cout, g = case
    d = workloads.small_layer(seed, N, H, W, Cin, Cout, 4, g)
    check_direct(wq, d.x, d.w, d.bias, g, "random%d" % seed, bits=8 if seed % 2 else 4)


def test_direct_largest_pixel_count(wq):
    """Just under the largest pixel count a plan takes (65535 pixel tiles of 64)."""
    d = workloads.small_layer(78, 1, 2047, 2048, 32, 32, 4, 32)
    check_direct(wq, d.x, d.w, d.bias, 32, "largest")


@pytest.mark.parametrize("case", [
    # P    Cin  Cout  g   (linear: every launch shape of the tile choice, with ragged pixels and channels)
    (16, 64, 33, 32), (17, 128, 16, 64), (257, 192, 260, 64), (400, 128, 1000, 32), (700, 256, 500, 128),
    (1601, 64, 2050, 64), (3300, 64, 2100, 32), (12500, 32, 1030, 32), (192003, 32, 16, 32), (192003, 32, 50, 32),
    (100009, 64, 30, 32), (50003, 128, 32, 32),
], ids=lambda c: "p%d_%d-%d_g%d" % c)
def test_every_tile_choice_of_the_quantized_gemm(wq, case):
    """Rows and channels that end inside a tile, from 16 rows to narrow layers of 192003 (against the
    oracle in fp64); every kernel instance runs in test_every_instance_of_the_quantized_gemm."""
    R, Cin, Cout, g = case
    rng = np.random.default_rng(R)
    x, w = rng.standard_normal((R, Cin)).astype(np.float32), rng.standard_normal((Cout, Cin)).astype(np.float32)
    ref = oracle.linear_pipeline(x, w, None, g)
    plan = wq.DirectPlan(R, 1, 1, Cin, Cout, g, linear=True)
    blob, ws, y = plan.alloc_blob(), plan.alloc_workspace(), plan.alloc_output()
    y.fill_(float("nan"))
    plan.weight_prepare(torch.from_numpy(w).cuda(), None, blob)
    plan.forward(torch.from_numpy(x).cuda(), blob, ws, y)
    got = y.cpu().numpy().reshape(R, Cout).astype(np.float64)
    assert np.isfinite(got).all()
    assert np.abs(got - ref["y64"]).max() <= Y_TOL * np.abs(ref["y64"]).max()


@pytest.mark.parametrize("shape", [(2, 16, 15, 64, 48, 64), (1, 34, 33, 32, 130, 32), (3, 40, 40, 64, 300, 64)],
                         ids=lambda s: "%dx%dx%d_%d-%d_g%d" % s)
@pytest.mark.parametrize("splits", [1, 3, 9])
def test_slices_of_the_quantized_convolution(wq, shape, splits):
    """The reduction shared by 1, 3 or 9 waves, on images whose rows do not match the tiles."""
    N, H, W, Cin, Cout, g = shape
    d = workloads.small_layer(400 + H, N, H, W, Cin, Cout, 4, g)
    ref = oracle.direct_pipeline(d.x, d.w, d.bias, g)
    plan = wq.DirectPlan(N, H, W, Cin, Cout, g).tune(splits)
    blob, ws, y = plan.alloc_blob(), plan.alloc_workspace(), plan.alloc_output()
    ws.fill_(0xff)   # every bit set: a NaN wherever a scale is read that nobody wrote
    y.fill_(float("nan"))
    plan.weight_prepare(torch.from_numpy(d.w).cuda(), torch.from_numpy(d.bias).cuda(), blob)
    plan.forward(torch.from_numpy(d.x).cuda(), blob, ws, y)
    got = y.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    assert np.abs(got - ref["y64"]).max() <= Y_TOL * np.abs(ref["y64"]).max()


def forward_on_poisoned_buffers(wq, x, w, bias, g, bits=8):
    """y of one forward pass with every byte of the workspace 0xff beforehand (NaN as a scale)."""
    N, H, W, Cin = x.shape
    plan = wq.DirectPlan(N, H, W, Cin, w.shape[0], g, weight_bits=bits)
    blob, ws, y = plan.alloc_blob(), plan.alloc_workspace(), plan.alloc_output()
    ws.fill_(0xff)
    y.fill_(float("nan"))
    plan.weight_prepare(torch.from_numpy(w).cuda(), None if bias is None else torch.from_numpy(bias).cuda(), blob)
    plan.forward(torch.from_numpy(x).cuda(), blob, ws, y)
    return y.cpu().numpy()


@pytest.mark.parametrize("bits", [8, 4], ids=["w8", "w4"])
@pytest.mark.parametrize("Cout", [20, 200])
@pytest.mark.parametrize("g", [32, 64, 128])
def test_an_infinite_input_reaches_only_the_windows_that_hold_it(wq, g, Cout, bits):
    """An Inf at the edges of image 1: outputs whose 3x3 window does not hold it, in the same image and
    in its neighbours in the batch, are what they are without it."""
    d = workloads.small_layer(500 + g, 3, 9, 14, 2 * g, Cout, 4, g)
    clean = forward_on_poisoned_buffers(wq, d.x, d.w, d.bias, g, bits)
    assert np.isfinite(clean).all()
    x, held = d.x.copy(), np.zeros(d.x.shape[:3], bool)
    for h, v in ((0, 0), (0, 13), (4, 13), (5, 0), (8, 0), (8, 13)):
        x[1, h, v, (h + v) % (2 * g)] = np.inf if h % 2 else -np.inf
        held[1, max(0, h - 1):h + 2, max(0, v - 1):v + 2] = True
    got = forward_on_poisoned_buffers(wq, x, d.w, d.bias, g, bits)
    assert np.array_equal(got[~held].view(np.uint32), clean[~held].view(np.uint32))
    assert not np.isfinite(got[held]).any()


@pytest.mark.parametrize("W", [1, 5, 64, 200])
@pytest.mark.parametrize("Cout", [1, 32, 33])
def test_a_single_row_of_pixels(wq, W, Cout):
    """One image one pixel high: every tap above and below it lies outside, and a row is as long as all
    the pixels together."""
    d = workloads.small_layer(600 + W, 1, 1, W, 96, Cout, 4, 32)
    ref = oracle.direct_pipeline(d.x, d.w, d.bias, 32)
    got = forward_on_poisoned_buffers(wq, d.x, d.w, d.bias, 32).astype(np.float64)
    assert np.isfinite(got).all()
    assert np.abs(got - ref["y64"]).max() <= Y_TOL * np.abs(ref["y64"]).max()


@pytest.mark.parametrize("exponent", [124, -90])
@pytest.mark.parametrize("bits", [8, 4], ids=["w8", "w4"])
@pytest.mark.parametrize("g", [32, 64, 128])
def test_outputs_near_the_ends_of_the_range(wq, g, bits, exponent):
    """Activations scaled by a power of two scale the outputs by it, exactly, up to the largest floats."""
    d = workloads.small_layer(700 + g, 2, 6, 7, 2 * g, 40, 4, g)
    d.x /= np.float32(8.0)   # |y| stays below 16
    base = forward_on_poisoned_buffers(wq, d.x, d.w, None, g, bits)
    assert 1.0 < np.abs(base).max() < 16.0
    got = forward_on_poisoned_buffers(wq, np.ldexp(d.x, exponent), d.w, None, g, bits)
    want = np.ldexp(base.astype(np.float64), exponent).astype(np.float32)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


def forward_and_fp64_reference(wq, taps, N, H, W, Cin, Cout, g, bits=8, launch=None):
    """y of a layer of random data, and the fp64 sums of the codes and scales it was computed from."""
    gen = torch.Generator(device="cuda").manual_seed(31)
    P, groups = N * H * W, Cin // g
    x = torch.randn(P, Cin, generator=gen, device="cuda")
    w = torch.randn(Cout, Cin * taps, generator=gen, device="cuda")
    plan = wq.DirectPlan(N, H, W, Cin, Cout, g, linear=taps == 1, weight_bits=bits)
    if launch:
        assert plan.launch == launch
    blob, ws, y = plan.alloc_blob(), plan.alloc_workspace(), plan.alloc_output()
    ws.fill_(0xff)
    y.fill_(float("nan"))
    plan.weight_prepare(w, None, blob)
    plan.forward(x, blob, ws, y)
    Wq, sW, _ = plan.blob_views(blob)
    xq, sx = plan.workspace_views(ws)
    xd = (xq.view(P, groups, g).double() * sx.view(P, groups, 1).double()).view(N, H, W, Cin)
    xd = torch.nn.functional.pad(xd, (0, 0, 1, 1, 1, 1))
    ref = torch.zeros(P, Cout, dtype=torch.float64, device="cuda")
    for t in range(taps):
        u, v = (t // 3, t % 3) if taps == 9 else (1, 1)
        wd = Wq[t, :Cout].view(Cout, groups, g).double() * sW[t, :, :Cout].t().unsqueeze(2).double()
        ref += xd[:, u:u + H, v:v + W].reshape(P, Cin) @ wd.view(Cout, Cin).t().contiguous()
    return y.view(P, Cout).double(), ref


@pytest.mark.parametrize("case", [
    # taps N  H   W   Cin   Cout  g   chains
    (9, 2, 32, 32, 1280, 320, 32, 9), (9, 2, 16, 16, 1280, 1280, 64, 9), (9, 4, 19, 22, 896, 64, 64, 9),
    (1, 64, 1, 1, 5120, 2048, 32, 16), (1, 16, 1, 1, 5120, 5120, 32, 8), (1, 64, 1, 1, 5120, 640, 512, 2),
    (1, 300, 1, 1, 512, 2560, 128, 2), (1, 1100, 1, 1, 512, 1280, 256, 1), (1, 260, 1, 1, 1280, 2560, 256, 1),
    (1, 64, 1, 1, 768, 640, 256, 1), (1, 700, 1, 1, 1024, 1280, 128, 4), (1, 1817, 1, 1, 512, 3264, 128, 1), (9, 1, 61, 40, 64, 512, 64, 3),
    (9, 3, 18, 18, 640, 640, 128, 9), (9, 3, 20, 19, 128, 544, 128, 9), (9, 1, 30, 41, 384, 640, 64, 9),
    (1, 2699, 1, 1, 384, 384, 128, 1), (1, 700, 1, 1, 1280, 1280, 256, 1), (1, 100, 1, 1, 1024, 480, 256, 1),
], ids=lambda c: "t%d_%dx%dx%d_%d-%d_g%d_%d" % c)
def test_error_of_the_sums_over_groups(wq, case):
    """Distance from the fp64 sum of the same codes and scales, against what `chains` fp32 chains of
    groups, added up one after the other, are away from it.  A rounding of a sum is off by
    u = 2^-23 sqrt(3 / (8 ln 2) / 12) of it in the root mean square (uniform over half an ulp, mantissas
    log-uniform); with terms of random sign a sum's square grows by one term's per group, so the G
    products of two scales, the sums inside c chains and the sums of chains make
    u^2 (1 + (G / c + 1) / 2 + (c + 1) / 2 - 1 / c) relative to the result.  (6 % for the formula.)"""
    taps, N, H, W, Cin, Cout, g, chains = case
    y, ref = forward_and_fp64_reference(wq, *case[:7])
    groups = Cin // g
    err = float((y - ref).norm() / ref.norm())
    G = taps * groups
    bound = 2.0 ** -23 * np.sqrt(3 / (8 * np.log(2)) / 12 * (2 + G / (2 * chains) + chains / 2 - 1 / chains))
    print(f"error {err:.3e}, {chains} chains of fp32 {bound:.3e}")
    assert err <= 1.06 * bound


@pytest.mark.parametrize("tile", [
    # N  H   W   Cout  wave tile       (pixels and channels that end inside it, rows that do not match it)
    ((1, 9, 7, 33), (16, 16)), ((4, 21, 25, 57), (16, 64)), ((2, 22, 25, 130), (32, 64)), ((3, 67, 69, 130), (64, 64)),
], ids=lambda t: "%dx%d" % t[1])
@pytest.mark.parametrize("taps", [1, 9])
@pytest.mark.parametrize("bits", [8, 4], ids=["w8", "w4"])
@pytest.mark.parametrize("g", [32, 64, 128])
def test_every_instance_of_the_quantized_gemm(wq, g, bits, taps, tile):
    """K-step and group class x width of the weight codes x 3x3 or linear x wave tile, each as the plan's own
    choice."""
    (N, H, W, Cout), (channels, pixels) = tile
    groups = 2 if taps == 9 else 4
    plan = wq.DirectPlan(N, H, W, groups * g, Cout, g, linear=taps == 1, weight_bits=bits)
    assert plan.launch[:2] == (channels, pixels)
    y, ref = forward_and_fp64_reference(wq, taps, N, H, W, groups * g, Cout, g, bits)
    assert bool(torch.isfinite(y).all())
    assert float((y - ref).abs().max()) <= Y_TOL * float(ref.abs().max())


@pytest.mark.parametrize("bits", [8, 4], ids=["w8", "w4"])
@pytest.mark.parametrize("case", [
    # taps N  H   W   Cin  Cout  g   (channels, pixels, waves)
    (1, 20, 1, 1, 1280, 500, 64, (16, 16, 8)), (1, 100, 1, 1, 768, 100, 256, (16, 16, 3)),
    (1, 2100, 1, 1, 1280, 57, 64, (16, 64, 8)), (9, 2, 12, 13, 448, 250, 64, (16, 16, 4)),
    (9, 3, 23, 24, 128, 330, 64, (32, 64, 4)), (9, 1, 30, 41, 448, 500, 64, (32, 64, 8)),
    (9, 3, 31, 33, 64, 500, 64, (32, 64, 4)), (9, 3, 45, 46, 64, 330, 64, (32, 64, 2)),
    (9, 4, 63, 65, 64, 300, 64, (64, 64, 4)), (9, 3, 67, 69, 64, 450, 64, (64, 64, 2)),
    (9, 5, 67, 69, 64, 600, 64, (64, 64, 1)), (1, 3300, 1, 1, 640, 130, 64, (64, 64, 4)),
    (1, 2700, 1, 1, 384, 290, 64, (32, 64, 2)), (1, 4000, 1, 1, 320, 700, 64, (64, 64, 2)),
    (1, 4000, 1, 1, 320, 1250, 64, (32, 64, 1)), (1, 6000, 1, 1, 320, 1250, 64, (64, 64, 1)),
    (1, 2700, 1, 1, 192, 290, 64, (16, 64, 1)), (1, 12500, 1, 1, 640, 1030, 64, (64, 64, 1)),
], ids=lambda c: "t%d_%dx%dx%d_%d-%d_g%d_%s" % (c[:7] + ("x".join(map(str, c[7])),)))
def test_every_slice_count_the_plan_picks(wq, case, bits):
    """The waves that share a tile's reduction, as chosen for the shape, with ragged pixels and channels."""
    y, ref = forward_and_fp64_reference(wq, *case[:7], bits=bits, launch=case[7])
    assert bool(torch.isfinite(y).all())
    assert float((y - ref).abs().max()) <= Y_TOL * float(ref.abs().max())
