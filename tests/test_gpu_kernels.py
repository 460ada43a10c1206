"""Per-kernel parity on a real MI355X: each gfx950 kernel, called through the C ABI, against the
fp64 oracle on identical seeded fp32 inputs.  Integer outputs (sign masks, pool indices) are
bit-exact; floating point is compared normwise per tensor (activations 1e-4, gradients 1e-3)."""
import numpy as np
import pytest

from oracle import numerics as nm
from workloads import tensors as wt
import paper_2010_14501_amd as M
from paper_2010_14501_amd import monet

pytestmark = pytest.mark.gpu

from parity_util import ACT_TOL, GRAD_TOL, rel, check_close


def torch_mod():
    import torch
    return torch


def dev(a):
    torch = torch_mod()
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


CONV_CASES = [
    # N, H, W, C, K, R, stride, pad
    (2, 16, 16, 16, 16, 3, 1, 1),       # the tiny chain's layer
    (3, 14, 14, 64, 128, 3, 1, 1),      # several tiles, ragged M (588 rows)
    (2, 15, 13, 32, 80, 3, 2, 1),       # stride 2, odd sizes, ragged K
    (2, 28, 28, 64, 256, 1, 1, 0),      # 1x1
    (2, 28, 28, 128, 64, 1, 2, 0),      # 1x1 stride 2 (downsample path)
    (2, 32, 32, 3, 64, 7, 2, 3),        # stem: C=3 takes the scalar-load path
    (1, 9, 9, 20, 24, 3, 1, 1),         # C % 16 != 0 and K % 16 != 0
    (5, 7, 7, 512, 512, 3, 1, 1),       # deep reduction (4608)
    (2, 14, 14, 160, 320, 3, 1, 1),     # an inception 3x3: channel counts that are multiples of 16 but not of 128
    (2, 28, 28, 24, 144, 1, 1, 0),      # 1x1 with 24 input channels: aligned forward loader, last reduction step half empty
    (2, 28, 28, 144, 24, 1, 1, 0),      # ... and 24 output channels: the same in the input gradient
    (3, 15, 13, 40, 36, 1, 2, 0),       # both at once, stride 2, ragged rows and columns
    (2, 9, 9, 4, 8, 1, 1, 0),           # a single, mostly empty step
    # reduction steps that straddle filter taps (channels a multiple of 4, not of 16)
    (2, 14, 14, 24, 64, 5, 1, 2),       # an inception 5x5
    (3, 13, 17, 60, 92, 3, 1, 1),       # both directions, last step partly empty
    (2, 9, 11, 4, 8, 3, 1, 1),          # four taps to a step
    (2, 10, 9, 36, 28, 3, 2, 1),        # stride 2: input-gradient classes with one, two and four taps
    (5, 6, 7, 132, 44, 2, 2, 0),        # even filter, no padding
]


@pytest.mark.parametrize("case", CONV_CASES)
def test_conv_trio_matches_oracle(case):
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (rng.standard_normal((K, R, R, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (C * R * R))))
    P = (H + 2 * pad - R) // stride + 1
    Q = (W + 2 * pad - R) // stride + 1
    dy = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    xo, wo, dyo = wt.act_to_oracle(x), wt.weight_to_oracle(w), wt.act_to_oracle(dy)
    dx, dwt, ddy = dev(x), dev(w), dev(dy)
    # forward
    y = torch.empty((N, P, Q, K), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1, None, 0)
    want = wt.act_from_oracle(nm.conv2d_fwd(xo, wo, stride, pad))
    check_close(y.cpu().numpy(), want, ACT_TOL)
    need = max(monet.call("monet_conv_workspace_bytes", which, N, H, W, C, K, R, R, stride, pad, 5) for which in (0, 1))
    big = torch.empty(need // 4, dtype=torch.float32, device="cuda")     # split workspace
    for splits in (2, 5):
        y.fill_(float("nan"))
        monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, R, R, stride, pad,
                   splits, big.data_ptr(), big.numel() * 4)
        check_close(y.cpu().numpy(), want, ACT_TOL, what=splits)
    # input gradient, plain and accumulating
    gx = torch.full((N, H, W, C), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_dgrad", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, R, R, stride, pad, 0, 1, None, 0)
    want = wt.act_from_oracle(nm.conv2d_dgrad(dyo, wo, xo.shape, stride, pad))
    check_close(gx.cpu().numpy(), want, GRAD_TOL)
    monet.call("monet_conv_dgrad", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1, 1, None, 0)
    check_close(gx.cpu().numpy(), 2 * want, GRAD_TOL)
    for splits in (2, 5):
        gx.fill_(float("nan"))
        monet.call("monet_conv_dgrad", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, R, R, stride, pad, 0,
                   splits, big.data_ptr(), big.numel() * 4)
        check_close(gx.cpu().numpy(), want, GRAD_TOL, what=splits)
        monet.call("monet_conv_dgrad", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1,
                   splits, big.data_ptr(), big.numel() * 4)
        check_close(gx.cpu().numpy(), 2 * want, GRAD_TOL, what=splits)
    # weight gradient: no workspace, and split with workspace
    want = wt.weight_from_oracle(nm.conv2d_wgrad(xo, dyo, R, R, stride, pad))
    for splits in (1, 3, 8):
        gw = torch.full((K, R, R, C), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.empty(splits * K * R * R * C, dtype=torch.float32, device="cuda")
        monet.call("monet_conv_wgrad", None, dx.data_ptr(), ddy.data_ptr(), gw.data_ptr(), N, H, W, C, K, R, R, stride, pad,
                   splits, ws.data_ptr(), ws.numel() * 4)
        check_close(gw.cpu().numpy(), want, GRAD_TOL, what=splits)


@pytest.mark.parametrize("case", [
    # N, H, W, C, K, R, stride, pad: element-wise loaders; results stored element by element (C no multiple of 4: four rows of a residue class
    # in one go, across ends of rows and images) or in 16-byte pieces (C a multiple of 4)
    (5, 3, 2, 7, 5, 3, 2, 1), (9, 5, 1, 6, 9, 1, 2, 0), (7, 2, 3, 11, 3, 2, 3, 1), (40, 4, 5, 3, 2, 1, 4, 0), (3, 9, 7, 130, 6, 3, 2, 1),
    (5, 3, 2, 8, 5, 3, 2, 1), (3, 13, 9, 64, 2, 1, 1, 0), (2, 13, 9, 132, 3, 3, 2, 1), (2, 11, 9, 416, 1, 3, 1, 0), (2, 9, 9, 145, 17, 2, 3, 0),
])
def test_input_gradient_on_element_wise_loaders(case):
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad = case
    rng = np.random.default_rng(31)
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    w = rng.standard_normal((K, R, R, C), dtype=np.float32)
    dy = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    want = wt.act_from_oracle(nm.conv2d_dgrad(wt.act_to_oracle(dy), wt.weight_to_oracle(w), (N, C, H, W), stride, pad))
    gd, gw = dev(dy), dev(w)
    guard = 64
    for acc in (0, 1):
        flat = torch.full((N * H * W * C + 2 * guard,), -7.0, device="cuda")
        dx = flat[guard:guard + N * H * W * C].view(N, H, W, C)
        dx.copy_(dev(x))
        monet.call("monet_conv_dgrad", None, gd.data_ptr(), gw.data_ptr(), dx.data_ptr(), N, H, W, C, K, R, R, stride, pad, acc, 1, None, 0)
        # fp32 sums of at most 54 products and the accumulated value: 1e-6 in the norm
        check_close(dx.cpu().numpy(), want + x.astype(np.float64) * acc, 1e-6, what=acc)
        assert (flat[:guard] == -7.0).all() and (flat[guard + N * H * W * C:] == -7.0).all()


@pytest.mark.parametrize("tile", range(6))
@pytest.mark.parametrize("case", [(3, 15, 14, 48, 112, 3, 1, 1), (2, 11, 13, 20, 76, 3, 2, 1), (2, 9, 8, 30, 70, 3, 1, 1), (2, 20, 18, 132, 72, 1, 1, 0)])
def test_conv_trio_on_every_tile_shape(case, tile):
    """Each of the shape numbers that can be forced (128x128, 128x64, 64x128, 64x64 and those that stand for another), with rows and columns beyond a tile's edge, aligned, straddling and element-wise loaders,
    whole and in ranges, forward and both gradients, plain and accumulating."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad = case
    rng = np.random.default_rng(11)
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = rng.standard_normal((K, R, R, C), dtype=np.float32)
    dy = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    xo, wo, dyo = wt.act_to_oracle(x), wt.weight_to_oracle(w), wt.act_to_oracle(dy)
    want_y = wt.act_from_oracle(nm.conv2d_fwd(xo, wo, stride, pad))
    want_dx = wt.act_from_oracle(nm.conv2d_dgrad(dyo, wo, xo.shape, stride, pad))
    want_dw = wt.weight_from_oracle(nm.conv2d_wgrad(xo, dyo, R, R, stride, pad))
    gx, gw, gd = dev(x), dev(w), dev(dy)
    ws = torch.empty(3 * max(x.size, dy.size, w.size), device="cuda")
    dims = (N, H, W, C, K, R, R, stride, pad)
    lib = monet.load_library()
    lib.monet_conv_force_tile(tile)
    try:
        for splits in (1, 3):
            y, dx, dw = (torch.full(a.shape, float("nan"), device="cuda") for a in (dy, x, w))
            wsp, wsb = (ws.data_ptr(), ws.numel() * 4) if splits > 1 else (None, 0)
            monet.call("monet_conv_fwd", None, gx.data_ptr(), gw.data_ptr(), y.data_ptr(), *dims, splits, wsp, wsb)
            monet.call("monet_conv_dgrad", None, gd.data_ptr(), gw.data_ptr(), dx.data_ptr(), *dims, 0, splits, wsp, wsb)
            monet.call("monet_conv_dgrad", None, gd.data_ptr(), gw.data_ptr(), dx.data_ptr(), *dims, 1, splits, wsp, wsb)
            monet.call("monet_conv_wgrad", None, gx.data_ptr(), gd.data_ptr(), dw.data_ptr(), *dims, splits, wsp, wsb)
            # fp32 sums of at most 1008 products: 1e-6 in the norm
            check_close(y.cpu().numpy(), want_y, 1e-6, what=splits)
            check_close(dx.cpu().numpy(), 2 * want_dx, 1e-6, what=splits)
            check_close(dw.cpu().numpy(), want_dw, 1e-6, what=splits)
    finally:
        lib.monet_conv_force_tile(-1)


SPECIAL_CASES = [
    # N, H, W, C, K: 1x1 layers (no padding: a padded zero times an infinity is a NaN in any implementation that stages zeros)
    (1, 16, 16, 36, 40),        # aligned loaders, last reduction step partly empty
    (2, 12, 12, 64, 128),       # two tiles of rows, only one of which holds special values
    (1, 9, 9, 30, 17),          # element-wise loaders
]


@pytest.mark.parametrize("case", SPECIAL_CASES)
@pytest.mark.parametrize("kind", ["inf", "nan", "inf_times_zero", "inf_times_subnormal", "both_inf", "near_max", "overflow", "tiny"])
def test_conv_of_infinities_nans_and_extreme_values(case, kind):
    """The matrix products are worked in three bf16 pieces per float: infinities, NaNs, values that round to infinity in bf16 and
    products that overflow have to come out as the fp32 product's, with the finite results beside them as close as ever.
    Reference: the same sums in fp64, rounded to fp32."""
    torch = torch_mod()
    N, H, W, C, K = case
    rng = np.random.default_rng(5)
    x = (rng.standard_normal((N, H, W, C)) + 3.0).astype(np.float32)
    w = (np.abs(rng.standard_normal((K, 1, 1, C))) + 0.5).astype(np.float32)
    dy = (rng.standard_normal((N, H, W, K)) + 2.0).astype(np.float32)
    inf = np.float32(np.inf)
    if kind == "inf":
        x[0, 1, 2, 3], x[0, 3, 3, 7], dy[0, 2, 2, 5], w[4, 0, 0, 6] = inf, -inf, -inf, inf
    elif kind == "nan":
        x[0, 1, 2, 3], dy[0, 2, 2, 5] = np.nan, np.nan
    elif kind == "inf_times_zero":
        x[0, 1, 2, 3], w[2, 0, 0, 3], w[3, 0, 0, 3], dy[0, 1, 2, 9] = inf, 0.0, -0.0, 0.0
    elif kind == "inf_times_subnormal":      # 1e-41 is below bf16's smallest number
        x[0, 1, 2, 3], w[2, 0, 0, 3], w[3, 0, 0, 3], dy[0, 1, 2, 9] = inf, 1e-41, -1e-41, 1e-41
    elif kind == "both_inf":
        x[0, 1, 2, 3], w[2, 0, 0, 3], w[3, 0, 0, 3], dy[0, 1, 2, 9] = inf, inf, -inf, -inf
    elif kind == "near_max":      # 3.4e38 rounds to infinity in bf16
        x[0, 1, 2, 3], w[:, 0, 0, 3], dy[0, 1, 2, 9] = 3.4e38, 1e-3, 1e-4
    elif kind == "overflow":
        x[0, 1, 2, 3], w[2, 0, 0, 3], w[3, 0, 0, 3], dy[0, 1, 2, 9] = 1.7e38, 1.3e38, -1.9e30, 1.1e33
    else:
        x[0, 1, 2, 3], w[2, 0, 0, 3] = 1e-40, 1e-39
    with np.errstate(all="ignore"):
        x2, w2, g2 = x.reshape(-1, C).astype(np.float64), w.reshape(K, C).astype(np.float64), dy.reshape(-1, K).astype(np.float64)

        def product(a, b):      # a[m, r] b[r, n] in fp32 semantics (every product and the sum rounded to fp32's range) and sum |a b|
            p = (a[:, :, None] * b[None, :, :]).astype(np.float32).astype(np.float64)
            return p.sum(1).astype(np.float32), np.abs(p).sum(1)

        def rows(a, b):
            parts = [product(a[i:i + 8], b) for i in range(0, len(a), 8)]
            return tuple(np.concatenate([q[j] for q in parts]) for j in (0, 1))
        want = dict(y=rows(x2, w2.T), dx=rows(g2, w2), dw=rows(g2.T, x2))
    gx, gw, gd = dev(x), dev(w), dev(dy)
    got = dict(y=torch.empty(N * H * W, K, device="cuda"), dx=torch.empty(N * H * W, C, device="cuda"), dw=torch.empty(K, C, device="cuda"))
    dims = (N, H, W, C, K, 1, 1, 1, 0)
    ws = torch.empty(3 * max(t.numel() for t in got.values()), device="cuda")
    for splits in (1, 3):
        wsp = (ws.data_ptr(), ws.numel() * 4)
        monet.call("monet_conv_fwd", None, gx.data_ptr(), gw.data_ptr(), got["y"].data_ptr(), *dims, splits, *wsp)
        monet.call("monet_conv_dgrad", None, gd.data_ptr(), gw.data_ptr(), got["dx"].data_ptr(), *dims, 0, splits, *wsp)
        monet.call("monet_conv_wgrad", None, gx.data_ptr(), gd.data_ptr(), got["dw"].data_ptr(), *dims, splits, *wsp)
        for name, t in got.items():
            a, (b, mag) = t.cpu().numpy(), want[name]
            assert np.array_equal(np.isnan(a), np.isnan(b)), (name, splits)
            assert np.array_equal(np.isinf(a), np.isinf(b)) and np.array_equal(a[np.isinf(b)], b[np.isinf(b)]), (name, splits)
            fine = np.isfinite(b)
            err = np.abs(a[fine].astype(np.float64) - b[fine]) / mag[fine]
            # sums of n products, n additions rounded to 2^-24 each and the terms the pieces leave out (2^-24): at worst
            # (n + 1) 2^-24 of sum |a b| apiece, and over many results, whose roundings do not add up, sqrt(n) 2^-24 in the norm
            n = dict(y=C, dx=K, dw=N * H * W)[name]
            assert err.max() <= (n + 1) * 2.0 ** -24, (name, splits, err.max() * 2.0 ** 24)
            assert np.sqrt((err ** 2).mean()) <= np.sqrt(n) * 2.0 ** -24, (name, splits, np.sqrt((err ** 2).mean()) * 2.0 ** 24)


def test_conv_of_one_infinity_leaves_its_neighbours_precise():
    """Four products per result, every operand 1 + 2^-7 - 2^-23 (the largest rest that eight bits can leave), one infinity in each
    activation: the finite results of the same tile are as close as fp32 sums are, 4 * 2^-24."""
    torch = torch_mod()
    N, H, W, C, K = 1, 2, 2, 4, 4
    v = np.float32(1 + 2.0 ** -7 - 2.0 ** -23)
    x, w, dy = (np.full(s, v, np.float32) for s in ((4, C), (K, C), (4, K)))
    x[0, 0], dy[0, 0] = np.inf, np.inf
    gx, gw, gd = dev(x), dev(w), dev(dy)
    y, dx, dw = (torch.empty(4, 4, device="cuda") for _ in range(3))
    dims = (N, H, W, C, K, 1, 1, 1, 0)
    monet.call("monet_conv_fwd", None, gx.data_ptr(), gw.data_ptr(), y.data_ptr(), *dims, 1, None, 0)
    monet.call("monet_conv_dgrad", None, gd.data_ptr(), gw.data_ptr(), dx.data_ptr(), *dims, 0, 1, None, 0)
    monet.call("monet_conv_wgrad", None, gx.data_ptr(), gd.data_ptr(), dw.data_ptr(), *dims, 1, None, 0)
    want = 4 * np.float64(v) ** 2
    for got, rows in ((y, 1), (dx, 1)):
        got = got.cpu().numpy()
        assert np.all(np.isposinf(got[:rows])) and np.all(np.abs(got[rows:] - want) <= 4 * 2.0 ** -24 * want), (got[1, 1] / want - 1) * 2.0 ** 24
    got = dw.cpu().numpy()
    assert np.all(np.isposinf(got[0])) and np.all(np.isposinf(got[:, 0]))
    assert np.all(np.abs(got[1:, 1:] - want) <= 4 * 2.0 ** -24 * want), (got[1, 1] / want - 1) * 2.0 ** 24


# every way a reduction is walked: aligned, partly empty last step, straddling filter taps, strided residue classes, element-wise
WALK_CASES = [
    # N, H, W, C, K, R, stride, pad
    (2, 13, 11, 64, 96, 1, 1, 0),
    (2, 13, 11, 36, 44, 1, 1, 0),
    (2, 13, 11, 32, 48, 3, 1, 1),
    (2, 13, 11, 36, 28, 3, 1, 1),
    (2, 14, 11, 20, 32, 3, 2, 1),
    (1, 13, 11, 27, 33, 3, 1, 1),
    (2, 12, 12, 512, 32, 1, 1, 0),
]


@pytest.mark.parametrize("case", WALK_CASES)
@pytest.mark.parametrize("splits", [1, 3])
def test_conv_of_infinities_on_every_loader_and_in_ranges(case, splits):
    """An infinity in the first and in the last reduction indices (whole reductions and ranges that start in the middle): the
    results that it meets are infinite with its sign, the others are as precise as without it."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad = case
    rng = np.random.default_rng(17)
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (np.abs(rng.standard_normal((K, R, R, C))) + 0.1).astype(np.float32)
    dy = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    dpos = (np.abs(dy) + 0.1).astype(np.float32)
    xi, dyi = x.copy(), dy.copy()
    xi[0, 2, 3, 1], xi[N - 1, H - 2, W - 2, C - 2] = np.inf, -np.inf
    dyi[0, 1, 1, 0], dyi[N - 1, P - 2, Q - 2, K - 1] = -np.inf, np.inf
    wo = wt.weight_to_oracle(w)
    with np.errstate(all="ignore"):
        want_y = wt.act_from_oracle(nm.conv2d_fwd(wt.act_to_oracle(xi), wo, stride, pad))
        want_dx = wt.act_from_oracle(nm.conv2d_dgrad(wt.act_to_oracle(dyi), wo, (N, C, H, W), stride, pad))
        want_dw = wt.weight_from_oracle(nm.conv2d_wgrad(wt.act_to_oracle(xi), wt.act_to_oracle(dpos), R, R, stride, pad))
    gx, gw, gd, gp = dev(xi), dev(w), dev(dyi), dev(dpos)
    y, dx, dw = (torch.full(a.shape, float("nan"), device="cuda") for a in (want_y, want_dx, want_dw))
    ws = torch.empty(3 * max(want_y.size, want_dx.size, want_dw.size), device="cuda")
    dims = (N, H, W, C, K, R, R, stride, pad)
    wsp = (ws.data_ptr(), ws.numel() * 4)
    monet.call("monet_conv_fwd", None, gx.data_ptr(), gw.data_ptr(), y.data_ptr(), *dims, splits, *wsp)
    monet.call("monet_conv_dgrad", None, gd.data_ptr(), gw.data_ptr(), dx.data_ptr(), *dims, 0, splits, *wsp)
    monet.call("monet_conv_wgrad", None, gx.data_ptr(), gp.data_ptr(), dw.data_ptr(), *dims, splits, *wsp)
    for name, t, b in (("y", y, want_y), ("dx", dx, want_dx), ("dw", dw, want_dw)):
        a = t.cpu().numpy()
        assert np.isinf(b).any() and np.isfinite(b).any(), name
        assert np.array_equal(np.isnan(a), np.isnan(b)), name
        assert np.array_equal(a[np.isinf(b)], b[np.isinf(b)]) and np.array_equal(np.isinf(a), np.isinf(b)), name
        fine = np.isfinite(b)
        check_close(a[fine], b[fine], 1e-6, what=name)      # fp32 sums of at most 512 products: 1e-6 in the norm


@pytest.mark.parametrize("case", WALK_CASES)
@pytest.mark.parametrize("exponent,other", [(-100, 60), (-112, 60), (-118, 60), (-125, 60), (-62, -62)])
def test_conv_of_operands_at_the_bottom_of_the_range(case, exponent, other):
    """One operand of about 2^exponent (at -125 one element in three is subnormal), the other of 2^60: the result is an ordinary
    number and as precise as for operands of about 1, whole and in ranges, on every loader.  Likewise where the terms of a
    product, not the operands, reach the bottom of the range (2^-62 each)."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad = case
    rng = np.random.default_rng(23)
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    small, big = np.float64(2.0 ** exponent), np.float64(2.0 ** other)

    def of_size(scale, shape):      # (fp32 tensor, the same values over the scale in 64 bits)
        t = (rng.standard_normal(shape) * scale).astype(np.float32)
        return t, t.astype(np.float64) / scale
    (x, xn), (dy, dyn) = of_size(small, (N, H, W, C)), of_size(small, (N, P, Q, K))
    (w, wn), (z, zn) = of_size(big, (K, R, R, C)), of_size(big, (N, P, Q, K))
    unit = small * big
    want = dict(y=wt.act_from_oracle(nm.conv2d_fwd(wt.act_to_oracle(xn), wt.weight_to_oracle(wn), stride, pad)),
                dx=wt.act_from_oracle(nm.conv2d_dgrad(wt.act_to_oracle(dyn), wt.weight_to_oracle(wn), (N, C, H, W), stride, pad)),
                dw=wt.weight_from_oracle(nm.conv2d_wgrad(wt.act_to_oracle(xn), wt.act_to_oracle(zn), R, R, stride, pad)))
    gx, gw, gd, gz = dev(x), dev(w), dev(dy), dev(z)
    ws = torch.empty(3 * max(a.size for a in want.values()), device="cuda")
    dims = (N, H, W, C, K, R, R, stride, pad)
    wsp = (ws.data_ptr(), ws.numel() * 4)
    for splits in (1, 3):
        got = {k: torch.full(a.shape, float("nan"), device="cuda") for k, a in want.items()}
        monet.call("monet_conv_fwd", None, gx.data_ptr(), gw.data_ptr(), got["y"].data_ptr(), *dims, splits, *wsp)
        monet.call("monet_conv_dgrad", None, gd.data_ptr(), gw.data_ptr(), got["dx"].data_ptr(), *dims, 0, splits, *wsp)
        monet.call("monet_conv_wgrad", None, gx.data_ptr(), gz.data_ptr(), got["dw"].data_ptr(), *dims, splits, *wsp)
        for name, b in want.items():
            # fp32 sums of at most 512 products: 1e-6 in the norm, as for operands of any other size
            check_close(got[name].cpu().numpy().astype(np.float64) / unit, b, 1e-6, what=(name, splits))


def test_conv_of_one_product_is_the_rounded_product():
    """1x1 layers with a single input channel (forward) and a single output channel (input gradient): nothing is summed, so the
    result is the fp32 product itself."""
    torch = torch_mod()
    rng = np.random.default_rng(29)
    a = rng.standard_normal((3, 9, 11, 1), dtype=np.float32)
    b = rng.standard_normal((1, 20), dtype=np.float32)
    ga, gb, y = dev(a), dev(b), torch.empty(3, 9, 11, 20, device="cuda")
    monet.call("monet_conv_fwd", None, ga.data_ptr(), gb.data_ptr(), y.data_ptr(), 3, 9, 11, 1, 20, 1, 1, 1, 0, 1, None, 0)
    assert np.array_equal(y.cpu().numpy(), a * b[0])
    y.fill_(float("nan"))
    monet.call("monet_conv_dgrad", None, ga.data_ptr(), gb.data_ptr(), y.data_ptr(), 3, 9, 11, 20, 1, 1, 1, 1, 0, 0, 1, None, 0)
    assert np.array_equal(y.cpu().numpy(), a * b[0])


def test_conv_of_few_tiles_uses_the_workspace_it_is_given():
    """splits == 1 and a workspace: a launch of few tiles cuts its reduction by itself, as many ranges as the workspace holds and
    at least eight steps each, with the bits of the call that asks for as many; one that holds a single result changes nothing."""
    torch = torch_mod()
    for N, H, W, C, K, R, ranges in ((1, 7, 7, 512, 512, 3, 16), (2, 9, 9, 48, 64, 3, 3), (6, 28, 28, 256, 130, 1, 2)):
        rng = np.random.default_rng(37)
        x, dy = rng.standard_normal((N, H, W, C), dtype=np.float32), rng.standard_normal((N, H, W, K), dtype=np.float32)
        w = rng.standard_normal((K, R, R, C), dtype=np.float32)
        gx, gw, gd = dev(x), dev(w), dev(dy)
        for name, src, out, adj in (("monet_conv_fwd", gx, K, ()), ("monet_conv_dgrad", gd, C, (1,))):
            n = N * H * W * out
            dims = (N, H, W, C, K, R, R, 1, R // 2) + adj
            red = R * R * (C if out == K else K)
            most = max(1, min(ranges, -(-red // 16) // 8, 256 // (-(-N * H * W // 128) * -(-out // 128))))
            ws = torch.empty(ranges * n, device="cuda")

            def go(splits, floats):
                ws.fill_(float("nan"))
                y = torch.full((N, H, W, out), 1.0, device="cuda")
                monet.call(name, None, src.data_ptr(), gw.data_ptr(), y.data_ptr(), *dims, splits, ws.data_ptr() if floats else None, floats * 4)
                return y, int((~torch.isnan(ws)).sum()) // n
            y, used = go(1, ranges * n)
            assert used == (most if most > 1 else 0), (name, used, most)
            assert torch.equal(y, go(most, ranges * n)[0]), (name, "as many ranges, asked for")
            y, used = go(1, 2 * n - 1)
            assert used == 0 and torch.equal(y, go(1, 0)[0]), (name, "room for one result")


def test_conv_of_a_ragged_last_round_leaves_its_workspace_alone():
    """More than 256 tiles and not a multiple of it, with the workspace that earlier kernels cut the tiles of the last round with.
    Several calls in a row, forward and input gradient with accumulation, against the oracle and against the call
    without a workspace."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad = 48, 28, 28, 128, 128, 1, 1, 0          # 37632 rows = 294 tiles of 128
    rng = np.random.default_rng(7)
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (rng.standard_normal((K, R, R, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / C)))
    dy = rng.standard_normal((N, H, W, K), dtype=np.float32)
    xo, wo, dyo = wt.act_to_oracle(x), wt.weight_to_oracle(w), wt.act_to_oracle(dy)
    dx, dwt, ddy = dev(x), dev(w), dev(dy)
    need = [monet.call("monet_conv_workspace_bytes", which, N, H, W, C, K, R, R, stride, pad, 1) for which in (0, 1)]
    assert need[0] == need[1] == 2 * 38 * 128 * 128 * 4                      # 38 tiles beyond 256, in two ranges
    ws = torch.full((need[0] // 4,), float("nan"), dtype=torch.float32, device="cuda")
    want_y = wt.act_from_oracle(nm.conv2d_fwd(xo, wo, stride, pad))
    want_dx = wt.act_from_oracle(nm.conv2d_dgrad(dyo, wo, xo.shape, stride, pad))
    y0 = torch.empty((N, H, W, K), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y0.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1, None, 0)
    # a refused call (workspace announced smaller than two partial results) enqueues nothing; monet_conv_reset_arrivals, kept
    # for earlier callers, changes nothing
    with pytest.raises(monet.MonetError):
        monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y0.data_ptr(), N, H, W, C, K, R, R, stride, pad, 2, ws.data_ptr(), 1024)
    for rep in range(3):
        if rep == 1:
            monet.call("monet_conv_reset_arrivals", None)
        y = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1, ws.data_ptr(), need[0])
        check_close(y.cpu().numpy(), want_y, ACT_TOL, what=rep)
        assert torch.equal(y, y0) and torch.isnan(ws).all()
        gx = torch.full((N, H, W, C), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_conv_dgrad", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, R, R, stride, pad, 0, 1, ws.data_ptr(), need[1])
        check_close(gx.cpu().numpy(), want_dx, GRAD_TOL, what=rep)
        monet.call("monet_conv_dgrad", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1, 1, ws.data_ptr(), need[1])
        check_close(gx.cpu().numpy(), 2 * want_dx, GRAD_TOL, what=rep)


@pytest.mark.parametrize("case", [
    (3, 14, 14, 64, 128, 3, 1, 1),      # ragged last row group (588 rows)
    (2, 28, 28, 64, 256, 1, 1, 0),      # two column tiles
    (2, 15, 13, 32, 80, 3, 2, 1),       # stride 2, a column tile that is only partly used (80 of 128)
    (2, 28, 28, 128, 64, 1, 2, 0),      # 64 columns
    (48, 28, 28, 128, 128, 1, 1, 0),    # more tiles than CUs, and no multiple of them
    (2, 28, 28, 24, 144, 1, 1, 0),      # 1x1 with 24 input channels (last reduction step half empty)
    (3, 15, 13, 40, 36, 1, 2, 0),
])
@pytest.mark.parametrize("room", [True, False])
def test_statistics_from_the_conv_epilogue_are_the_stand_alone_bits(case, room):
    """BatchNorm's forward statistics come out of the convolution's epilogue with the same bits as from a pass
    over the convolution's output, and match the oracle; likewise behind a reduction cut into ranges (few tiles and a workspace)."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (rng.standard_normal((K, R, R, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (C * R * R))))
    w += np.float32(0.05)                                                # non-zero channel means
    P = (H + 2 * pad - R) // stride + 1
    Q = (W + 2 * pad - R) // stride + 1
    dx, dwt = dev(x), dev(w)
    rows = N * P * Q
    groups = (rows + 63) // 64
    sb = 8 * (groups + (groups + 63) // 64) * K                      # first and second level of the statistics
    scratch = torch.full((sb // 4,), float("nan"), dtype=torch.float32, device="cuda")
    need = monet.call("monet_conv_workspace_bytes", 0, N, H, W, C, K, R, R, stride, pad, 1) if room else 0
    ws = torch.empty(max(need // 4, 1), dtype=torch.float32, device="cuda")
    y = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
    fused = torch.full((2 * K,), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_fwd_bn_stats", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, R, R, stride, pad,
               ws.data_ptr() if need else None, need, fused.data_ptr(), 1e-5, scratch.data_ptr(), sb)
    y2 = torch.empty_like(y)
    monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y2.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1,
               ws.data_ptr() if need else None, need)
    assert torch.equal(y, y2)
    alone = torch.full((2 * K,), float("nan"), dtype=torch.float32, device="cuda")
    scratch.fill_(float("nan"))
    monet.call("monet_bn_stats", None, y2.data_ptr(), alone.data_ptr(), rows, K, 1e-5, scratch.data_ptr(), sb)
    assert torch.equal(fused, alone)
    mean, invstd = nm.bn_stats(wt.act_to_oracle(y2.cpu().numpy()), 1e-5)
    got = fused.cpu().numpy()
    check_close(got[:K], mean, ACT_TOL)
    check_close(got[K:], invstd, ACT_TOL)


@pytest.mark.parametrize("case", [
    (3, 14, 14, 64, 128, 3, 1, 1, 0),      # implicit GEMM, ragged rows
    (2, 28, 28, 64, 256, 1, 1, 0, 0),      # two column tiles
    (2, 15, 13, 32, 80, 3, 2, 1, 0),       # stride 2, a column tile that is only partly used
    (2, 28, 28, 128, 64, 1, 2, 0, 0),      # 64 columns
    (48, 28, 28, 128, 128, 1, 1, 0, 0),    # more tiles than CUs, and no multiple of them
    (2, 28, 28, 24, 128, 1, 1, 0, 0),      # 1x1 with 24 input channels (last reduction step half empty)
    (3, 14, 14, 64, 128, 3, 1, 1, 2),      # Winograd, 2x2 output tiles
    (3, 14, 14, 64, 128, 3, 1, 1, 4),      # Winograd, 4x4 output tiles (last tile row / column partly outside)
    (2, 9, 7, 32, 48, 3, 1, 1, 4),
])
@pytest.mark.parametrize("room", [True, False])
def test_batchnorm_apply_in_the_conv_epilogue_is_the_stand_alone_bits(case, room):
    """A recomputed convolution that applies the BatchNorm behind it in its epilogue writes exactly what the
    convolution followed by the in-place apply kernel writes (implicit GEMM, whole and cut into ranges where there is room for
    them, and both Winograd forms)."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad, m = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (rng.standard_normal((K, R, R, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (C * R * R))))
    gamma = rng.uniform(0.5, 1.5, K).astype(np.float32)
    beta = rng.standard_normal(K, dtype=np.float32)
    stats = np.concatenate([rng.standard_normal(K, dtype=np.float32) * np.float32(0.3), rng.uniform(0.5, 2.0, K).astype(np.float32)])
    P = (H + 2 * pad - R) // stride + 1
    Q = (W + 2 * pad - R) // stride + 1
    dx, dwt, dg_, db_, dst = dev(x), dev(w), dev(gamma), dev(beta), dev(stats)
    if m:
        need = monet.call("monet_conv_winograd_workspace_bytes", N, H, W, C, K, m)
    else:
        need = monet.call("monet_conv_workspace_bytes", 0, N, H, W, C, K, R, R, stride, pad, 1) if room else 0
    ws = torch.empty(max(need // 4, 1), dtype=torch.float32, device="cuda")
    wsp = ws.data_ptr() if need else None
    fused = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_fwd_bn_apply", None, dx.data_ptr(), dwt.data_ptr(), fused.data_ptr(), N, H, W, C, K, R, R, stride, pad, m,
               wsp, need, dg_.data_ptr(), db_.data_ptr(), dst.data_ptr())
    y = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
    if m:
        monet.call("monet_conv_winograd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, m, 0, 0, wsp, need)
    else:
        monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1, wsp, need)
    monet.call("monet_bn_apply", None, y.data_ptr(), y.data_ptr(), dg_.data_ptr(), db_.data_ptr(), dst.data_ptr(), N * P * Q, K)
    assert torch.equal(fused, y)
    yo = nm.conv2d_fwd(wt.act_to_oracle(x), wt.weight_to_oracle(w), stride, pad)
    want = nm.bn_apply(yo, gamma.astype(np.float64), beta.astype(np.float64), stats[:K].astype(np.float64), stats[K:].astype(np.float64))
    check_close(fused.cpu().numpy(), wt.act_from_oracle(want), ACT_TOL)
    # ... and with the ReLU / ReLU6 behind the BatchNorm in the same epilogue: the bits of the stand-alone ReLU kernel run in
    # place on the tensor above (values scaled so that the upper clamp of ReLU6 is reached)
    for six in (0, 1):
        g6 = dev(gamma * np.float32(4.0 if six else 1.0))
        plain = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_conv_fwd_bn_apply", None, dx.data_ptr(), dwt.data_ptr(), plain.data_ptr(), N, H, W, C, K, R, R, stride, pad, m,
                   wsp, need, g6.data_ptr(), db_.data_ptr(), dst.data_ptr())
        monet.call("monet_relu_fwd", None, plain.data_ptr(), plain.data_ptr(), None, N * P * Q * K, six)
        both = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), both.data_ptr(), N, H, W, C, K, R, R, stride, pad, m,
                   wsp, need, g6.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, None, None)
        assert torch.equal(both, plain), six
        assert float(both.min()) == 0.0 and (not six or float(both.max()) == 6.0)
        # the ReLU's result beside the BatchNorm's (the BatchNorm output is kept for its own backward operator)
        bn_out = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
        relu_out = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), bn_out.data_ptr(), N, H, W, C, K, R, R, stride, pad, m,
                   wsp, need, g6.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, relu_out.data_ptr(), None)
        want_bn = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_conv_fwd_bn_apply", None, dx.data_ptr(), dwt.data_ptr(), want_bn.data_ptr(), N, H, W, C, K, R, R, stride, pad, m,
                   wsp, need, g6.data_ptr(), db_.data_ptr(), dst.data_ptr())
        assert torch.equal(bn_out, want_bn) and torch.equal(relu_out, plain), six
        # ... and the ReLU's sign code from the same epilogue: the words of the stand-alone kernel (64 | K; the Winograd
        # forms with transformed tensors in memory refuse it)
        words = (N * P * Q * K + 63) // 64
        mask = torch.full((words,), -1, dtype=torch.int64, device="cuda")
        if K % 64 == 0 and m == 0:
            for out2 in (None, relu_out):
                mask.fill_(-1)
                if out2 is not None:
                    out2.fill_(float("nan"))
                bn_out.fill_(float("nan"))
                monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), bn_out.data_ptr(), N, H, W, C, K, R, R, stride, pad, m,
                           wsp, need, g6.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, out2.data_ptr() if out2 is not None else None,
                           mask.data_ptr())
                want_mask = torch.full((words,), -1, dtype=torch.int64, device="cuda")
                scratch = torch.empty_like(want_bn)
                monet.call("monet_relu_fwd", None, want_bn.data_ptr(), scratch.data_ptr(), want_mask.data_ptr(), N * P * Q * K, six)
                assert torch.equal(mask, want_mask), (six, out2 is None)
                assert torch.equal(bn_out if out2 is None else out2, plain), six
                if out2 is not None:
                    assert torch.equal(bn_out, want_bn)
        else:
            with pytest.raises(monet.MonetError):
                monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), bn_out.data_ptr(), N, H, W, C, K, R, R, stride, pad, m,
                           wsp, need, g6.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, relu_out.data_ptr(), mask.data_ptr())
    with pytest.raises(monet.MonetError):       # no Winograd form with 3x3 output tiles
        monet.call("monet_conv_fwd_bn_apply", None, dx.data_ptr(), dwt.data_ptr(), fused.data_ptr(), N, H, W, C, K, R, R, stride, pad, 3,
                   wsp, need, dg_.data_ptr(), db_.data_ptr(), dst.data_ptr())


@pytest.mark.parametrize("m", [2, 4])
@pytest.mark.parametrize("case", [
    (2, 14, 14, 64, 128),       # even map (for 4x4 tiles: the last tile row / column is half outside)
    (3, 7, 9, 32, 48),          # odd sizes: the last tile row / column is partly outside the map
    (1, 5, 5, 16, 16),          # smallest aligned channel counts
    (5, 7, 7, 512, 512),        # deep reduction
    (2, 56, 56, 64, 64),        # many tiles (1568 resp. 392 per GEMM)
    (1, 3, 2, 16, 16),          # a map smaller than one 4x4 tile
])
def test_winograd_convolution_matches_oracle(case, m):
    """F(2x2, 3x3) and F(4x4, 3x3): forward, input gradient (written and accumulated) and filter gradient against the
    oracle's direct definitions."""
    torch = torch_mod()
    N, H, W, C, K = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (rng.standard_normal((K, 3, 3, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (9 * C))))
    dy = rng.standard_normal((N, H, W, K), dtype=np.float32)
    xo, wo, dyo = wt.act_to_oracle(x), wt.weight_to_oracle(w), wt.act_to_oracle(dy)
    dx, dwt, ddy = dev(x), dev(w), dev(dy)
    need = monet.call("monet_conv_winograd_workspace_bytes", N, H, W, C, K, m)
    tiles = N * ((H + m - 1) // m) * ((W + m - 1) // m)
    assert need == (m + 2) ** 2 * 4 * (K * C + tiles * (C + K))
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
    y = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_winograd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, m, 0, 0, ws.data_ptr(), need)
    check_close(y.cpu().numpy(), wt.act_from_oracle(nm.conv2d_fwd(xo, wo, 1, 1)), ACT_TOL)
    gx = torch.full((N, H, W, C), float("nan"), dtype=torch.float32, device="cuda")
    want = wt.act_from_oracle(nm.conv2d_dgrad(dyo, wo, xo.shape, 1, 1))
    monet.call("monet_conv_winograd", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, m, 1, 0, ws.data_ptr(), need)
    check_close(gx.cpu().numpy(), want, GRAD_TOL)
    monet.call("monet_conv_winograd", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, m, 1, 1, ws.data_ptr(), need)
    check_close(gx.cpu().numpy(), 2 * want, GRAD_TOL)
    with pytest.raises(monet.MonetError):
        monet.call("monet_conv_winograd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, 3, 0, 0, ws.data_ptr(), need)
    # a workspace that holds one image at a time: the layer goes through in N chunks, with the same bits
    per_img = (m + 2) ** 2 * 4 * ((H + m - 1) // m) * ((W + m - 1) // m) * (C + K)
    small = (m + 2) ** 2 * 4 * K * C + per_img + 64
    if N > 1:
        y2 = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_conv_winograd", None, dx.data_ptr(), dwt.data_ptr(), y2.data_ptr(), N, H, W, C, K, m, 0, 0, ws.data_ptr(), small)
        assert torch.equal(y, y2)
        if N > 2:      # two images at a time: the last chunk is shorter
            y2.fill_(float("nan"))
            monet.call("monet_conv_winograd", None, dx.data_ptr(), dwt.data_ptr(), y2.data_ptr(), N, H, W, C, K, m, 0, 0, ws.data_ptr(), small + per_img)
            assert torch.equal(y, y2)
    with pytest.raises(monet.MonetError):
        monet.call("monet_conv_winograd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, m, 0, 0, ws.data_ptr(), small - per_img)
    # filter gradient in the transformed domain
    need = monet.call("monet_conv_winograd_wgrad_workspace_bytes", N, H, W, C, K, m)
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
    gw = torch.full((K, 3, 3, C), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_winograd_wgrad", None, dx.data_ptr(), ddy.data_ptr(), gw.data_ptr(), N, H, W, C, K, m, ws.data_ptr(), need)
    want_w = wt.weight_from_oracle(nm.conv2d_wgrad(xo, dyo, 3, 3, 1, 1))
    check_close(gw.cpu().numpy(), want_w, GRAD_TOL)
    if N > 1:       # in chunks of one image: the chunks' shares are added in image order
        planes, tiles_img = (m + 2) ** 2, ((H + m - 1) // m) * ((W + m - 1) // m)
        ranges = max(1, min(1024 // (planes * ((K + 127) // 128) * ((C + 127) // 128)), tiles_img // 128))
        small = per_img + planes * 4 * K * C * (2 + (ranges if ranges > 1 else 0))
        ws.fill_(float("nan"))
        gw.fill_(float("nan"))
        monet.call("monet_conv_winograd_wgrad", None, dx.data_ptr(), ddy.data_ptr(), gw.data_ptr(), N, H, W, C, K, m, ws.data_ptr(), min(small, need))
        check_close(gw.cpu().numpy(), want_w, GRAD_TOL)


@pytest.mark.parametrize("case", [
    (2, 14, 14, 64, 128),       # two blocks of 64 output channels; the last tile row / column is half outside the map
    (3, 7, 9, 32, 48),          # odd sizes, output channels no multiple of 32, fewer tiles than a workgroup takes
    (1, 5, 5, 8, 4),            # smallest channel counts
    (2, 7, 7, 512, 512),        # deep reduction (64 chunks), eight channel blocks
    (3, 56, 56, 64, 64),        # many tiles: 588 per channel block, ragged last workgroup (588 = 18 * 32 + 12)
    (1, 3, 2, 16, 16),          # a map smaller than one 4x4 tile
    (2, 12, 20, 24, 40),        # reduction channels a multiple of 8 only, 40 output channels (second half mostly padding)
    # more work items than CUs with a short remainder, which is worked as half items of 32 output channels:
    (3, 224, 224, 8, 72),       # forward 588 items (512 + 76 halved, every second one with 8 channels in its first half and none
                                # in its second), input gradient 294 (256 + 38 halved, 8 output channels)
    (3, 120, 124, 8, 160),      # 264 items (256 + 8 halved) of three channel blocks, the third half empty; ragged last tile block
])
def test_fused_winograd_convolution_matches_oracle(case):
    """F(4x4, 3x3) in one kernel (no transformed tensors in memory): forward, input gradient written and accumulated,
    and the forward form with a BatchNorm apply step, against the oracle's direct definitions."""
    torch = torch_mod()
    N, H, W, C, K = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (rng.standard_normal((K, 3, 3, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (9 * C))))
    dy = rng.standard_normal((N, H, W, K), dtype=np.float32)
    xo, wo, dyo = wt.act_to_oracle(x), wt.weight_to_oracle(w), wt.act_to_oracle(dy)
    dx, dwt, ddy = dev(x), dev(w), dev(dy)
    need = monet.call("monet_conv_winograd_fused_workspace_bytes", N, H, W, C, K, 0)
    assert need == 36 * 4 * ((K + 63) // 64 * 64) * C
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
    y = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_winograd_fused", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, 0, 0, ws.data_ptr(), need)
    want_y = nm.conv2d_fwd(xo, wo, 1, 1)
    check_close(y.cpu().numpy(), wt.act_from_oracle(want_y), ACT_TOL)
    with pytest.raises(monet.MonetError):
        monet.call("monet_conv_winograd_fused", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, 0, 0, ws.data_ptr(), need - 4)
    # BatchNorm apply step in the epilogue: the bits of the stand-alone apply kernel on the stored output
    gamma = rng.uniform(0.5, 1.5, K).astype(np.float32)
    beta = (0.1 * rng.standard_normal(K)).astype(np.float32)
    stats = np.concatenate([0.1 * rng.standard_normal(K), rng.uniform(0.5, 2.0, K)]).astype(np.float32)
    dg_, db_, dst = dev(gamma), dev(beta), dev(stats)
    fused = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_fwd_bn_apply", None, dx.data_ptr(), dwt.data_ptr(), fused.data_ptr(), N, H, W, C, K, 3, 3, 1, 1, 5,
               ws.data_ptr(), need, dg_.data_ptr(), db_.data_ptr(), dst.data_ptr())
    if K % 4 == 0:
        monet.call("monet_bn_apply", None, y.data_ptr(), y.data_ptr(), dg_.data_ptr(), db_.data_ptr(), dst.data_ptr(), N * H * W, K)
        assert torch.equal(fused, y)
        for six in (0, 1):      # the ReLU behind the BatchNorm in the same epilogue
            both = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
            monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), both.data_ptr(), N, H, W, C, K, 3, 3, 1, 1, 5,
                       ws.data_ptr(), need, dg_.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, None, None)
            plain = y.clone()
            monet.call("monet_relu_fwd", None, plain.data_ptr(), plain.data_ptr(), None, N * H * W * K, six)
            assert torch.equal(both, plain), six
            bn_out = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
            relu_out = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
            monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), bn_out.data_ptr(), N, H, W, C, K, 3, 3, 1, 1, 5,
                       ws.data_ptr(), need, dg_.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, relu_out.data_ptr(), None)
            assert torch.equal(bn_out, y) and torch.equal(relu_out, plain), six
            words = (N * H * W * K + 63) // 64
            mask = torch.full((words,), -1, dtype=torch.int64, device="cuda")
            if K % 64 == 0:      # the ReLU's sign code from the same epilogue: the words of the stand-alone kernel
                bn_out.fill_(float("nan"))
                relu_out.fill_(float("nan"))
                monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), bn_out.data_ptr(), N, H, W, C, K, 3, 3, 1, 1, 5,
                           ws.data_ptr(), need, dg_.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, relu_out.data_ptr(), mask.data_ptr())
                want_mask = torch.full((words,), -1, dtype=torch.int64, device="cuda")
                scratch = torch.empty_like(y)
                monet.call("monet_relu_fwd", None, y.data_ptr(), scratch.data_ptr(), want_mask.data_ptr(), N * H * W * K, six)
                assert torch.equal(mask, want_mask), six
                assert torch.equal(bn_out, y) and torch.equal(relu_out, plain), six
            else:
                with pytest.raises(monet.MonetError):
                    monet.call("monet_conv_fwd_bn_relu", None, dx.data_ptr(), dwt.data_ptr(), bn_out.data_ptr(), N, H, W, C, K, 3, 3, 1, 1, 5,
                               ws.data_ptr(), need, dg_.data_ptr(), db_.data_ptr(), dst.data_ptr(), six, relu_out.data_ptr(), mask.data_ptr())
    want = nm.bn_apply(want_y, gamma.astype(np.float64), beta.astype(np.float64), stats[:K].astype(np.float64), stats[K:].astype(np.float64))
    check_close(fused.cpu().numpy(), wt.act_from_oracle(want), ACT_TOL)
    # input gradient: reduction over K, which must be a multiple of 8
    if K % 8 == 0:
        need = monet.call("monet_conv_winograd_fused_workspace_bytes", N, H, W, C, K, 1)
        assert need == 36 * 4 * ((C + 63) // 64 * 64) * K
        ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
        gx = torch.full((N, H, W, C), float("nan"), dtype=torch.float32, device="cuda")
        want = wt.act_from_oracle(nm.conv2d_dgrad(dyo, wo, xo.shape, 1, 1))
        monet.call("monet_conv_winograd_fused", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, 1, 0, ws.data_ptr(), need)
        check_close(gx.cpu().numpy(), want, GRAD_TOL)
        monet.call("monet_conv_winograd_fused", None, ddy.data_ptr(), dwt.data_ptr(), gx.data_ptr(), N, H, W, C, K, 1, 1, ws.data_ptr(), need)
        check_close(gx.cpu().numpy(), 2 * want, GRAD_TOL)
    else:
        with pytest.raises(monet.MonetError):
            monet.call("monet_conv_winograd_fused", None, ddy.data_ptr(), dwt.data_ptr(), dx.data_ptr(), N, H, W, C, K, 1, 0, ws.data_ptr(), need)


# launches of few results: a 64 x 32 block per workgroup, reduction steps dealt to eight waves
SHORT_CASES = [
    # N, H, W, C, K, R, stride, pad; the directions that take that form (from four steps and up to 512)
    (1, 8, 8, 64, 32, 1, 1, 0, "fw"),       # one block exactly, four steps forward, fewer waves at work than there are
    (1, 5, 13, 132, 36, 1, 1, 0, "fw"),     # a row and a column block more; a last step of four indices
    (2, 9, 7, 20, 44, 3, 1, 1, "fdw"),      # steps that straddle taps
    (1, 11, 10, 32, 64, 3, 2, 1, "fd"),     # residue classes of 4, 2, 2 and 1 taps
    (3, 7, 7, 16, 72, 1, 3, 0, "d"),        # classes without a tap
    (1, 6, 6, 1024, 40, 3, 1, 1, "d"),      # 576 steps forward: the tile kernel; 23 in the input gradient
    (1, 4, 5, 4, 256, 5, 1, 2, "fd"),       # window as large as the map
]


def kernels_of(torch, call):
    """Names of the kernels that a call launches."""
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.name for e in prof.events() if "monet::" in e.name]


def conv_taps(a, R, st, pad, P, Q):
    """What lies under every filter tap, N,P,Q,C."""
    ap = np.pad(a, ((0, 0), (pad, pad), (pad, pad), (0, 0)))
    return {(r, s): ap[:, r:r + (P - 1) * st + 1:st, s:s + (Q - 1) * st + 1:st, :] for r in range(R) for s in range(R)}


def conv64(x, w, dy, st, pad):
    """(y, dx, dw) in 64 bits."""
    x, w, dy = (v.astype(np.float64) for v in (x, w, dy))
    (N, H, W, C), (K, R), (P, Q) = x.shape, w.shape[:2], dy.shape[1:3]
    under = conv_taps(x, R, st, pad, P, Q)
    y = sum(under[r, s] @ w[:, r, s, :].T for r, s in under)
    dx = np.zeros((N, H + 2 * pad, W + 2 * pad, C))
    dw = np.zeros((K, R, R, C))
    for r, s in under:
        dx[:, r:r + (P - 1) * st + 1:st, s:s + (Q - 1) * st + 1:st, :] += dy @ w[:, r, s, :]
        dw[:, r, s, :] = np.tensordot(dy, under[r, s], ((0, 1, 2), (0, 1, 2)))
    return y, dx[:, pad:pad + H, pad:pad + W, :], dw


@pytest.mark.gpu
@pytest.mark.parametrize("case", SHORT_CASES)
@pytest.mark.parametrize("kind", ["plain", "tiny", "infinite"])
def test_convolutions_of_few_results_match_64_bits(case, kind):
    """Forward pass, input gradient (written and accumulated) and filter gradient without workspace.  A sum of n products of fp32 operands, rounded once per step
    of 16 at most: 2e-7 of the sum of the products' sizes bounds it.  Operands near 2^-120 and an infinity go through the fp32 instruction, which rounds after
    every product: n * 2^-24 of it."""
    torch = torch_mod()
    N, H, W, C, K, R, st, pad, short = case
    P, Q = (H + 2 * pad - R) // st + 1, (W + 2 * pad - R) // st + 1
    rng = np.random.default_rng(21)
    x, dy = rng.standard_normal((N, H, W, C), dtype=np.float32), rng.standard_normal((N, P, Q, K), dtype=np.float32)
    w = rng.standard_normal((K, R, R, C), dtype=np.float32)
    if kind == "tiny":
        x, dy = x * np.float32(2.0 ** -118), dy * np.float32(2.0 ** -121)
    dims = (N, H, W, C, K, R, R, st, pad)
    xs, ws, ds = dev(x), dev(w), dev(dy)
    if kind == "infinite":
        xs[0, 0, 0, 0] = ds[0, 0, 0, 0] = float("inf")

    want, size = conv64(x, w, dy, st, pad), conv64(np.abs(x), np.abs(w), np.abs(dy), st, pad)
    y = torch.full((N, P, Q, K), float("nan"), device="cuda")
    dx, dw = torch.full((N, H, W, C), float("nan"), device="cuda"), torch.full((K, R, R, C), float("nan"), device="cuda")
    calls = {"f": lambda: monet.call("monet_conv_fwd", None, xs.data_ptr(), ws.data_ptr(), y.data_ptr(), *dims, 1, None, 0),
             "d": lambda: monet.call("monet_conv_dgrad", None, ds.data_ptr(), ws.data_ptr(), dx.data_ptr(), *dims, 0, 1, None, 0),
             "w": lambda: monet.call("monet_conv_wgrad", None, xs.data_ptr(), ds.data_ptr(), dw.data_ptr(), *dims, 1, None, 0)}
    for mode, (direction, call) in enumerate(calls.items()):
        if kind == "plain": assert any(f"conv_short_kernel<{mode}>" in k for k in kernels_of(torch, call)) == (direction in short), direction
        else: call()
    twice = dx.clone()
    monet.call("monet_conv_dgrad", None, ds.data_ptr(), ws.data_ptr(), twice.data_ptr(), *dims, 1, 1, None, 0)
    outs = [t.cpu().numpy() for t in (y, dx, dw)]
    for got, ref, sz, n in zip(outs, want, size, (C * R * R, K * R * R, N * P * Q)):
        if kind == "infinite":
            sure = np.isfinite(got)      # untouched by the infinities: as many as the definition says, checked below
            got, ref, sz = got[sure], ref[sure], sz[sure]
        assert (np.abs(got - ref) <= (2e-7 if kind == "plain" else max(2e-7, n * 2.0 ** -24)) * sz + 2.0 ** -148).all()
    if kind == "infinite":
        xi, di = x.copy(), dy.copy()
        xi[0, 0, 0, 0] = di[0, 0, 0, 0] = np.inf
        with np.errstate(invalid="ignore"):
            under = conv_taps(xi, R, st, pad, P, Q)
            hit = sum((~np.isfinite(under[k])).any(-1) for k in under) > 0
        assert (np.isfinite(outs[0]).all(-1) == ~hit).all()
        assert not np.isfinite(outs[1]).all() and not np.isfinite(outs[2]).all()
    else:
        assert (torch.abs(twice - 2 * dx) <= 1e-6 * torch.abs(dx) + 2.0 ** -148).all()


# launches of few results with a workgroup per 32 rows, and the edges of that rule
@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    # direction, N, H, W, C, K, R, stride, pad, ranges, form (rows per workgroup, 0: the tile kernel)
    ("f", 1, 1, 1, 64, 4, 1, 1, 0, 1, 32),           # one row
    ("f", 1, 4, 8, 64, 36, 1, 1, 0, 1, 32),          # 32 rows, two blocks of columns
    ("f", 1, 3, 11, 20, 32, 3, 1, 1, 1, 32),         # 33
    ("f", 128, 8, 8, 64, 32, 1, 1, 0, 1, 32),        # 128 blocks of 64 rows
    ("f", 129, 8, 8, 64, 32, 1, 1, 0, 1, 64),        # 129
    ("f", 8, 8, 8, 1280, 32, 1, 1, 0, 8, 32),        # cut, 80 steps
    ("f", 8, 8, 8, 1284, 32, 1, 1, 0, 8, 0),         # 81
    ("f", 7, 8, 8, 640, 32, 1, 1, 0, 4, 0),          # seven blocks, cut
    ("d", 5, 13, 11, 36, 28, 3, 2, 1, 1, 32),        # residue classes of different sizes
    ("d", 8, 8, 8, 32, 1280, 1, 1, 0, 8, 32),
    ("d", 8, 8, 8, 32, 1284, 1, 1, 0, 8, 0),
    ("a", 8, 8, 8, 32, 1088, 1, 1, 0, 8, 32),        # accumulating: 68 steps
    ("a", 8, 8, 8, 32, 1092, 1, 1, 0, 8, 0),
    ("w", 1, 8, 8, 64, 33 * 4, 3, 1, 1, 1, 32),      # 132 rows
    ("w", 2, 16, 20, 48, 32, 3, 1, 1, 4, 32),        # cut, at most 64 rows, 40 steps
    ("w", 2, 16, 21, 48, 32, 3, 1, 1, 4, 0),         # 42
    ("w", 2, 16, 29, 48, 68, 3, 1, 1, 4, 32),        # more than 64 rows, 58
    ("w", 2, 16, 30, 48, 68, 3, 1, 1, 4, 0),         # 60
])
def test_convolutions_of_few_results_in_blocks_of_32_rows_match_64_bits(case):
    """Bounds as above."""
    torch = torch_mod()
    direction, N, H, W, C, K, R, st, pad, splits, form = case
    P, Q = (H + 2 * pad - R) // st + 1, (W + 2 * pad - R) // st + 1
    rng = np.random.default_rng(23)
    x, dy = rng.standard_normal((N, H, W, C), dtype=np.float32), rng.standard_normal((N, P, Q, K), dtype=np.float32)
    w = rng.standard_normal((K, R, R, C), dtype=np.float32)
    i = {"f": 0, "d": 1, "a": 1, "w": 2}[direction]
    want, size = conv64(x, w, dy, st, pad)[i], conv64(np.abs(x), np.abs(w), np.abs(dy), st, pad)[i]
    before = x if direction == "a" else np.full(want.shape, np.nan, dtype=np.float32)
    xs, ws, ds, out = dev(x), dev(w), dev(dy), dev(before)
    room = torch.empty(splits * out.numel(), device="cuda")
    dims, tail = (N, H, W, C, K, R, R, st, pad), (splits, room.data_ptr() if splits > 1 else None, room.numel() * 4 if splits > 1 else 0)

    def call():
        out.copy_(dev(before))
        if i == 0: monet.call("monet_conv_fwd", None, xs.data_ptr(), ws.data_ptr(), out.data_ptr(), *dims, *tail)
        elif i == 1: monet.call("monet_conv_dgrad", None, ds.data_ptr(), ws.data_ptr(), out.data_ptr(), *dims, int(direction == "a"), *tail)
        else: monet.call("monet_conv_wgrad", None, xs.data_ptr(), ds.data_ptr(), out.data_ptr(), *dims, *tail)

    name = f"rows{form}::conv_short_kernel<{i}>" if form else f"conv_tile_kernel<{i},"
    assert any(name in k for k in kernels_of(torch, call)), name
    if direction == "a":
        want, size = want + x, size + np.abs(x)
    assert (np.abs(out.cpu().numpy() - want) <= 2e-7 * size).all()


@pytest.mark.gpu
@pytest.mark.parametrize("value", [1.2345678 * 2.0 ** -122, float("inf"), float("nan")])
@pytest.mark.parametrize("R", [1, 3])
def test_convolution_of_few_results_has_the_same_bits_with_and_without_statistics(R, value):
    """The first run of a layer leaves the statistics of its output and works 64 rows at a time, its recomputation 32: rows that hold nothing special must not be worked on
    another instruction in one of them because of a neighbour that the pieces cannot hold."""
    torch = torch_mod()
    N, H, W, C, K = 2, 12, 12, 64, 64
    g = torch.Generator().manual_seed(3)
    x, w = torch.randn(N, H, W, C, generator=g), torch.randn(K, R, R, C, generator=g) * 0.1
    x[0, 0, 5, 7] = value
    x[1, 7, 11, 60] = value
    x, w = x.cuda(), w.cuda()
    gamma, beta = torch.rand(K, generator=g).cuda() + 0.5, torch.randn(K, generator=g).cuda()
    first, plain, again = (torch.full((N, H, W, K), -1.0, device="cuda") for _ in range(3))
    stats, scratch = torch.empty(2 * K, device="cuda"), torch.empty(1 << 20, device="cuda")
    dims = (N, H, W, C, K, R, R, 1, R // 2)
    runs = {
        "rows64": lambda: monet.call("monet_conv_fwd_bn_stats", None, x.data_ptr(), w.data_ptr(), first.data_ptr(), *dims, None, 0, stats.data_ptr(), 1e-5, scratch.data_ptr(), scratch.numel() * 4),
        "rows32": lambda: monet.call("monet_conv_fwd", None, x.data_ptr(), w.data_ptr(), plain.data_ptr(), *dims, 1, None, 0),
    }
    for form, call in runs.items():
        assert any(form + "::conv_short_kernel<0>" in k for k in kernels_of(torch, call))
    stats = torch.cat([torch.randn(K, generator=g), torch.rand(K, generator=g) + 0.5]).cuda()      # of finite values
    monet.call("monet_bn_apply", None, first.data_ptr(), first.data_ptr(), gamma.data_ptr(), beta.data_ptr(), stats.data_ptr(), N * H * W, K)
    monet.call("monet_bn_apply", None, plain.data_ptr(), plain.data_ptr(), gamma.data_ptr(), beta.data_ptr(), stats.data_ptr(), N * H * W, K)
    monet.call("monet_conv_fwd_bn_apply", None, x.data_ptr(), w.data_ptr(), again.data_ptr(), *dims, 0, None, 0, gamma.data_ptr(), beta.data_ptr(), stats.data_ptr())
    bits = [t.view(torch.int32).cpu() for t in (first, plain, again)]
    assert torch.equal(bits[0], bits[1]) and torch.equal(bits[0], bits[2])


# tile shapes and wave groups of the forward pass and the input gradient
GROUP_CASES = [
    # N, H, W, C, K, R, stride, pad, splits; kernel of the forward pass and of the input gradient: rows / 64, columns / 32, loader, groups (None: the form of few results)
    (5, 28, 28, 80, 160, 3, 1, 1, 1, (2, 2, 1, 2), None),                 # two groups on 128x64 tiles, 45 steps: one turn more for the first
    (5, 28, 28, 160, 80, 3, 1, 1, 1, None, (2, 2, 1, 2)),                 # the same in the input gradient
    (9, 27, 28, 176, 176, 3, 1, 1, 1, (2, 2, 1, 2), (2, 2, 1, 2)),        # 99 steps, ragged tiles
    (4, 28, 28, 192, 512, 3, 2, 1, 1, None, (2, 2, 1, 2)),                # residue classes of 128, 64, 64 and 32 steps
    (6, 28, 28, 256, 512, 1, 2, 0, 1, (2, 2, 1, 1), (2, 2, 1, 2)),        # three of four classes without a tap
    (5, 28, 28, 192, 192, 3, 1, 1, 3, (2, 4, 1, 2), (2, 4, 1, 2)),        # two groups on 128x128 tiles, cut into three ranges of 36 steps
    (2, 208, 200, 16, 24, 3, 1, 1, 1, (2, 1, 1, 1), (2, 1, 3, 1)),        # 128x32 tiles: 24 columns forward; 16 and steps that straddle taps in the input gradient
    (2, 208, 200, 20, 32, 3, 1, 1, 1, (2, 1, 3, 1), (2, 1, 1, 1)),        # and the other way about
    (1, 5, 11, 512, 132, 1, 1, 0, 4, (1, 4, 1, 1), None),                 # 64x128 tiles: at most 64 rows of a cut 1x1 layer
    (1, 5, 11, 132, 512, 1, 1, 0, 4, None, (1, 4, 1, 1)),
    (64, 1, 1, 1284, 516, 1, 1, 0, 8, (1, 4, 2, 1), None),                # and a last step of four indices
    (64, 1, 1, 516, 1284, 1, 1, 0, 8, None, (1, 4, 2, 1)),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", GROUP_CASES)
@pytest.mark.parametrize("infinite", [False, True])
def test_convolution_tiles_and_wave_groups_match_64_bits(case, infinite):
    """Bounds as above; `infinite`: a tile is worked again on the fp32 instruction, by both groups."""
    torch = torch_mod()
    N, H, W, C, K, R, st, pad, splits, *kernels = case
    P, Q = (H + 2 * pad - R) // st + 1, (W + 2 * pad - R) // st + 1
    rng = np.random.default_rng(22)
    x, dy = rng.standard_normal((N, H, W, C), dtype=np.float32), rng.standard_normal((N, P, Q, K), dtype=np.float32)
    w = rng.standard_normal((K, R, R, C), dtype=np.float32)
    want, size = conv64(x, w, dy, st, pad), conv64(np.abs(x), np.abs(w), np.abs(dy), st, pad)
    xs, ws, ds = dev(x), dev(w), dev(dy)
    if infinite:
        xs[0, 0, 0, 0] = ds[0, 0, 0, 0] = float("inf")
    y, dx = torch.full((N, P, Q, K), float("nan"), device="cuda"), torch.full((N, H, W, C), float("nan"), device="cuda")
    room = torch.empty(splits * max(y.numel(), dx.numel()), device="cuda")
    dims = (N, H, W, C, K, R, R, st, pad)
    wsp, wsb = (room.data_ptr(), room.numel() * 4) if splits > 1 else (None, 0)
    calls = (lambda: monet.call("monet_conv_fwd", None, xs.data_ptr(), ws.data_ptr(), y.data_ptr(), *dims, splits, wsp, wsb),
             lambda: monet.call("monet_conv_dgrad", None, ds.data_ptr(), ws.data_ptr(), dx.data_ptr(), *dims, 0, splits, wsp, wsb))
    for mode, (call, kernel) in enumerate(zip(calls, kernels)):
        name = f"conv_short_kernel<{mode}>" if kernel is None else "conv_tile_kernel<%d, %d, %d, %d, 0, %d>" % (mode, *kernel)
        assert any(name in k for k in kernels_of(torch, call)), name
    for got, ref, sz, n in zip((y.cpu().numpy(), dx.cpu().numpy()), want, size, (C * R * R, K * R * R)):
        sure = np.isfinite(got)
        assert sure.all() != infinite and sure.mean() > (0.9 if N * P * Q > 100 else 0.5)
        bound = max(2e-7, n * 2.0 ** -24) if infinite else 2e-7
        assert (np.abs(got - ref)[sure] <= bound * sz[sure]).all()


def times_taken_and_forced(torch, call, runs):
    """Microseconds of a convolution call by itself and with the 128x64 tile forced, in turn, the least of a few measurements each."""
    best = [float("inf"), float("inf")]
    try:
        for _ in range(8):
            for forced in (0, 1):
                monet.call("monet_conv_force_tile", 3 if forced else -1)
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                call()
                a.record()
                for _ in range(runs):
                    call()
                b.record()
                torch.cuda.synchronize()
                best[forced] = min(best[forced], a.elapsed_time(b) * 1e3 / runs)
    finally:
        monet.call("monet_conv_force_tile", -1)
    return best


@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    # mode, N, H, W, C, K, R, stride, pad
    ("dgrad", 26, 77, 80, 8, 180, 3, 1, 0),       # 1252 workgroups of 128 rows: two rounds on either tile
    ("dgrad", 100, 31, 31, 8, 968, 1, 3, 0),      # nine residue classes, one of them with a tap: 95 workgroups that multiply
    ("fwd", 61, 50, 50, 176, 20, 3, 1, 1),        # 1192 workgroups
    ("fwd", 32, 69, 72, 312, 8, 2, 1, 0),         # 1207
    ("fwd", 83, 41, 41, 344, 16, 1, 1, 0),        # 1091, a 1x1 layer
])
def test_narrow_results_take_no_slower_tile_than_the_128x64_one(case):
    torch = torch_mod()
    mode, N, H, W, C, K, R, st, pad = case
    P, Q = (H + 2 * pad - R) // st + 1, (W + 2 * pad - R) // st + 1
    x, w, y = torch.randn(N, H, W, C, device="cuda"), torch.randn(K, R, R, C, device="cuda"), torch.randn(N, P, Q, K, device="cuda")
    dims = (N, H, W, C, K, R, R, st, pad)

    def call():
        if mode == "fwd": monet.call("monet_conv_fwd", None, x.data_ptr(), w.data_ptr(), y.data_ptr(), *dims, 1, None, 0)
        else: monet.call("monet_conv_dgrad", None, y.data_ptr(), w.data_ptr(), x.data_ptr(), *dims, 0, 1, None, 0)

    taken, wide = times_taken_and_forced(torch, call, 20)
    assert taken < 1.08 * wide + 0.5


@pytest.mark.gpu
@pytest.mark.parametrize("case", [
    # N, H, W, C, K, R, stride, pad, ranges
    (3, 17, 17, 56, 712, 1, 1, 0, 5),       # 45 steps, 28 blocks of 64x32
    (34, 8, 8, 40, 80, 3, 1, 1, 5),         # 45 steps, 68 blocks
    (1, 16, 16, 48, 32, 5, 1, 2, 6),        # 50 steps, 8 blocks
])
def test_cut_input_gradients_that_accumulate_take_the_faster_form(case):
    """Against the tile kernel with as many ranges."""
    torch = torch_mod()
    N, H, W, C, K, R, st, pad, splits = case
    P, Q = (H + 2 * pad - R) // st + 1, (W + 2 * pad - R) // st + 1
    dx, w, dy = torch.zeros(N, H, W, C, device="cuda"), torch.randn(K, R, R, C, device="cuda"), torch.randn(N, P, Q, K, device="cuda")
    ws = torch.empty(splits * dx.numel(), device="cuda")

    def call():
        monet.call("monet_conv_dgrad", None, dy.data_ptr(), w.data_ptr(), dx.data_ptr(), N, H, W, C, K, R, R, st, pad, 1, splits, ws.data_ptr(), ws.numel() * 4)

    taken, tile = times_taken_and_forced(torch, call, 60)
    assert taken < 1.04 * tile + 0.3


@pytest.mark.gpu
@pytest.mark.parametrize("rows, C, slabs, kernel", [
    # slabs: partial results that the scratch holds (0: 4 MiB of them)
    (1, 4, 0, "small"), (33, 16, 0, "small"), (512, 16, 0, "small"), (2047, 16, 0, "small"), (4099, 16, 0, "final"), (70, 60, 0, "small"), (300, 256, 0, "small"),
    (300, 260, 0, "small"), (40, 1024, 0, "small"),
    (8192, 4, 0, "few"), (8193, 4, 0, "final"),                          # 16 and 17 slabs of 512 rows
    (1025, 36, 0, "few"), (1344, 36, 0, "few"), (1345, 36, 0, "final"),      # nine channel groups: of 64, rounded up to three sweeps of 28
    (2500, 256, 16, "few"), (2500, 256, 17, "final"), (2500, 260, 16, "final"),
    (5000, 20, 1, "few"),
])
def test_bn_backward_of_few_and_many_slabs_matches_64_bits(rows, C, slabs, kernel):
    """Partial sums that every apply workgroup adds for itself (up to 16 slabs and 256 channels) and beyond; tensors of few rows go through one kernel.  Sums of `rows` terms in
    fp32, in slabs: 1e-5 of the terms' sizes."""
    torch = torch_mod()
    rng = np.random.default_rng(9)
    dy, x = rng.standard_normal((rows, C), dtype=np.float32), rng.standard_normal((rows, C), dtype=np.float32) + np.float32(0.5)
    gamma, beta = rng.uniform(0.5, 1.5, C).astype(np.float32), rng.standard_normal(C).astype(np.float32)
    mean, inv = x.astype(np.float64).mean(0), 1 / np.sqrt(x.astype(np.float64).var(0) + 1e-5)
    stats = np.concatenate([mean, inv]).astype(np.float32)
    g, xhat = dy.astype(np.float64), (x - stats[:C].astype(np.float64)) * stats[C:].astype(np.float64)
    want_b, want_g = g.sum(0), (g * xhat).sum(0)
    scale = gamma.astype(np.float64) * stats[C:]
    want_dx = scale * (g - want_b / rows - xhat * (want_g / rows))
    dx = torch.full((rows, C), float("nan"), device="cuda")
    dgamma, dbeta = torch.full((C,), float("nan"), device="cuda"), torch.full((C,), float("nan"), device="cuda")
    scratch = torch.empty((slabs + 1) * 8 * C if slabs else 4 << 20, dtype=torch.uint8, device="cuda")
    dyd, xd, gd, bd, sd = dev(dy), dev(x), dev(gamma), dev(beta), dev(stats)
    names = kernels_of(torch, lambda: monet.call("monet_bn_bwd", None, dyd.data_ptr(), xd.data_ptr(), 0, gd.data_ptr(), bd.data_ptr(), sd.data_ptr(), dx.data_ptr(), dgamma.data_ptr(),
                                                 dbeta.data_ptr(), rows, C, 0, scratch.data_ptr(), scratch.numel()))
    assert any({"small": "bn_bwd_small<", "few": "bn_bwd_apply<false, 0, true>", "final": "bn_bwd_final"}[kernel] in k for k in names), names
    size_b, size_g = np.abs(g).sum(0), (np.abs(g) * (np.abs(xhat) + np.abs(stats[:C]) * stats[C:])).sum(0)
    assert (np.abs(dbeta.cpu().numpy() - want_b) <= 1e-5 * size_b).all()
    assert (np.abs(dgamma.cpu().numpy() - want_g) <= 1e-5 * size_g).all()
    bound = 1e-5 * scale * (np.abs(g) + size_b / rows + (np.abs(xhat) + np.abs(stats[:C]) * stats[C:]) * (1 + size_g / rows))
    assert (np.abs(dx.cpu().numpy() - want_dx) <= bound).all()


# the edges of what one launch takes and of the rows and channel groups a workgroup is given: rows, channels, whether one launch takes them written and accumulated
ONE_LAUNCH_CASES = [
    (1, 4, 1, 1), (2, 36, 1, 1), (49, 1028, 1, 1), (512, 32, 1, 1), (1400, 64, 1, 1), (1401, 64, 1, 0), (2048, 256, 1, 0), (2049, 32, 0, 0), (2048, 28, 1, 0), (513, 20, 1, 1), (1025, 288, 0, 0),
    (320, 68, 1, 1), (321, 68, 1, 0), (320, 36, 1, 1), (784, 60, 1, 0), (785, 60, 0, 0), (1024, 68, 1, 0), (1025, 68, 0, 0), (1024, 48, 1, 0), (1025, 48, 0, 0), (128, 132, 1, 1), (129, 132, 1, 1),
    (1024, 2048, 1, 1), (1025, 260, 0, 0), (2049, 64, 0, 0), (4096, 60, 0, 0), (4097, 8, 0, 0), (1024, 25088, 0, 0), (63, 16388, 0, 0), (63, 16384, 1, 1), (64, 20004, 1, 1),
    (1, 65536, 0, 0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("rows, C, written, accumulated", ONE_LAUNCH_CASES)
def test_bn_backward_in_one_launch_matches_64_bits(rows, C, written, accumulated):
    """From the input and from the output, written and accumulated.  Sums as above: 1e-5 of the terms' sizes."""
    torch = torch_mod()
    rng = np.random.default_rng(rows + C)
    dy, x = rng.standard_normal((rows, C), dtype=np.float32), rng.standard_normal((rows, C), dtype=np.float32) + np.float32(0.5)
    gamma, beta = rng.uniform(0.5, 1.5, C).astype(np.float32), rng.standard_normal(C).astype(np.float32)
    mean, inv = x.astype(np.float64).mean(0), 1 / np.sqrt(x.astype(np.float64).var(0) + 1e-5)
    stats = np.concatenate([mean, inv]).astype(np.float32)
    xhat = (x - stats[:C].astype(np.float64)) * stats[C:].astype(np.float64)
    y = (gamma * xhat + beta).astype(np.float32)
    dyd, gd, bd, sd = dev(dy), dev(gamma), dev(beta), dev(stats)
    scratch = torch.empty(4 << 20, dtype=torch.uint8, device="cuda")
    scale = gamma.astype(np.float64) * stats[C:]
    g = dy.astype(np.float64)
    want_b, want_g = g.sum(0), (g * xhat).sum(0)
    want_dx = scale * (g - want_b / rows - xhat * (want_g / rows))
    for from_output in (0, 1):
        # an xhat taken from the output carries the output's rounding, and what beta takes from it
        size_x = np.abs(xhat) + (np.abs(stats[:C]) * stats[C:] if not from_output else (np.abs(y) + np.abs(beta)) / gamma)
        size_b, size_g = np.abs(g).sum(0), (np.abs(g) * size_x).sum(0)
        bound = 1e-5 * scale * (np.abs(g) + size_b / rows + size_x * (1 + size_g / rows))
        for acc in (0, 1):
            dx = dev(x) if acc else torch.full((rows, C), float("nan"), device="cuda")
            dgamma, dbeta = torch.full((C,), float("nan"), device="cuda"), torch.full((C,), float("nan"), device="cuda")
            td = dev(y if from_output else x)
            names = kernels_of(torch, lambda: monet.call("monet_bn_bwd", None, dyd.data_ptr(), td.data_ptr(), from_output, gd.data_ptr(), bd.data_ptr(), sd.data_ptr(), dx.data_ptr(),
                                                         dgamma.data_ptr(), dbeta.data_ptr(), rows, C, acc, scratch.data_ptr(), scratch.numel()))
            assert any("bn_bwd_small" in k for k in names) == bool(accumulated if acc else written), names
            assert (np.abs(dbeta.cpu().numpy() - want_b) <= 1e-5 * size_b).all()
            assert (np.abs(dgamma.cpu().numpy() - want_g) <= 1e-5 * size_g).all()
            assert (np.abs(dx.cpu().numpy() - (want_dx + (x if acc else 0))) <= bound + 1e-7 * acc * np.abs(x)).all()


# one-kernel Winograd form on fp16 pieces: reductions of 64 channels and more, in chunks of 16
PIECES_CASES = [
    # N, H, W, C, K
    (1, 4, 4, 64, 64),          # one tile, the shortest reduction, square for both directions
    (3, 9, 10, 80, 64),         # ragged tiles, five chunks; one block of tiles and a part of a second
    (2, 13, 17, 64, 96),        # half-empty second channel block forward; two blocks of outputs in the input gradient
    (1, 5, 30, 112, 72),        # odd chunk count; 72 reduction channels in the input gradient keep the fp32 form
    (11, 28, 28, 64, 64),       # 17 whole blocks of tiles
    (1, 4, 5, 560, 1008),       # filters in workgroups of two chunks, the last of one
]


def winograd_one_kernel(torch, src, w, out, dims, adjoint, accumulate=0):
    need = monet.call("monet_conv_winograd_fused_workspace_bytes", *dims, adjoint)
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_winograd_fused", None, src.data_ptr(), w.data_ptr(), out.data_ptr(), *dims, adjoint, accumulate, ws.data_ptr(), need)
    return out


def winograd64(x, w):
    """3x3 / stride 1 / pad 1 in 64 bits; x: N,H,W,C, w: K,3,3,C."""
    n, h, wd, _ = x.shape
    xp = np.pad(x.astype(np.float64), ((0, 0), (1, 1), (1, 1), (0, 0)))
    return sum(xp[:, r:r + h, s:s + wd, :] @ w[:, r, s, :].astype(np.float64).T for r in range(3) for s in range(3))


@pytest.mark.gpu
@pytest.mark.parametrize("case", PIECES_CASES)
def test_winograd_on_pieces_matches_64_bits(case):
    """Forward pass and input gradient (written, accumulated).  F(4x4, 3x3) in fp32 is within 4e-6 of 64 bits for up to 512 channels (measured
    1.3e-6 .. 3.5e-6); the pieces have fewer roundings, so 4e-6 bounds both.  Beyond, the rounding of the sums grows with the square root of the number of
    chunks."""
    torch = torch_mod()
    N, H, W, C, K = case
    rng = np.random.default_rng(5)
    x, dy = rng.standard_normal((N, H, W, C), dtype=np.float32), rng.standard_normal((N, H, W, K), dtype=np.float32)
    w = rng.standard_normal((K, 3, 3, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (9 * C)))
    turned = np.ascontiguousarray(w[:, ::-1, ::-1, :].transpose(3, 1, 2, 0))
    for src, filt, out_c, adjoint in ((x, w, K, 0), (dy, turned, C, 1)):
        want = winograd64(src, filt)
        out = torch.full((N, H, W, out_c), float("nan"), dtype=torch.float32, device="cuda")
        got = winograd_one_kernel(torch, dev(src), dev(w), out, case, adjoint).cpu().numpy()
        bound = 4e-6 * max(1.0, np.sqrt(src.shape[3] / 512))
        assert np.linalg.norm(got - want) < bound * np.linalg.norm(want)
        twice = winograd_one_kernel(torch, dev(src), dev(w), out, case, adjoint, 1).cpu().numpy()
        assert np.linalg.norm(twice - 2 * want) < 2 * bound * np.linalg.norm(want)


# (batch, map, C, K, images that the workspace holds at a time: 0 all of them)
WGRAD_MAPS_CASES = [
    (1, 1, 1, 4, 4, 0),            # one tile, four channels
    (1, 3, 2, 8, 60, 0),           # a map smaller than a tile, channels short of a block
    (3, 17, 20, 64, 68, 0),        # 75 tiles, one row of which is a quarter full; a second block of four filters
    (5, 12, 4, 68, 64, 1),         # tiles one above the other; chunks of one image with three tiles
    (1, 4, 60, 132, 64, 0),        # 15 tiles, one short of a chunk; three blocks of channels
    (1, 4, 64, 64, 132, 0),        # 16: one chunk
    (1, 4, 68, 64, 64, 0),         # 17
    (2, 31, 33, 320, 260, 0),      # 144 tiles and 25 pairs of blocks: not this form
    (1, 8, 11, 320, 260, 0),       # 6 tiles and 25 pairs of blocks
    (3, 40, 44, 96, 128, 2),       # four pairs of blocks, two ranges of seven chunks of tiles; the last chunk of images is shorter
    (2, 120, 132, 64, 64, 1),      # 16 ranges of four chunks per image
    (1, 200, 240, 68, 68, 0),      # ten ranges of 19 chunks, eleven to a partial sum: the second one is added in memory
    (2, 200, 240, 68, 68, 1),      # the same in two chunks of images
]


def wgrad_maps(torch, x, dy, case):
    N, H, W, C, K, imgs = case
    need = monet.call("monet_conv_winograd_wgrad_workspace_bytes", N, H, W, C, K, 4)
    if imgs:      # what the check of the workspace asks for `imgs` images and one partial result
        tiles = ((H + 3) // 4) * ((W + 3) // 4)
        ranges = max(1, min(1024 // (36 * ((K + 127) // 128) * ((C + 127) // 128)), imgs * tiles // 128))
        need = min(need, 4 * 36 * (imgs * tiles * (C + K) + K * C * (2 + (ranges if ranges > 1 else 0))))
    ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
    dw = torch.full((K, 3, 3, C), float("nan"), dtype=torch.float32, device="cuda")
    dx, ddy = dev(x), dev(dy)
    monet.call("monet_conv_winograd_wgrad", None, dx.data_ptr(), ddy.data_ptr(), dw.data_ptr(), N, H, W, C, K, 4, ws.data_ptr(), need)
    return dw.cpu().numpy()


def wgrad64(x, dy):
    n, h, w, C = x.shape
    xp = np.pad(x.astype(np.float64), ((0, 0), (1, 1), (1, 1), (0, 0)))
    g = dy.astype(np.float64).reshape(-1, dy.shape[3])
    return np.stack([np.stack([g.T @ xp[:, r:r + h, s:s + w, :].reshape(-1, C) for s in range(3)], 1) for r in range(3)], 1)


@pytest.mark.gpu
@pytest.mark.parametrize("case", WGRAD_MAPS_CASES)
def test_winograd_wgrad_with_horizontal_maps_in_the_gemm_matches_64_bits(case):
    """The transforms' rounding makes the filter gradient of F(4x4, 3x3) 0.5 .. 2.1e-6 normwise (measured, up to 140000 tiles); these have at most
    6000, whose sums add less: 2e-6.  Twice the same bits."""
    torch = torch_mod()
    N, H, W, C, K, _ = case
    rng = np.random.default_rng(3)
    x, dy = np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0), rng.standard_normal((N, H, W, K), dtype=np.float32) * np.float32(1e-3)
    want = wgrad64(x, dy)
    got = wgrad_maps(torch, x, dy, case)
    assert np.linalg.norm(got - want) <= 2e-6 * np.linalg.norm(want)
    assert np.abs(got - want).max() <= 50 * 2e-6 * np.sqrt((want ** 2).mean()) + 1e-30
    assert np.array_equal(got, wgrad_maps(torch, x, dy, case))


@pytest.mark.gpu
@pytest.mark.parametrize("case, taken", [
    # batch, map, C, K: blocks of 64 channels and filters, tiles
    ((1, 4, 4, 448, 384), True), ((1, 4, 4, 448, 448), False), ((1, 4, 4, 64, 2752), False),      # 42, 49 and 43 pairs of blocks
    ((1, 64, 32, 68, 68), True), ((1, 172, 12, 68, 68), False),                                   # 128 and 129 tiles, two blocks on either side
    ((1, 60, 68, 68, 68), False), ((1, 64, 64, 68, 68), True),                                    # 255, 256
    ((1, 120, 120, 68, 132), True), ((1, 68, 212, 68, 68), False),                                # 900, 901
    ((1, 116, 412, 68, 68), False), ((1, 200, 240, 68, 68), True),                                # 2987, 3000
    ((1, 68, 212, 64, 320), True), ((1, 68, 212, 64, 324), False), ((1, 64, 64, 448, 64), False),      # one block on one side: five, six, seven pairs
])
def test_winograd_wgrad_takes_the_faster_form(case, taken):
    """Horizontal maps in the GEMM, or tiles mapped both ways in the workspace: the form on either side of its lines, and that it is right there.  Bound as above."""
    torch = torch_mod()
    N, H, W, C, K = case
    rng = np.random.default_rng(5)
    x, dy = rng.standard_normal((N, H, W, C), dtype=np.float32), rng.standard_normal((N, H, W, K), dtype=np.float32)
    got = []
    names = kernels_of(torch, lambda: got.append(wgrad_maps(torch, x, dy, case + (0,))))
    assert any("wino4_wgrad_kernel" in k for k in names) == taken, names
    want = wgrad64(x, dy)
    assert np.linalg.norm(got[0] - want) <= 2e-6 * np.linalg.norm(want)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["tiny", "huge", "infinity", "nan"])
@pytest.mark.parametrize("case", [
    (2, 13, 18, 72, 40, 0),        # three chunks of tiles: one range, one partial sum
    (3, 40, 44, 96, 128, 2),       # two ranges, added to the first images' gradient
    (1, 200, 240, 68, 68, 0),      # ten ranges of two partial sums each
    (2, 200, 240, 68, 68, 1),      # the same, added to the first image's
])
def test_winograd_wgrad_with_operands_beyond_the_pieces(case, kind):
    """Mapped values below 2^-110 leave bits over in the split, infinities and NaN show in the sums: such a workgroup works its range again on the fp32
    instruction, over what it has written.  A channel without such a value keeps its gradient.  That instruction rounds eight times a chunk where pieces round once: 88 times in a
    partial sum of eleven chunks.  Measured with pieces 1.40e-6 at 35 and 1.79e-6 at 64 chunks; roundings add in the square, so 2.1e-6 at 88, and 3e-6 is the bound."""
    torch = torch_mod()
    N, H, W, C, K, _ = case
    rng = np.random.default_rng(4)
    x, dy = rng.standard_normal((N, H, W, C), dtype=np.float32), rng.standard_normal((N, H, W, K), dtype=np.float32)
    if kind == "tiny": x *= np.float32(1e-34)
    if kind == "huge": x *= np.float32(1e30)      # x 100 and dy 225 times as large when mapped, sums of 6000 of either sign: up to 1e37 (1e35 would overflow in any order)
    want = wgrad64(x, dy)
    keep = np.ones(C, bool)
    if kind in ("infinity", "nan"):
        x[N - 1, H - 7, W - 11, C - 2] = np.inf if kind == "infinity" else np.nan
        keep[C - 2] = False
    got = wgrad_maps(torch, x, dy, case)
    assert np.linalg.norm(got[..., keep] - want[..., keep]) <= (2e-6 if N * H * W < 1000 else 3e-6) * np.linalg.norm(want[..., keep])
    assert not np.isfinite(got[..., ~keep]).any()


def pieces_operands(kind):
    rng = np.random.default_rng(11)
    N, H, W, C, K = 4, 9, 10, 64, 40
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = rng.standard_normal((K, 3, 3, C), dtype=np.float32) * np.float32(0.05)
    per_c = np.ldexp(np.float32(1), rng.integers(-24, 25, C)).astype(np.float32)
    if kind == "tiny": x *= np.float32(1e-33)
    if kind == "huge": x *= np.float32(1e33)
    if kind == "tiny filters": w *= np.float32(1e-34)
    if kind == "both small": x *= np.float32(1e-18); w *= np.float32(1e-17)
    if kind == "images apart": x *= np.array([1e-25, 1, 1e25, 1e-3], np.float32)[:, None, None, None]
    if kind == "filters apart": w *= np.ldexp(np.float32(1), rng.integers(-80, 60, K)).astype(np.float32)[:, None, None, None]
    if kind == "zero chunk first": x[..., :32] = 0
    if kind == "growing chunks": x *= np.repeat(np.array([1e-9, 1e-3, 1, 1e6], np.float32), 16)
    if kind == "channels apart, filters against": x *= per_c; w /= per_c
    if kind == "zero image": x[1] = 0
    if kind == "zero filters": w[3:9] = 0
    if kind == "sparse": x *= rng.random(x.shape) < 0.002
    if kind == "dominant weight":      # every product but one channel's lies below what the pieces hold, all of one sign
        x[..., 5] *= np.float32(0.92 * 2.0 ** -5)
        x[..., :5], x[..., 6:16], x[..., 16:] = 1, 1, 15.99
        w[...] = 0.999 * 2.0 ** -36
        w[..., 5] = 0
        w[:, 2, 2, 5] = 1
    return x, w


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["plain", "tiny", "huge", "tiny filters", "both small", "images apart", "filters apart", "zero chunk first", "growing chunks",
                                  "channels apart, filters against", "zero image", "zero filters", "sparse", "dominant weight"])
def test_winograd_on_pieces_keeps_the_range_of_fp32(kind):
    """Scales that fp16 pieces cannot hold: every image and every output channel is as close to 64 bits as the fp32 form, whose error
    is relative to the products' sizes: 4e-6 of |x| * |w| for each (image, channel), plus fp32's smallest number per output."""
    torch = torch_mod()
    x, w = pieces_operands(kind)
    N, H, W, C = x.shape
    K = w.shape[0]
    want = winograd64(x, w)
    size = winograd64(np.abs(x), np.abs(w))
    turned = np.ascontiguousarray(w[:, ::-1, ::-1, :].transpose(3, 1, 2, 0))      # x as an output gradient: the same numbers
    for filt, dims, adjoint in ((w, (N, H, W, C, K), 0), (turned, (N, H, W, K, C), 1)):
        out = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
        got = winograd_one_kernel(torch, dev(x), dev(filt), out, dims, adjoint).cpu().numpy().astype(np.float64)
        assert np.isfinite(got).all()
        err = np.linalg.norm((got - want).reshape(N, H * W, K), axis=1)
        bound = 4e-6 * np.linalg.norm(size.reshape(N, H * W, K), axis=1) + 1e-44 * H * W
        assert (err <= bound).all(), (adjoint, (err / bound).max())


@pytest.mark.gpu
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.0e38])
def test_winograd_on_pieces_with_values_beyond_the_pieces(value):
    """An infinity or a NaN stays within the 4x4 tiles whose patch holds it; a value near the largest float gives finite results where the fp32
    form's are finite.  The epilogue with BatchNorm and ReLU runs behind the second pass as behind the first."""
    torch = torch_mod()
    x, w = pieces_operands("plain")
    N, H, W, C = x.shape
    K = w.shape[0]
    if value > 1e38 and np.isfinite(value): w = w * np.float32(1e-3)
    x[2, 4, 5, 40] = value
    out = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
    got = winograd_one_kernel(torch, dev(x), dev(w), out, (N, H, W, C, K), 0).cpu().numpy()
    clean = np.ones((N, H, W), bool)
    clean[2, 4:8, 4:8] = False      # tile rows and columns 4 .. 7 hold pixel (4, 5); its patch reaches one further on each side:
    clean[2, 0:4, 4:8] = False      # row 4 is the last row of the patches of tile rows 0 .. 3
    x[2, 4, 5, 40] = 0
    want = winograd64(x, w)
    assert np.linalg.norm(got[clean] - want[clean]) < 4e-6 * np.linalg.norm(want[clean])
    if not np.isfinite(value): assert not np.isfinite(got[2, 4, 5]).any()
    need = monet.call("monet_conv_winograd_fused_workspace_bytes", N, H, W, C, K, 0)
    ws = torch.empty(need // 4, dtype=torch.float32, device="cuda")
    gamma, beta, stats = (dev(v.astype(np.float32)) for v in (np.linspace(0.5, 1.5, K), np.linspace(-0.1, 0.1, K), np.linspace(0.5, 1.0, 2 * K)))
    x[2, 4, 5, 40] = value
    fused, xd, wd = torch.empty((N, H, W, K), dtype=torch.float32, device="cuda"), dev(x), dev(w)
    monet.call("monet_conv_fwd_bn_apply", None, xd.data_ptr(), wd.data_ptr(), fused.data_ptr(), N, H, W, C, K, 3, 3, 1, 1, 5, ws.data_ptr(), need,
               gamma.data_ptr(), beta.data_ptr(), stats.data_ptr())
    monet.call("monet_bn_apply", None, out.data_ptr(), out.data_ptr(), gamma.data_ptr(), beta.data_ptr(), stats.data_ptr(), N * H * W, K)
    assert torch.equal(torch.nan_to_num(fused), torch.nan_to_num(out))


@pytest.mark.gpu
@pytest.mark.parametrize("C", [64, 256])
@pytest.mark.parametrize("present, factor", [(1.0, 1.0), (0.3, 1.4), (0.1, 1.7), (0.03, 1.7)])
def test_winograd_on_pieces_against_the_fp32_form(C, present, factor):
    """Error against 64 bits beside the fp32 instruction's, which works the same layer with eight channels of zeros more (they change no sum).  Dense operands: the pieces'
    sums have fewer roundings than the fp32 form's and are the closer ones.  Where only a share of the (image, channel) planes is present the fp32 form rounds only their
    products, and the pieces' operands (23 of 24 bits) and three roundings per 16 channels show: measured 1.1 - 1.25 times its error at 30 %, 1.4 - 1.6 times at 10 and 3 %."""
    torch = torch_mod()
    N, H, W, K = 8, 20, 20, 64
    ratios = []
    for seed in range(3):
        rng = np.random.default_rng(seed)
        x = np.maximum(rng.standard_normal((N, H, W, C), dtype=np.float32), 0) * (rng.random((N, 1, 1, C)) < present).astype(np.float32)
        w = rng.standard_normal((K, 3, 3, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (9 * C)))
        want = winograd64(x, w)
        errors = []
        for pad in (0, 8):
            xp, wp = np.pad(x, ((0, 0), (0, 0), (0, 0), (0, pad))), np.pad(w, ((0, 0), (0, 0), (0, 0), (0, pad)))
            out = torch.full((N, H, W, K), float("nan"), dtype=torch.float32, device="cuda")
            errors.append(np.linalg.norm(winograd_one_kernel(torch, dev(xp), dev(wp), out, (N, H, W, C + pad, K), 0).cpu().numpy() - want))
        ratios.append(errors[0] / errors[1])
    assert max(ratios) < factor


def winograd_time(torch, x, w):
    """Microseconds of the one-kernel forward pass."""
    dims = (*x.shape, w.shape[0])
    need = monet.call("monet_conv_winograd_fused_workspace_bytes", *dims, 0)
    ws, out, xd, wd = torch.empty(need // 4, device="cuda"), torch.empty((*x.shape[:3], w.shape[0]), device="cuda"), dev(x), dev(w)
    best = float("inf")
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            monet.call("monet_conv_winograd_fused", torch.cuda.current_stream().cuda_stream, xd.data_ptr(), wd.data_ptr(), out.data_ptr(), *dims, 0, 0, ws.data_ptr(), need)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["zero filters", "small channels first", "channels grow", "few values", "second pass"])
def test_winograd_on_pieces_takes_ordinary_operands_at_full_speed(kind):
    """Operands that a network brings do not send work to the second pass.  Where every part of the launch has to be worked again (the large inputs meet weights of almost
    nothing) it takes about three times as long."""
    torch = torch_mod()
    rng = np.random.default_rng(12)
    x = np.maximum(rng.standard_normal((64, 28, 28, 64), dtype=np.float32), 0)
    w = rng.standard_normal((64, 3, 3, 64), dtype=np.float32) * np.float32(0.05)
    plain = winograd_time(torch, x, w)
    if kind == "zero filters": w[::32] = 0      # one in each half item
    if kind == "small channels first": x[..., :16] *= np.float32(1 / 200)
    if kind == "few values": x *= rng.random(x.shape) < 0.01
    if kind == "second pass":
        x[..., 3] = 1e6
        w[..., 3] *= np.float32(1e-9)
    if kind == "channels grow": x *= np.repeat(np.array([1e-2, 1, 1e2, 1e4], np.float32), 16)
    assert winograd_time(torch, x, w) < (4.5 if kind == "second pass" else 1.4) * plain + 5


@pytest.mark.gpu
def test_winograd_on_pieces_transforms_long_filters_in_proportion():
    """Four times the weights take four times as long, not sixteen times (a workgroup that reads all weights of its channels for every 16 of them)."""
    torch = torch_mod()
    rng = np.random.default_rng(13)

    def time(C):
        return winograd_time(torch, rng.standard_normal((1, 7, 7, C), dtype=np.float32), rng.standard_normal((C, 3, 3, C), dtype=np.float32))

    assert time(2048) < 4.5 * time(1024)


IM2COL_CASES = [
    # N, H, W, C, K, R, stride, pad, chunk images (0: the recommended workspace)
    (2, 16, 16, 16, 16, 3, 1, 1, 0),
    (5, 14, 14, 64, 128, 3, 1, 1, 2),      # three chunks, the last one ragged
    (3, 15, 13, 32, 80, 3, 2, 1, 1),       # stride 2, odd sizes, one image per chunk
    (2, 32, 32, 3, 64, 7, 2, 3, 0),        # stem: 147 floats per patch, padded to 160 (filters padded too)
    (2, 9, 9, 20, 24, 3, 1, 1, 0),         # R*S*C = 180, padded to 192
    (4, 7, 7, 512, 512, 3, 1, 1, 3),
]


@pytest.mark.parametrize("case", IM2COL_CASES)
def test_convolution_through_patch_matrix_matches_oracle(case):
    """Forward (plain and accumulating) and filter gradient of the explicit patch-matrix form against the oracle, with
    the recommended workspace and with workspaces that force several chunks; a workspace below one image is refused."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad, chunk = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    w = (rng.standard_normal((K, R, R, C), dtype=np.float32) * np.float32(np.sqrt(2.0 / (C * R * R))))
    P = (H + 2 * pad - R) // stride + 1
    Q = (W + 2 * pad - R) // stride + 1
    dy = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    y0 = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    xo, wo, dyo = wt.act_to_oracle(x), wt.weight_to_oracle(w), wt.act_to_oracle(dy)
    want_y = wt.act_from_oracle(nm.conv2d_fwd(xo, wo, stride, pad))
    want_w = wt.weight_from_oracle(nm.conv2d_wgrad(xo, dyo, R, R, stride, pad))
    dx, dwt, ddy = dev(x), dev(w), dev(dy)
    ld = -(-(C * R * R) // 16) * 16
    sizes = {}
    for wgrad in (0, 1):
        rec = monet.call("monet_conv_im2col_workspace_bytes", N, H, W, C, K, R, R, stride, pad, wgrad)
        if chunk:       # exactly `chunk` images of patches (+ padded filters / the gradient's tail, taken from the recommendation)
            rec_imgs_bytes = rec - 4 * min(N, max(1, (256 << 20) // 4 // (P * Q * ld))) * P * Q * ld
            rec = 4 * chunk * P * Q * ld + max(rec_imgs_bytes, 0) + (4 * K * ld * 260 if wgrad else 0)
        sizes[wgrad] = rec
    ws = torch.full((max(sizes.values()) // 4 + 64,), float("nan"), dtype=torch.float32, device="cuda")
    y = torch.empty((N, P, Q, K), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_im2col_fwd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, R, R, stride, pad, 0, ws.data_ptr(), sizes[0])
    check_close(y.cpu().numpy(), want_y, ACT_TOL, what="forward")
    yacc = dev(y0)
    monet.call("monet_conv_im2col_fwd", None, dx.data_ptr(), dwt.data_ptr(), yacc.data_ptr(), N, H, W, C, K, R, R, stride, pad, 1, ws.data_ptr(), sizes[0])
    check_close(yacc.cpu().numpy(), want_y + y0, ACT_TOL, what="forward, accumulating")
    ws.fill_(float("nan"))
    dw = torch.full((K, R, R, C), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_im2col_wgrad", None, dx.data_ptr(), ddy.data_ptr(), dw.data_ptr(), N, H, W, C, K, R, R, stride, pad, ws.data_ptr(), sizes[1])
    check_close(dw.cpu().numpy(), want_w, GRAD_TOL, what="filter gradient")
    with pytest.raises(M.MonetError):
        monet.call("monet_conv_im2col_fwd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, C, K, R, R, stride, pad, 0, ws.data_ptr(),
                   4 * (P * Q * ld - 16))


MANY_RANGE_CASES = [
    # N, H, W, C, K, R, stride, pad, splits: reduction ranges of a few steps each, several workgroups per compute unit
    (16, 112, 112, 16, 96, 1, 1, 0, 1792),      # MobileNetV2's first expansion (reduced batch): 7 steps per range, a second table begun
    (16, 112, 112, 16, 96, 1, 1, 0, 3136),      # 4 steps per range: one table, one turn of the pipelined loop
    (16, 112, 112, 16, 96, 1, 1, 0, 12544),     # a single step
    (16, 56, 56, 64, 64, 3, 1, 1, 640),         # padded 3x3: rows of a step straddle image borders; 5 steps
    (64, 14, 14, 256, 256, 3, 1, 1, 96),        # 9 steps: the first table written again while the second is read
    (16, 57, 57, 32, 48, 3, 2, 1, 640),         # stride 2, odd size; 2 steps, empty ranges behind the last
]


@pytest.mark.parametrize("case", MANY_RANGE_CASES)
def test_filter_gradient_with_many_short_ranges_on_every_tile_shape(case):
    """The aligned filter-gradient loader shares tables of output positions (four steps each, two of them in turn) through LDS; this
    runs it with hundreds to thousands of reduction ranges of one to nine steps (several workgroups resident per compute unit, the
    loop entered and left after one or two turns) on every tile shape, against the oracle, twice: the two runs must
    agree bit for bit.  With a forced shape the launch takes the ranges as asked: every one of their partial results is written."""
    torch = torch_mod()
    N, H, W, C, K, R, stride, pad, splits = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    P = (H + 2 * pad - R) // stride + 1
    Q = (W + 2 * pad - R) // stride + 1
    dy = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    want = wt.weight_from_oracle(nm.conv2d_wgrad(wt.act_to_oracle(x), wt.act_to_oracle(dy), R, R, stride, pad))
    dx, ddy = dev(x), dev(dy)
    ws = torch.empty(splits * K * R * R * C, dtype=torch.float32, device="cuda")
    try:
        for cfg in range(6):
            monet.call("monet_conv_force_tile", cfg)
            got = []
            for rep in range(2):
                dw = torch.full((K, R, R, C), float("nan"), dtype=torch.float32, device="cuda")
                ws.fill_(float("nan"))
                monet.call("monet_conv_wgrad", None, dx.data_ptr(), ddy.data_ptr(), dw.data_ptr(), N, H, W, C, K, R, R, stride, pad, splits,
                           ws.data_ptr(), ws.numel() * 4)
                torch.cuda.synchronize()
                got.append(dw.cpu().numpy())
                assert not torch.isnan(ws).any(), (cfg, "fewer ranges than asked")
            assert np.array_equal(got[0], got[1]), (cfg, "two runs differ")
            check_close(got[0], want, 1e-5, what=f"tile shape {cfg}")
    finally:
        monet.call("monet_conv_force_tile", -1)


STEM_CASES = [
    # N, H, W, K, R, stride, pad, splits: the first layers of the five networks at reduced batch, sizes that leave ragged
    # tiles (odd maps, a last row tile with fewer rows, rows no multiple of four floats), rows wider than one tile
    (2, 224, 224, 64, 7, 2, 3, 64),       # ResNet-50 / inception: two output rows per tile
    (2, 224, 224, 32, 3, 2, 1, 64),       # MobileNetV2: one wave per position group
    (2, 224, 224, 64, 3, 1, 1, 64),       # VGG-16: one output row per tile
    (3, 37, 29, 64, 7, 2, 3, 16),
    (3, 37, 29, 32, 3, 2, 1, 7),
    (2, 33, 31, 96, 3, 1, 1, 5),
    (1, 40, 608, 64, 3, 1, 1, 9),         # UNet: rows of 608 positions in segments of 224
    (1, 19, 300, 128, 3, 1, 1, 4),
    (5, 9, 9, 32, 3, 1, 1, 2),
    (1, 7, 5, 64, 7, 2, 3, 2),            # a map smaller than the filter's reach
]


@pytest.mark.parametrize("case", STEM_CASES)
def test_first_layer_forward_and_filter_gradient_from_rows_staged_in_lds(case):
    """Convolutions of a three-channel image through the kernels that stage input rows in LDS: forward pass and filter
    gradient against the oracle, the filter gradient twice (bit-identical), and monet_conv_fwd / monet_conv_wgrad with
    the same arguments give the same bits, i.e. take these forms by themselves."""
    torch = torch_mod()
    N, H, W, K, R, stride, pad, splits = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, 3), dtype=np.float32)
    w = (rng.standard_normal((K, R, R, 3), dtype=np.float32) * np.float32(np.sqrt(2.0 / (3 * R * R))))
    P = (H + 2 * pad - R) // stride + 1
    Q = (W + 2 * pad - R) // stride + 1
    dy = rng.standard_normal((N, P, Q, K), dtype=np.float32)
    xo, wo, dyo = wt.act_to_oracle(x), wt.weight_to_oracle(w), wt.act_to_oracle(dy)
    dx, dwt, ddy = dev(x), dev(w), dev(dy)
    y = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_stem_fwd", None, dx.data_ptr(), dwt.data_ptr(), y.data_ptr(), N, H, W, K, R, R, stride, pad)
    check_close(y.cpu().numpy(), wt.act_from_oracle(nm.conv2d_fwd(xo, wo, stride, pad)), ACT_TOL, what="forward")
    y2 = torch.full((N, P, Q, K), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_conv_fwd", None, dx.data_ptr(), dwt.data_ptr(), y2.data_ptr(), N, H, W, 3, K, R, R, stride, pad, 1, None, 0)
    assert torch.equal(y, y2), "monet_conv_fwd did not take the first-layer form"
    ws = torch.empty(splits * K * R * R * 3, dtype=torch.float32, device="cuda")
    got = []
    for entry in ("monet_conv_stem_wgrad", "monet_conv_stem_wgrad", "monet_conv_wgrad"):
        gw = torch.full((K, R, R, 3), float("nan"), dtype=torch.float32, device="cuda")
        ws.fill_(float("nan"))
        if entry == "monet_conv_wgrad":
            monet.call(entry, None, dx.data_ptr(), ddy.data_ptr(), gw.data_ptr(), N, H, W, 3, K, R, R, stride, pad, splits, ws.data_ptr(), ws.numel() * 4)
        else:
            monet.call(entry, None, dx.data_ptr(), ddy.data_ptr(), gw.data_ptr(), N, H, W, K, R, R, stride, pad, splits, ws.data_ptr(), ws.numel() * 4)
        torch.cuda.synchronize()
        got.append(gw.cpu().numpy())
    assert np.array_equal(got[0], got[1]), "two runs differ"
    assert np.array_equal(got[0], got[2]), "monet_conv_wgrad did not take the first-layer form"
    check_close(got[0], wt.weight_from_oracle(nm.conv2d_wgrad(xo, dyo, R, R, stride, pad)), GRAD_TOL, what="filter gradient")


STEM7_CASES = [(2, 40, 38, 64), (1, 24, 24, 32), (1, 31, 29, 96), (1, 15, 300, 96)]      # N, H, W, K; the last: rows in segments, the last one shorter


@pytest.mark.parametrize("kind", ["finite", "inf", "inf_at_the_edges", "nan", "near_max", "2^-112", "2^-118", "2^-125"])
@pytest.mark.parametrize("case", STEM7_CASES)
def test_first_layer_filter_gradient_of_infinities_and_small_values(case, kind):
    """7x7 / stride 2 filter gradient (bf16 pieces): special values come out as the fp32 products' sums, also in the image's corners
    and beside tile positions that do not exist, the finite results beside them and those of small operands are as precise as ever."""
    torch = torch_mod()
    N, H, W, K = case
    rng = np.random.default_rng(3)
    P, Q = (H - 1) // 2 + 1, (W - 1) // 2 + 1
    x = (np.abs(rng.standard_normal((N, H, W, 3))) + 0.5).astype(np.float32)
    dy = (np.abs(rng.standard_normal((N, P, Q, K))) + 0.5).astype(np.float32)
    unit = 1.0
    if kind == "inf":
        dy[0, 3, 5, 3], x[0, 8, 9, 1] = -np.inf, np.inf
    elif kind == "inf_at_the_edges":
        x[0, 0, 0, 0], x[0, 0, W - 1, 0], x[N - 1, H - 1, 0, 0], x[N - 1, H - 1, W - 1, 0] = (np.inf,) * 4
    elif kind == "nan":
        dy[0, 3, 5, 3], x[0, 8, 9, 1] = np.nan, np.nan
    elif kind == "near_max":      # rounds to infinity in bf16
        dy[0, 3, 5, 3] = 3.4e38
        x[0, 3:10, 7:14] *= 1e-4
    elif kind != "finite":
        small = np.float64(2.0 ** int(kind[2:]))
        dy, x, unit = (dy * small).astype(np.float32), x * np.float32(2.0 ** 60), small * 2.0 ** 60
    pad = np.zeros((N, H + 6, W + 6, 3), np.float64)
    pad[:, 3:3 + H, 3:3 + W] = x
    want = np.empty((K, 7, 7, 3))
    g64 = dy.reshape(-1, K).astype(np.float64)
    with np.errstate(all="ignore"):
        for r in range(7):
            for s in range(7):
                win = pad[:, r:r + 2 * P - 1:2, s:s + 2 * Q - 1:2].reshape(-1, 3)
                want[:, r, s] = (g64[:, :, None] * win[:, None, :]).sum(0)
    splits = 4
    ws = torch.empty(splits * K * 147, device="cuda")
    gx, gd, dw = dev(x), dev(dy), torch.empty((K, 7, 7, 3), device="cuda")
    monet.call("monet_conv_stem_wgrad", None, gx.data_ptr(), gd.data_ptr(), dw.data_ptr(), N, H, W, K, 7, 7, 2, 3, splits, ws.data_ptr(), ws.numel() * 4)
    got, want = dw.cpu().numpy().astype(np.float64) / unit, want / unit
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)]) and np.array_equal(np.isinf(got), np.isinf(want))
    fine = np.isfinite(want)
    # n products of one sign: fp32 sums within n 2^-24 of fp64's, and in the norm, where the roundings do not add up, sqrt(n) 2^-24
    n = N * P * Q
    err = np.abs(got[fine] - want[fine]) / np.abs(want[fine])
    assert err.max() <= n * 2.0 ** -24 and np.sqrt((err ** 2).mean()) <= np.sqrt(n) * 2.0 ** -24, (err.max() * 2.0 ** 24, n)


def test_first_layer_kernels_refuse_what_they_are_not_for():
    torch = torch_mod()
    t = torch.zeros(1 << 20, device="cuda")
    for (N, H, W, K, R, stride, pad) in [
        (1, 32, 32, 48, 3, 1, 1),      # output channels no multiple of 32
        (1, 32, 32, 64, 5, 1, 2),      # 5x5 filter
        (1, 32, 32, 64, 7, 1, 3),      # 7x7 at stride 1
        (1, 32, 32, 160, 3, 1, 1),     # more than four blocks of 32 output channels
    ]:
        with pytest.raises(M.MonetError):
            monet.call("monet_conv_stem_fwd", None, t.data_ptr(), t.data_ptr(), t.data_ptr(), N, H, W, K, R, R, stride, pad)
    with pytest.raises(M.MonetError):      # no partial results asked for
        monet.call("monet_conv_stem_wgrad", None, t.data_ptr(), t.data_ptr(), t.data_ptr(), 1, 32, 32, 64, 3, 3, 1, 1, 1, t.data_ptr(), 1 << 22)
    with pytest.raises(M.MonetError):      # workspace one float short (five tiles of seven output rows: five workgroups)
        monet.call("monet_conv_stem_wgrad", None, t.data_ptr(), t.data_ptr(), t.data_ptr(), 1, 32, 32, 64, 3, 3, 1, 1, 8, t.data_ptr(),
                   5 * 64 * 27 * 4 - 4)


def stem7_64(x, w, pad):
    n, h, wd, _ = x.shape
    P, Q = (h + 2 * pad - 7) // 2 + 1, (wd + 2 * pad - 7) // 2 + 1
    xp = np.pad(x.astype(np.float64), ((0, 0), (pad, pad), (pad, pad), (0, 0)))
    return sum(xp[:, r:r + 2 * P - 1:2, s:s + 2 * Q - 1:2, :] @ w[:, r, s, :].astype(np.float64).T for r in range(7) for s in range(7))


@pytest.mark.gpu
@pytest.mark.parametrize("case, pieces", [
    # N, H, W, K, pad; whether LDS holds the rows in pieces (64 KiB)
    ((1, 7, 7, 32, 0), True),          # one position
    ((2, 9, 40, 64, 3), True),         # whole rows, several in a tile
    ((3, 61, 63, 64, 3), True),        # rows at odd offsets of a 16-byte piece; 224 positions are seven rows of 32
    ((2, 12, 300, 64, 3), True),       # 150 positions in a row: one row a tile
    ((1, 12, 339, 64, 0), True),       # 167
    ((1, 12, 341, 64, 0), False),      # 168
    ((1, 12, 379, 64, 0), False),      # 187 (wider ones are refused: more than eight pieces of 16 bytes per thread)
    ((2, 20, 96, 32, 3), True),        # one block of channels, the last tile two rows of four
    ((2, 65, 65, 96, 2), True),        # three blocks of channels, one group of position blocks
    ((2, 33, 65, 128, 3), True),       # four
    ((1, 20, 117, 128, 3), True),      # two rows of 59 positions
    ((1, 20, 119, 128, 3), False),     # 60
    ((1, 20, 129, 128, 3), True),      # one row of 65
    ((1, 20, 154, 128, 3), True),      # 77 positions in a row, one row a tile
    ((1, 20, 156, 128, 3), False),     # 78
    ((1, 20, 300, 128, 3), False),     # 150: a segment of 128 and one of 22
    ((12, 224, 224, 64, 3), True),     # 672 tiles: some workgroups take two, their waves' groups change places
])
def test_stem_7x7_on_pieces_matches_64_bits(case, pieces):
    """147 products in eleven steps, one rounding each: 7e-8 measured, bound 3e-7 (the fp32 instruction 2.2e-7)."""
    torch = torch_mod()
    N, H, W, K, pad = case
    rng = np.random.default_rng(6)
    x, w = rng.standard_normal((N, H, W, 3), dtype=np.float32), rng.standard_normal((K, 7, 7, 3), dtype=np.float32) * np.float32(0.117)
    want = stem7_64(x, w, pad)
    y = torch.full(want.shape, float("nan"), dtype=torch.float32, device="cuda")
    dx, dw = dev(x), dev(w)
    names = kernels_of(torch, lambda: monet.call("monet_conv_stem_fwd", None, dx.data_ptr(), dw.data_ptr(), y.data_ptr(), N, H, W, K, 7, 7, 2, pad))
    assert any(("stem7_fwd_kernel" if pieces else "stem_fwd_kernel<7, 7, 2>") in k for k in names), names
    got = y.cpu().numpy()
    assert np.linalg.norm(got - want) <= 3e-7 * np.linalg.norm(want)
    assert np.abs(got - want).max() <= 50 * 3e-7 * np.sqrt((want ** 2).mean())


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["tiny image", "tiny filter", "infinity", "nan", "large"])
def test_stem_7x7_with_operands_beyond_the_pieces(kind):
    """Tiles that pieces do not hold go through the fp32 instruction: an infinity or a NaN stays in the windows that hold it (a window's padded third group reaches one pixel
    further, where its filter value is zero), and numbers below 2^-110 or near the largest keep fp32's precision (150 products of up to 5: 1e36 stays finite)."""
    torch = torch_mod()
    N, H, W, K = 2, 31, 45, 64
    rng = np.random.default_rng(7)
    x, w = rng.standard_normal((N, H, W, 3), dtype=np.float32), rng.standard_normal((K, 7, 7, 3), dtype=np.float32) * np.float32(0.117)
    if kind == "tiny image": x *= np.float32(1e-35)
    if kind == "tiny filter": w *= np.float32(1e-35)
    if kind == "large": x *= np.float32(1e36)
    want = stem7_64(x, w, 3)
    hit = np.zeros(want.shape[:3], bool)
    if kind in ("infinity", "nan"):
        x[1, 14, 20, 1] = np.inf if kind == "infinity" else np.nan
        for p in range(want.shape[1]):
            for q in range(want.shape[2]):
                hit[1, p, q] = 0 <= 14 - (2 * p - 3) < 7 and 0 <= 20 - (2 * q - 3) < 7
    y = torch.full(want.shape, float("nan"), dtype=torch.float32, device="cuda")
    dx, dw = dev(x), dev(w)
    monet.call("monet_conv_stem_fwd", None, dx.data_ptr(), dw.data_ptr(), y.data_ptr(), N, H, W, K, 7, 7, 2, 3)
    got = y.cpu().numpy()
    assert np.linalg.norm(got[~hit] - want[~hit]) <= 1e-6 * np.linalg.norm(want[~hit])
    assert not np.isfinite(got[hit]).any()


POINTWISE_WGRAD_CASES = [
    # N, H, W, C, K, splits: the channel pairs of MobileNetV2's expansion / projection layers (each selects another
    # combination of 16-byte and 4-byte loads of the wide side), position counts that leave a ragged tail, workgroups
    # whose share is shorter than one group of 16 positions per wave
    (2, 56, 56, 16, 96, 64),
    (3, 37, 29, 16, 96, 48),
    (2, 56, 56, 96, 24, 64),
    (2, 56, 56, 24, 144, 64),
    (2, 56, 56, 144, 32, 64),
    (2, 56, 56, 32, 192, 64),
    (2, 56, 56, 192, 32, 64),
    (2, 56, 56, 32, 16, 64),
    (1, 33, 31, 24, 144, 8),
    (1, 33, 31, 144, 24, 8),
    (5, 9, 9, 8, 40, 2),
    (4, 75, 75, 16, 96, 300),     # more splits than workgroups: 256 partial results are used
    (1, 17, 16, 12, 4, 4),        # 68 positions per workgroup: one group each for waves 0..3 and a tail of four rows
]


@pytest.mark.parametrize("case", POINTWISE_WGRAD_CASES)
def test_pointwise_filter_gradient_streamed_into_the_matrix_instruction(case):
    """The 1x1 filter gradient with few channels on one side, read straight from memory into the lane layout of the
    matrix instruction: against the oracle, twice (bit-identical), and monet_conv_wgrad with the same arguments must
    give the same bits, i.e. take this form by itself."""
    torch = torch_mod()
    N, H, W, C, K, splits = case
    rng = np.random.default_rng(hash(case) % (2 ** 32))
    x = rng.standard_normal((N, H, W, C), dtype=np.float32)
    dy = rng.standard_normal((N, H, W, K), dtype=np.float32)
    want = wt.weight_from_oracle(nm.conv2d_wgrad(wt.act_to_oracle(x), wt.act_to_oracle(dy), 1, 1, 1, 0))
    dx, ddy = dev(x), dev(dy)
    ws = torch.empty(min(splits, 256) * K * C, dtype=torch.float32, device="cuda")
    got = []
    for entry in ("monet_conv_pointwise_wgrad", "monet_conv_pointwise_wgrad", "monet_conv_wgrad"):
        dw = torch.full((K, 1, 1, C), float("nan"), dtype=torch.float32, device="cuda")
        ws.fill_(float("nan"))
        if entry == "monet_conv_wgrad":
            monet.call(entry, None, dx.data_ptr(), ddy.data_ptr(), dw.data_ptr(), N, H, W, C, K, 1, 1, 1, 0, splits, ws.data_ptr(), ws.numel() * 4)
        else:
            monet.call(entry, None, dx.data_ptr(), ddy.data_ptr(), dw.data_ptr(), N, H, W, C, K, splits, ws.data_ptr(), ws.numel() * 4)
        torch.cuda.synchronize()
        got.append(dw.cpu().numpy())
    assert np.array_equal(got[0], got[1]), "two runs differ"
    assert np.array_equal(got[0], got[2]), "monet_conv_wgrad did not take the pointwise form"
    check_close(got[0], want, 1e-5, what="pointwise filter gradient")


def test_pointwise_filter_gradient_refuses_what_it_is_not_for():
    torch = torch_mod()
    t = torch.zeros(1 << 20, device="cuda")
    for (N, H, W, C, K, splits, ws_bytes) in [
        (2, 56, 56, 64, 64, 16, 1 << 22),      # both sides wider than 32 channels
        (2, 56, 56, 16, 256, 16, 1 << 22),     # wide side beyond 192
        (2, 56, 56, 16, 96, 1, 1 << 22),       # no partial results asked for
        (2, 56, 56, 16, 96, 16, 16 * 96 * 16 * 4 - 4),     # workspace one float short
        (1, 8, 8, 16, 96, 16, 1 << 22),        # fewer than 64 positions per workgroup
        (2, 56, 56, 18, 96, 16, 1 << 22),      # channels not a multiple of four
    ]:
        with pytest.raises(M.MonetError):
            monet.call("monet_conv_pointwise_wgrad", None, t.data_ptr(), t.data_ptr(), t.data_ptr(), N, H, W, C, K, splits, t.data_ptr(), ws_bytes)


def test_conv_wgrad_rejects_small_workspace():
    torch = torch_mod()
    t = torch.zeros(16 * 16 * 16 * 2, device="cuda")
    with pytest.raises(M.MonetError):
        monet.call("monet_conv_wgrad", None, t.data_ptr(), t.data_ptr(), t.data_ptr(), 2, 16, 16, 16, 16, 3, 3, 1, 1, 4, t.data_ptr(), 64)
    with pytest.raises(M.MonetError):
        monet.call("monet_conv_fwd", None, t.data_ptr(), t.data_ptr(), t.data_ptr(), 2, 16, 16, 16, 16, 3, 3, 0, 1, 1, None, 0)
    with pytest.raises(M.MonetError):
        monet.call("monet_conv_fwd", None, t.data_ptr(), t.data_ptr(), t.data_ptr(), 2, 16, 16, 16, 16, 3, 3, 1, 1, 4, t.data_ptr(), 64)


BN_CASES = [(2 * 16 * 16, 16), (3 * 14 * 14, 64), (1000, 256), (77, 2048), (5 * 33 * 31, 128), (4096, 24), (2 * 14 * 14, 320)]


@pytest.mark.parametrize("rows,C", BN_CASES)
def test_batchnorm_matches_oracle(rows, C):
    torch = torch_mod()
    rng = np.random.default_rng(rows * 131 + C)
    x = (rng.standard_normal((rows, C)) * rng.uniform(0.5, 3, C) + rng.standard_normal(C) * 2).astype(np.float32)
    gamma = rng.uniform(0.5, 1.5, C).astype(np.float32)
    beta = (0.1 * rng.standard_normal(C)).astype(np.float32)
    dy = rng.standard_normal((rows, C), dtype=np.float32)
    eps = 1e-5
    # oracle works on N,C,H,W: use N=rows, H=W=1
    xo = x.astype(np.float64).reshape(rows, C, 1, 1)
    dyo = dy.astype(np.float64).reshape(rows, C, 1, 1)
    yo, mean, invstd = nm.bn_fwd(xo, gamma.astype(np.float64), beta.astype(np.float64), eps)
    dxo, dgo, dbo = nm.bn_bwd_from_input(dyo, xo, gamma.astype(np.float64), mean, invstd)
    dx_, dg_, dbeta_, dd = dev(x), dev(gamma), dev(beta), dev(dy)
    scratch = torch.empty(2 << 20, dtype=torch.float32, device="cuda")
    stats = torch.empty(2 * C, dtype=torch.float32, device="cuda")
    monet.call("monet_bn_stats", None, dx_.data_ptr(), stats.data_ptr(), rows, C, eps, scratch.data_ptr(), scratch.numel() * 4)
    st = stats.cpu().numpy()
    assert rel(st[:C], mean) < 1e-5 and rel(st[C:], invstd) < 1e-5
    y = torch.empty_like(dx_)
    monet.call("monet_bn_apply", None, dx_.data_ptr(), y.data_ptr(), dg_.data_ptr(), dbeta_.data_ptr(), stats.data_ptr(), rows, C)
    check_close(y.cpu().numpy(), yo.reshape(rows, C), ACT_TOL)
    # in place
    xin = dx_.clone()
    monet.call("monet_bn_apply", None, xin.data_ptr(), xin.data_ptr(), dg_.data_ptr(), dbeta_.data_ptr(), stats.data_ptr(), rows, C)
    assert torch.equal(xin, y)
    for from_output, t in ((0, dx_), (1, y)):
        gx = torch.full((rows, C), float("nan"), dtype=torch.float32, device="cuda")
        gg = torch.empty(C, dtype=torch.float32, device="cuda")
        gb = torch.empty(C, dtype=torch.float32, device="cuda")
        monet.call("monet_bn_bwd", None, dd.data_ptr(), t.data_ptr(), from_output, dg_.data_ptr(), dbeta_.data_ptr(), stats.data_ptr(),
                   gx.data_ptr(), gg.data_ptr(), gb.data_ptr(), rows, C, 0, scratch.data_ptr(), scratch.numel() * 4)
        check_close(gx.cpu().numpy(), dxo.reshape(rows, C), GRAD_TOL)
        check_close(gg.cpu().numpy(), dgo, GRAD_TOL)
        check_close(gb.cpu().numpy(), dbo, GRAD_TOL)
        monet.call("monet_bn_bwd", None, dd.data_ptr(), t.data_ptr(), from_output, dg_.data_ptr(), dbeta_.data_ptr(), stats.data_ptr(),
                   gx.data_ptr(), gg.data_ptr(), gb.data_ptr(), rows, C, 1, scratch.data_ptr(), scratch.numel() * 4)
        check_close(gx.cpu().numpy(), 2 * dxo.reshape(rows, C), GRAD_TOL)


# edges of the ranges small tensors are cut into: one sweep of 256 16-byte elements per workgroup (64 rows of 16 channels), 512
# workgroups, slabs of two sweeps, the 256th slab; channel groups that are no power of two, and more than 512 of them.  (The backward pass of up to 2048 rows goes through one
# kernel, which leaves the scratch alone.)
@pytest.mark.parametrize("rows,C", [(3, 4), (63, 16), (64, 16), (65, 16), (127, 16), (129, 16), (32767, 16), (32769, 16), (300, 24), (9, 2052),
                                    (2111, 16), (2112, 16), (2113, 16), (4099, 24), (1100, 2052), (8191, 4), (8193, 4)])
@pytest.mark.parametrize("slabs", [1, 3, 1024])
def test_batchnorm_backward_on_small_tensors(rows, C, slabs):
    torch = torch_mod()
    rng = np.random.default_rng(rows * 131 + C)
    x = rng.standard_normal((rows, C), dtype=np.float32)
    gamma = rng.uniform(0.5, 1.5, C).astype(np.float32)
    beta = (0.1 * rng.standard_normal(C)).astype(np.float32)
    dy = rng.standard_normal((rows, C), dtype=np.float32)
    xo, dyo = x.astype(np.float64).reshape(rows, C, 1, 1), dy.astype(np.float64).reshape(rows, C, 1, 1)
    yo, mean, invstd = nm.bn_fwd(xo, gamma.astype(np.float64), beta.astype(np.float64), 1e-5)
    dxo, dgo, dbo = nm.bn_bwd_from_input(dyo, xo, gamma.astype(np.float64), mean, invstd)
    dx_, dg_, db_, dd = dev(x), dev(gamma), dev(beta), dev(dy)
    stats = dev(np.concatenate([mean.ravel(), invstd.ravel()]).astype(np.float32))
    y = torch.full((rows, C), float("nan"), dtype=torch.float32, device="cuda")
    monet.call("monet_bn_apply", None, dx_.data_ptr(), y.data_ptr(), dg_.data_ptr(), db_.data_ptr(), stats.data_ptr(), rows, C)
    check_close(y.cpu().numpy(), yo.reshape(rows, C), ACT_TOL)
    # scratch for `slabs` partial results and the two coefficient vectors, with a guard behind it
    floats = (slabs + 1) * 2 * C
    scratch = torch.full((floats + 64,), -7.0, dtype=torch.float32, device="cuda")
    gx = torch.full((rows, C), float("nan"), dtype=torch.float32, device="cuda")
    gg, gb = torch.empty(C, device="cuda"), torch.empty(C, device="cuda")
    monet.call("monet_bn_bwd", None, dd.data_ptr(), dx_.data_ptr(), 0, dg_.data_ptr(), db_.data_ptr(), stats.data_ptr(),
               gx.data_ptr(), gg.data_ptr(), gb.data_ptr(), rows, C, 0, scratch.data_ptr(), floats * 4)
    check_close(gx.cpu().numpy(), dxo.reshape(rows, C), GRAD_TOL)
    check_close(gg.cpu().numpy(), dgo, GRAD_TOL)
    check_close(gb.cpu().numpy(), dbo, GRAD_TOL)
    assert (scratch[floats:] == -7.0).all()


def test_batchnorm_statistics_with_large_offset():
    """Mean far from zero: a sum-of-squares formulation would lose the variance here."""
    torch = torch_mod()
    rows, C = 200000, 16
    rng = np.random.default_rng(7)
    x = (1000.0 + rng.standard_normal((rows, C))).astype(np.float32)
    mean, invstd = nm.bn_stats(x.astype(np.float64).reshape(rows, C, 1, 1), 1e-5)
    scratch = torch.empty(2 << 20, dtype=torch.float32, device="cuda")
    stats = torch.empty(2 * C, dtype=torch.float32, device="cuda")
    d = dev(x)
    monet.call("monet_bn_stats", None, d.data_ptr(), stats.data_ptr(), rows, C, 1e-5, scratch.data_ptr(), scratch.numel() * 4)
    st = stats.cpu().numpy()
    assert rel(st[:C], mean) < 1e-6 and rel(st[C:], invstd) < 1e-3


@pytest.mark.parametrize("shape", [(2, 16, 16, 16), (1, 5, 7, 3), (3, 9, 11, 40), (1, 1, 1, 64), (1, 1, 1, 1), (2, 33, 17, 130)])
@pytest.mark.parametrize("six", [0, 1])
def test_relu_and_mask_bit_exact(shape, six):
    torch = torch_mod()
    rng = np.random.default_rng(sum(shape) + six)
    x = (rng.standard_normal(shape) * (4 if six else 1)).astype(np.float32)
    flat = x.reshape(-1)
    flat[::7] = 0.0
    if flat.size > 3:
        flat[1] = -0.0
        flat[2] = np.nan
        flat[3] = 6.0
    n = x.size
    words = (n + 63) // 64
    d = dev(x)
    y = torch.empty_like(d)
    mask = torch.full((words + 1,), -1, dtype=torch.int64, device="cuda")     # one guard word
    monet.call("monet_relu_fwd", None, d.data_ptr(), y.data_ptr(), mask.data_ptr(), n, six)
    xo = wt.act_to_oracle(x)
    passes = nm.relu6_pass(xo) if six else nm.relu_pass(xo)
    want_mask = nm.pack_mask(passes)
    got_mask = mask.cpu().numpy().view(np.uint64)
    assert np.array_equal(got_mask[:words], want_mask)          # bit-exact, tail bits zero
    assert got_mask[words] == np.uint64(0xFFFFFFFFFFFFFFFF)     # nothing written past the end
    want_y = wt.act_from_oracle((nm.relu6_fwd if six else nm.relu_fwd)(xo))
    assert np.array_equal(y.cpu().numpy(), want_y.astype(np.float32))
    # in place, without a mask
    z = d.clone()
    monet.call("monet_relu_fwd", None, z.data_ptr(), z.data_ptr(), None, n, six)
    assert torch.equal(z, y)
    # backward: three variants give the same bits
    dz = rng.standard_normal(shape, dtype=np.float32)
    ddz = dev(dz)
    want = wt.act_from_oracle(wt.act_to_oracle(dz) * passes).astype(np.float32)
    for mode, t in ((0, d), (1, y), (2, mask)):
        gx = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_relu_bwd", None, ddz.data_ptr(), t.data_ptr(), mode, gx.data_ptr(), n, six, 0)
        assert np.array_equal(gx.cpu().numpy(), want), mode
        monet.call("monet_relu_bwd", None, ddz.data_ptr(), t.data_ptr(), mode, gx.data_ptr(), n, six, 1)
        assert np.array_equal(gx.cpu().numpy(), want + want), mode


@pytest.mark.parametrize("case", [(2, 16, 16, 8, 3, 2, 1), (1, 9, 7, 4, 2, 2, 0), (2, 12, 12, 64, 3, 2, 1), (1, 5, 5, 4, 3, 1, 1),
                                  (2, 14, 14, 64, 3, 1, 1), (1, 7, 9, 8, 3, 1, 1), (3, 28, 28, 192, 3, 1, 1),
                                  (1, 9, 7, 8, 3, 2, 1), (2, 13, 18, 12, 3, 2, 1), (1, 6, 5, 4, 3, 1, 1)])
def test_maxpool_index_bit_exact(case):
    torch = torch_mod()
    N, H, W, C, k, stride, pad = case
    rng = np.random.default_rng(sum(case))
    x = np.maximum(rng.standard_normal((N, H, W, C)), 0).astype(np.float32)      # post-ReLU: many exact ties at 0
    P = (H + 2 * pad - k) // stride + 1
    Q = (W + 2 * pad - k) // stride + 1
    dy = rng.standard_normal((N, P, Q, C), dtype=np.float32)
    yo, idxo = nm.maxpool_fwd(wt.act_to_oracle(x), k, stride, pad)
    d = dev(x)
    y = torch.empty((N, P, Q, C), dtype=torch.float32, device="cuda")
    idx = torch.empty((N, P, Q, C), dtype=torch.uint8, device="cuda")
    monet.call("monet_maxpool_fwd", None, d.data_ptr(), y.data_ptr(), idx.data_ptr(), N, H, W, C, k, stride, pad)
    assert np.array_equal(idx.cpu().numpy(), wt.act_from_oracle(idxo))
    assert np.array_equal(y.cpu().numpy(), wt.act_from_oracle(yo).astype(np.float32))
    want = wt.act_from_oracle(nm.maxpool_bwd_from_index(wt.act_to_oracle(dy), idxo, (N, C, H, W), k, stride, pad))
    ddy = dev(dy)
    got = {}
    for use_idx in (True, False):
        gx = torch.full((N, H, W, C), float("nan"), dtype=torch.float32, device="cuda")
        monet.call("monet_maxpool_bwd", None, ddy.data_ptr(), d.data_ptr(), idx.data_ptr() if use_idx else None, gx.data_ptr(),
                   N, H, W, C, k, stride, pad, 0)
        assert rel(gx.cpu().numpy(), want) < 1e-6
        got[use_idx] = gx.clone()
        # added to what is there: the same sum once more (doubling is exact)
        monet.call("monet_maxpool_bwd", None, ddy.data_ptr(), d.data_ptr(), idx.data_ptr() if use_idx else None, gx.data_ptr(),
                   N, H, W, C, k, stride, pad, 1)
        assert torch.equal(gx, got[use_idx] + got[use_idx])
    # the kernels that read the stored index (row segments, compile-time windows) add the windows in the general kernel's order
    assert torch.equal(got[True], got[False])
