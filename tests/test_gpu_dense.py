"""The reference pass's dense convolutions against f64, at the edges of their
tiles, stage columns and reduction splits, for every tile shape of the rule
(the tile follows from the output's pixels and channels)."""

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from workloads.nets import LayerSpec, to_storage

pytestmark = pytest.mark.gpu

# (dtype, batch, H, W, c_in, c_out, k, s, p)
CASES = [
    # one pixel; fewer pixels or channels than a 64x64 tile; one more
    ("bf16", 1, 1, 1, 8, 8, 1, 1, 0),
    ("f16", 1, 7, 9, 64, 64, 3, 1, 1),
    ("bf16", 1, 5, 13, 72, 72, 1, 1, 0),
    ("f32", 1, 5, 13, 36, 40, 3, 1, 1),
    # channels below, at and above a stage's columns; strides; 5x5; no pad
    ("f16", 2, 17, 11, 24, 56, 3, 2, 1),
    ("bf16", 1, 20, 23, 128, 24, 3, 1, 0),
    ("bf16", 1, 31, 33, 16, 80, 5, 2, 2),
    ("f32", 2, 19, 21, 16, 64, 3, 2, 1),
    ("f32", 1, 9, 14, 4, 64, 3, 1, 1),
    ("f16", 1, 33, 31, 40, 64, 1, 2, 0),
    # split reductions: few tiles, long, ragged last split
    ("bf16", 1, 6, 11, 512, 136, 3, 1, 1),
    ("f16", 1, 3, 5, 2048, 72, 1, 1, 0),
    ("f32", 1, 8, 8, 200, 72, 3, 1, 1),
    # 128x32, 128x64 (3 and 2 stages) and 128x128 tiles, ragged in pixels
    # and channels
    ("bf16", 1, 169, 170, 32, 24, 1, 1, 0),
    ("f32", 1, 169, 170, 16, 32, 1, 1, 0),
    ("bf16", 1, 169, 171, 64, 64, 3, 1, 1),
    ("f32", 1, 171, 169, 8, 56, 3, 1, 1),
    ("f16", 3, 210, 209, 16, 48, 1, 1, 0),
    ("bf16", 1, 363, 363, 8, 64, 1, 1, 0),
    ("bf16", 1, 171, 169, 128, 120, 1, 1, 0),
    ("f16", 1, 120, 121, 64, 200, 3, 1, 1),
    ("f32", 1, 121, 120, 24, 136, 1, 1, 0),
    # f32 of a little more than two tiles of 128x128 per CU: 128x64
    ("f32", 1, 170, 170, 16, 136, 1, 1, 0),
]


@pytest.mark.parametrize("act", [0, 2])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_dense_convolution(case, act):
    from paper_2410_20790_amd import SparseTemNet
    dtype, n, h, w, cin, cout, k, s, p = case
    print("dense", case, act, flush=True)
    rng = np.random.default_rng(7)
    std = (cin * k * k) ** -0.5
    L = LayerSpec(src=-1, c_in=cin, c_out=cout, k=(k, k), s=(s, s), p=(p, p),
                  act=act)
    L.weight = to_storage(rng.normal(0, std, (cout, cin, k, k)), dtype)
    L.bias = to_storage(rng.normal(0, 1, (cout,)), dtype)
    x = to_storage(rng.normal(0, 1, (n, h, w, cin)), dtype)
    net = SparseTemNet([L], n, h, w, cin, dtype)
    try:
        out = net.encode_reference(
            torch.from_numpy(x).to("cuda", net.tdtype)).cpu().double()
    finally:
        net.close()
    xd = torch.from_numpy(x).double().permute(0, 3, 1, 2)
    wd, bd = (torch.from_numpy(a).double() for a in (L.weight, L.bias))
    want = F.conv2d(xd, wd, bd, s, p)
    # f32 sums of exact products (half) or of rounded ones (f32): at most
    # one rounding of the running sum per term; |f'| <= 1.1 for SiLU
    size = F.conv2d(xd.abs(), wd.abs(), bd.abs(), s, p)
    bound = 1.1 * (2 + cin * k * k) * 2.0 ** -24 * size + 1e-6
    if act:
        want = F.silu(want)
    err = (out.permute(0, 3, 1, 2) - want).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


# (H, W, c_in, c_out, k, parts): parts by blocks of their own (1 and 96 tiles
# of 64x64; f32: every case of 4 parts, which then are 8), then by the block
# itself for every tile shape (64x64, 128x64, 128x128, 128x32), ragged in
# pixels
ORDER_CASES = [
    (7, 9, 2048, 40, 1, 4),
    (62, 99, 2048, 64, 1, 4),
    (64, 128, 2048, 56, 1, 4),
    (43, 190, 256, 64, 3, 4),
    (79, 121, 2048, 256, 1, 2),
    (85, 85, 256, 512, 3, 2),
    (129, 254, 2048, 32, 1, 2),
]


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("case", ORDER_CASES,
                         ids=lambda c: "-".join(map(str, c)))
def test_dense_sum_order(case, dtype):
    """A long reduction is the sum, in order, of its parts' sums (as the
    split of a diff frame adds them).  A stage (128 bytes of the reduction's
    columns) has one product: 2^28 in the first, -2^28 in the last, 8
    in some between, which 2^28 swallows and a part without it keeps (as
    multiples of 32, so that no sum is a tie of its rounding)."""
    from paper_2410_20790_amd import SparseTemNet
    h, w, cin, cout, k, parts = case
    print("order", case, dtype, flush=True)
    kc = 32 if dtype == "f32" else 64
    nst, spk = cin * k * k // kc, cin // kc
    if dtype == "f32" and parts == 4:
        parts = 8
    vals = np.zeros(nst, np.float32)
    for j in range(1, parts):
        at = j * nst // parts
        vals[at:at + (4 if j == parts - 1 else 8)] = 8
    vals[0], vals[-1] = 2.0 ** 28, -2.0 ** 28
    L = LayerSpec(src=-1, c_in=cin, c_out=cout, k=(k, k), s=(1, 1),
                  p=(k // 2, k // 2), act=0)
    L.weight = np.zeros((cout, cin, k, k), np.float32)
    for st, v in enumerate(vals):
        o = st // spk
        L.weight[:, st % spk * kc, o // k, o % k] = v / 2 ** 13
    net = SparseTemNet([L], 1, h, w, cin, dtype)
    try:
        x = torch.full((1, h, w, cin), 2.0 ** 13, dtype=net.tdtype,
                       device="cuda")
        out = net.encode_reference(x).cpu().numpy()
    finally:
        net.close()
    want = vals[1:-1].sum()  # (one chain would give 0)
    m = k // 2  # the pixels whose windows lie inside
    assert (out[0, m:h - m, m:w - m] == want).all(), (out[0, m, m, 0], want)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("option", ["carry", "se"])
def test_stem_sum_order(option, dtype):
    """With residual carry or squeeze-excitation a 7x7/2 stem's states are
    summed in the order of its diff frames: a reference frame leaves them bit
    for bit as a diff frame from zeros does."""
    from paper_2410_20790_amd import SparseTemNet
    from paper_2410_20790_amd import binding as B
    print("stem", option, dtype, flush=True)
    rng = np.random.default_rng(13)
    layers = [LayerSpec(src=-1, c_in=3, c_out=40, k=(7, 7), s=(2, 2),
                        p=(3, 3), act=1),
              LayerSpec(src=0, c_in=40, c_out=8, k=(1, 1), s=(1, 1),
                        p=(0, 0), act=2, se_mid=4 * (option == "se"))]
    for L in layers:
        n = L.c_in * L.k[0] ** 2
        L.weight = to_storage(rng.normal(0, n ** -0.5,
                                         (L.c_out, L.c_in) + L.k), dtype)
        L.bias = to_storage(rng.normal(0, 1, (L.c_out,)), dtype)
        if L.se_mid:
            for name, shape in (("se_w1", (4, 8)), ("se_b1", (4,)),
                                ("se_w2", (8, 4)), ("se_b2", (8,))):
                setattr(L, name, to_storage(rng.normal(0, 1, shape), dtype))
    x = to_storage(rng.normal(0, 1, (2, 33, 141, 3)), dtype)
    net = SparseTemNet(layers, 2, 33, 141, 3, dtype, carry=option == "carry")
    try:
        x = torch.from_numpy(x).to("cuda", net.tdtype)
        net.encode_reference(x)
        ref = B.st_debug_state(net.handle, 0, (2, 17, 71, 40))
        net.encode_reference(torch.zeros_like(x))
        net.encode_diff(x, [0.0] * 3)
        diff = B.st_debug_state(net.handle, 0, (2, 17, 71, 40))
    finally:
        net.close()
    assert np.array_equal(ref, diff)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("hw", [(9, 7), (169, 170)])
def test_dense_residual(dtype, hw):
    """A residual row added before the activation, on the smallest and a
    larger tile: every emitted row of the first layer is its rounded
    activation, so the second layer's sum is known from it."""
    from paper_2410_20790_amd import SparseTemNet
    from paper_2410_20790_amd import binding as B
    h, w = hw
    rng = np.random.default_rng(11)
    layers = []
    for src, cin, res in ((-1, 8, -2), (0, 40, 0)):
        L = LayerSpec(src=src, c_in=cin, c_out=40, k=(1, 1), s=(1, 1),
                      p=(0, 0), act=1, residual_src=res)
        L.weight = to_storage(rng.normal(0, cin ** -0.5, (40, cin, 1, 1)),
                              dtype)
        L.bias = to_storage(rng.normal(0, 1, (40,)), dtype)
        layers.append(L)
    x = to_storage(rng.normal(0, 1, (1, h, w, 8)), dtype)
    net = SparseTemNet(layers, 1, h, w, 8, dtype)
    try:
        out = net.encode_reference(
            torch.from_numpy(x).to("cuda", net.tdtype)).cpu().double()
        p0 = torch.from_numpy(B.st_debug_state(net.handle, 0,
                                               (1, h, w, 40)))
    finally:
        net.close()
    row = p0.clamp(min=0).to(net.tdtype).double().permute(0, 3, 1, 2)
    wd, bd = (torch.from_numpy(a).double()
              for a in (layers[1].weight, layers[1].bias))
    want = F.relu(F.conv2d(row, wd, bd) + row)
    size = F.conv2d(row.abs(), wd.abs(), bd.abs()) + row.abs()
    err = (out.permute(0, 3, 1, 2) - want).abs()
    assert bool((err <= 44 * 2.0 ** -24 * size + 1e-6).all())


# (dtype, batch, H, W, C, k, s, se_mid): channels below, at and past the
# vectors a block's threads share (65 of them: a ragged second block row),
# widths around a strip's four pixels, one pixel, both windows and strides,
# more images than a launch has grid rows
DW_CASES = [
    ("bf16", 1, 1, 1, 8, 3, 1, 0),
    ("f16", 2, 5, 3, 24, 5, 1, 3),
    ("f32", 1, 9, 13, 40, 3, 2, 5),
    ("bf16", 3, 12, 17, 144, 5, 2, 6),
    ("f16", 1, 33, 34, 520, 3, 1, 8),
    ("f32", 2, 7, 9, 1152, 5, 1, 48),
    ("bf16", 1, 70, 131, 32, 3, 1, 8),
    ("f32", 1, 11, 12, 16, 5, 2, 0),
    ("bf16", 65536, 1, 2, 8, 3, 1, 0),
    # many small maps: by rows, or from a share of a tile on by patches
    ("f16", 120, 3, 4, 136, 3, 1, 0),
    ("f32", 60, 6, 5, 152, 5, 1, 4),
    ("bf16", 90, 9, 8, 64, 5, 2, 0),
    ("f32", 70, 16, 15, 72, 3, 2, 0),
]


@pytest.mark.parametrize("case", DW_CASES,
                         ids=lambda c: "-".join(map(str, c)))
def test_dense_depthwise(case):
    from paper_2410_20790_amd import SparseTemNet
    dtype, n, h, w, c, k, s, mid = case
    print("depthwise", case, flush=True)
    rng = np.random.default_rng(5)
    L = LayerSpec(src=-1, c_in=c, c_out=c, k=(k, k), s=(s, s),
                  p=(k // 2, k // 2), groups=c, act=2, se_mid=mid)
    L.weight = to_storage(rng.normal(0, 1 / k, (c, 1, k, k)), dtype)
    L.bias = to_storage(rng.normal(0, 1, (c,)), dtype)
    if mid:
        L.se_w1 = to_storage(rng.normal(0, c ** -0.5, (mid, c)), dtype)
        L.se_b1 = to_storage(rng.normal(0, 0.1, (mid,)), dtype)
        L.se_w2 = to_storage(rng.normal(0, mid ** -0.5, (c, mid)), dtype)
        L.se_b2 = to_storage(rng.normal(0, 1, (c,)), dtype)
    x = to_storage(rng.normal(0, 1, (n, h, w, c)), dtype)
    net = SparseTemNet([L], n, h, w, c, dtype)
    try:
        out = net.encode_reference(
            torch.from_numpy(x).to("cuda", net.tdtype)).cpu().double()
    finally:
        net.close()

    def t(a):
        return torch.from_numpy(a).double()
    xd = t(x).permute(0, 3, 1, 2)
    pre = F.conv2d(xd, t(L.weight), t(L.bias), s, k // 2, 1, c)
    size = F.conv2d(xd.abs(), t(L.weight).abs(), t(L.bias).abs(), s, k // 2,
                    1, c)
    want = F.silu(pre)
    # as test_dense_convolution; the gate is within f32 roundings of sums
    # over at most 10^4 sites and 1152 channels, relative to their size
    bound = 1.1 * (2 + k * k) * 2.0 ** -24 * size + 1e-6
    if mid:
        z = F.silu(want.mean((2, 3)) @ t(L.se_w1).T + t(L.se_b1))
        g = torch.sigmoid(z @ t(L.se_w2).T + t(L.se_b2))[:, :, None, None]
        want = want * g
        bound = bound + 2e-5 * (want.abs() + 1e-2)
    err = (out.permute(0, 3, 1, 2) - want).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("kind", ["se", "se_carry", "se_frozen", "carry"])
def test_reference_artefacts(kind):
    """What the queries see after a reference frame, also after diff frames
    left other lists: every pixel a kept candidate, the geometry's rulebook,
    the rounded activations as rows and (residual carry) as views."""
    from paper_2410_20790_amd import SparseTemNet
    from paper_2410_20790_amd import binding as B
    from parity_util import to_dev
    from workloads import (efficientnet_mini_net, random_sparse_video,
                           resnet_mini_net)
    net = (resnet_mini_net if kind == "carry" else efficientnet_mini_net)(
        dtype="f16")
    frames = random_sparse_video(3, 2, 1, net.H, net.W, 3, 0.1, "f16")
    g = SparseTemNet(net.layers, 1, net.H, net.W, 3, "f16",
                     carry="carry" in kind, frozen_se=kind == "se_frozen")
    try:
        g.encode_reference(to_dev(frames[0], "f16"))
        g.encode_diff(to_dev(frames[1], "f16"), [0.0] * (g.n_layers + 1))
        g.encode_reference(to_dev(frames[1], "f16"))
        shape = {-1: g.in_shape[1:3]}
        for i, L in enumerate(net.layers):
            _, H, W, C = g.tensor_shape(i)
            shape[i] = (H, W)
            every = np.arange(H * W)
            pix, rows = B.st_debug_candidates(g.handle, i, C)
            np.testing.assert_array_equal(pix, every)
            np.testing.assert_array_equal(B.st_debug_active(g.handle, i),
                                          every)
            hi, wi = shape[L.src]
            ho = (hi + 2 * L.p[0] - L.k[0]) // L.s[0] + 1
            wo = (wi + 2 * L.p[1] - L.k[1]) // L.s[1] + 1
            want = [(k, iy * wi + ix, oy * wo + ox)
                    for k in range(L.k[0] * L.k[1])
                    for oy in range(ho) for ox in range(wo)
                    for iy in [oy * L.s[0] - L.p[0] + k // L.k[1]]
                    for ix in [ox * L.s[1] - L.p[1] + k % L.k[1]]
                    if 0 <= iy < hi and 0 <= ix < wi]
            got = B.st_debug_rulebook(g.handle, i)
            np.testing.assert_array_equal(np.asarray(got, np.int64),
                                          np.asarray(want, np.int64))
            if L.act == 1 and not L.pool_k[0] and i + 1 < g.n_layers:
                P = B.st_debug_state(g.handle, i, (1, H, W, C))
                np.testing.assert_array_equal(
                    rows, to_storage(np.maximum(P, 0), "f16").reshape(-1, C))
            if "carry" in kind:
                V = B.st_debug_carry(g.handle, i, (1, H, W, C))
                np.testing.assert_array_equal(V.reshape(-1, C), rows)
    finally:
        g.close()
