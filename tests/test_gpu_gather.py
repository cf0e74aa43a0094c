"""Gathered convolutions of diff frames and chunks where their tiles can go
wrong: row counts around a tile and a run-aligned tile step, site runs as
long as the chunk, channel counts that fill no stage or no tile, windows
whose offsets are partly without neighbours, residual rows."""

import numpy as np
import pytest
import torch

import oracle
from parity_util import RTOL, rel, to_dev
from workloads import LayerSpec, NetSpec, random_sparse_video, to_storage

pytestmark = pytest.mark.gpu


def gather_net(c, d, k, s, dtype, H, W, batch):
    rng = np.random.default_rng(c + d)
    kk = (k, k)
    layers = [
        LayerSpec(src=-1, c_in=8, c_out=c, k=(1, 1), p=(0, 0), act=1),
        LayerSpec(src=0, c_in=c, c_out=d, k=kk, s=(s, s),
                  p=(k // 2, k // 2), act=2),
        LayerSpec(src=1, c_in=d, c_out=d, k=(1, 1), p=(0, 0), act=1,
                  residual_src=1),
        LayerSpec(src=2, c_in=d, c_out=24, k=(1, 1), p=(0, 0), act=0)]
    for L in layers:
        L.weight = to_storage(rng.normal(
            0, (L.c_in * L.k[0] * L.k[1]) ** -0.5,
            (L.c_out, L.c_in) + L.k), dtype)
        L.bias = to_storage(rng.normal(0, 0.1, (L.c_out,)), dtype)
    return NetSpec("gather", layers, batch, H, W, 8, dtype)


# (c, d, k, s, H, W, batch, frames, share of the sites that change)
CASES = [
    (24, 40, 1, 1, 1, 1, 1, 3, 1.0),        # one row
    (72, 64, 1, 1, 7, 9, 1, 2, 1.0),        # 63 rows, a ragged stage
    (64, 72, 3, 1, 8, 8, 1, 9, 0.5),        # a tile, a partial channel tile
    (64, 136, 3, 2, 13, 5, 2, 4, 0.3),
    (128, 64, 3, 1, 3, 11, 1, 32, 1.0),     # runs of 32: tiles of one run
    (200, 24, 1, 1, 17, 19, 1, 31, 0.9),
    (512, 64, 3, 1, 5, 6, 1, 3, 0.05),      # split; offsets without rows
    # chunks of the most frames whose runs are never walked and one more,
    # tiles around the rows per run that are; residual layers of whole and
    # of ragged stages; a long reduction
    (64, 72, 3, 1, 13, 9, 1, 6, 1.0),
    (64, 72, 3, 1, 13, 9, 1, 7, 1.0),
    (40, 136, 1, 1, 29, 9, 1, 9, 0.6),
    (64, 64, 3, 1, 23, 7, 1, 12, 0.3),
    (264, 40, 1, 1, 9, 33, 1, 32, 0.2),
]


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_gather(case, dtype):
    from paper_2410_20790_amd import SparseTemNet
    c, d, k, s, H, W, batch, nf, frac = case
    net = gather_net(c, d, k, s, dtype, H, W, batch)
    frames = random_sparse_video(5, nf + 1, batch, H, W, 8, frac, dtype)
    thr = [0.0] * 5
    o = oracle.OracleNet(net.layers, batch, H, W, 8, dtype)
    nets = [SparseTemNet(net.layers, batch, H, W, 8, dtype, max_frames=n)
            for n in (nf, 1)]
    try:
        print("gather", case, dtype, flush=True)
        o.encode_reference(frames[0])
        for g in nets:
            g.encode_reference(to_dev(frames[0], dtype))
        chunk = nets[0].encode_chunk(torch.stack([to_dev(f, dtype)
                                                  for f in frames[1:]]), thr)
        for t in range(nf):
            o.encode_diff(frames[t + 1], thr)
            want = o.last["out"]
            live = nets[1].encode_diff(to_dev(frames[t + 1], dtype), thr)
            assert rel(chunk[t].cpu().numpy(), want) <= RTOL[dtype], t
            assert rel(live.cpu().numpy(), want) <= RTOL[dtype], t
    finally:
        for g in nets:
            g.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_gather_split_order(dtype):
    """A half-precision split is cut from the whole window's stages (64
    columns each), also where a tile's rows (one image row) reach only some
    of its offsets: 3x3 over 256 channels in four parts of nine stages, of
    which the middle row's offsets have stages 12 to 23.  2^28 in stage 12
    swallows the 8s in its part, up to 17."""
    from paper_2410_20790_amd import SparseTemNet
    print("split order", dtype, flush=True)
    W = 40
    vals = np.zeros(36, np.float32)
    vals[15:18] = vals[18:21] = 8, 8, 16
    vals[12], vals[23] = 2.0 ** 28, -2.0 ** 28
    L = LayerSpec(src=-1, c_in=256, c_out=64, k=(3, 3), p=(1, 1), act=0)
    L.weight = np.zeros((64, 256, 3, 3), np.float32)
    for st, v in enumerate(vals):
        L.weight[:, st % 4 * 64, st // 4 // 3, st // 4 % 3] = v / 2 ** 13
    net = SparseTemNet([L], 1, 1, W, 256, dtype)
    try:
        x = torch.zeros((1, 1, W, 256), dtype=net.tdtype, device="cuda")
        net.encode_reference(x)
        out = net.encode_diff(torch.full_like(x, 2.0 ** 13), [0.0, 0.0])
        out = out.cpu().numpy()
    finally:
        net.close()
    assert (out[0, 0, 1:W - 1] == 32).all(), out[0, 0, :, 0]
