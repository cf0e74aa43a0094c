"""Frames whose pixels are whole 16-byte vectors (read as vectors) and frames
that are not, or do not start on one: same kept lists, rows and outputs."""

import numpy as np
import pytest
import torch

from workloads import LayerSpec, random_sparse_video, to_storage

pytestmark = pytest.mark.gpu


def on_device(a, tdtype, shift):
    """A contiguous device tensor that starts `shift` elements past an
    aligned address."""
    t = torch.from_numpy(np.ascontiguousarray(a)).to(tdtype)
    buf = torch.empty(t.numel() + shift, dtype=tdtype, device="cuda")
    out = buf[shift:].view(t.shape)
    out.copy_(t)
    assert out.is_contiguous()
    return out


@pytest.mark.parametrize("dtype,C", [("f32", 4), ("f32", 8), ("f32", 16),
                                     ("f32", 5), ("f16", 4), ("f16", 8),
                                     ("f16", 16), ("bf16", 16)])
def test_frame_alignment(dtype, C):
    from paper_2410_20790_amd import SparseTemNet
    from paper_2410_20790_amd import binding as B
    rng = np.random.default_rng(3)
    L = LayerSpec(src=-1, c_in=C, c_out=16, k=(3, 3), act=0)
    L.weight = to_storage(rng.normal(0, 0.2, (16, C, 3, 3)), dtype)
    L.bias = to_storage(rng.normal(0, 0.2, (16,)), dtype)
    frames = np.stack(random_sparse_video(9, 4, 2, 7, 9, C, 0.3, dtype))
    got = []
    for shift in (0, 1):
        net = SparseTemNet([L], 2, 7, 9, C, dtype, max_frames=3)
        try:
            print("frames", dtype, C, shift, flush=True)
            x = on_device(frames, net.tdtype, shift)
            ref = net.encode_reference(x[0]).cpu()
            out = net.encode_chunk(x[1:], [0.05, 0.0]).cpu()
            pix, rows = B.st_debug_candidates(net.handle, -1, C)
            again = net.encode_chunk(x[1:], [0.05, 0.0]).cpu()
            got.append((ref, out, again, torch.from_numpy(pix),
                        torch.from_numpy(rows)))
        finally:
            net.close()
    # the rows are the frames' differences to the last kept value
    n = 2 * 7 * 9
    kept = np.sort(got[0][3].numpy())
    xh = frames[0].reshape(n, C).copy()
    want = []
    for t in (1, 2, 3):
        f = frames[t].reshape(n, C)
        keep = np.abs(f - xh).max(axis=1) > np.float32(0.05)
        want += [(t - 1) * n + p for p in np.flatnonzero(keep)]
        xh[keep] = f[keep]
    np.testing.assert_array_equal(kept, want)
    for a, b in zip(*got):
        assert torch.equal(a, b)
