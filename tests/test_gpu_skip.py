"""Residual skips by themselves (calls per layer): channels in pieces of 16 bytes and one by one, views smaller than a block's
pieces, ragged last ones, ring origins off zero; the lists and marks that go with them.  More pieces than the launch has threads."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,C,H,W", [("f16", 8, 1, 1), ("f16", 24, 7, 5), ("f16", 5, 9, 14), ("f16", 512, 10, 14), ("f32", 4, 3, 2),
                                         ("f32", 7, 12, 11), ("f32", 36, 17, 31), ("f16", 12, 40, 66)])
def test_skip(dtype, C, H, W):
    import gpu_harness as H_
    from inputs.nets import NetSpec, _Builder
    net = NetSpec("skip", dtype, H, W, 1)
    b = _Builder(net, np.random.default_rng(C + H), 0.1)
    x, y, z = b.site("in", C, 1, "input", False, 0.05), b.site("mid", C, 1, "preact", True, 0.05), b.site("out", C, 1, "output", False, 0.0)
    b.identity(x, y)
    b.conv(x, y, 1, 1)
    b.identity(y, z)
    rng = np.random.default_rng(H * 100 + W)
    f = rng.normal(0, 1, (H, W, C)).astype(np.float32)
    frames = [f.astype(net.np_dtype)]
    for _ in range(3):
        f = f.copy()
        f[rng.random((H, W)) < 0.3] += 0.5
        frames.append(f.astype(net.np_dtype))
    H_.teacher_forced(net, frames, [(0, 0), (0, 0), (1, 0), (0, -1)])


def test_more_pieces_than_the_launch_has_threads():
    """65536 blocks of 256 pieces are the most a launch has: 12 channels one by one on 1201 x 1184 pixels are 17.1 million.  Whole
    numbers, so that every sum is exact: what is read out is the frame."""
    import gpu_harness as H_
    import torch
    from inputs.nets import NetSpec, _Builder
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuNet
    H, W, C = 1201, 1184, 12
    assert H * W * C > 65536 * 256
    net = NetSpec("skip", "f16", H, W, 1)
    b = _Builder(net, np.random.default_rng(0), 0.0)
    b.identity(b.site("in", C, 1, "input", False, 0.0), b.site("out", C, 1, "output", False, 0.0))
    rng = np.random.default_rng(3)
    f = rng.integers(-8, 9, (H, W, C)).astype(np.float16)
    g = GpuNet(net)
    try:
        for t, (dy, dx) in enumerate([(0, 0), (0, 0), (1, 0)]):
            if t:
                f = f.copy()
                f[rng.random((H, W)) < 0.01] += 3
                f[-3:, -70:] -= 2
            g.shift_camera(dy, dx)
            g.layer_forward(0, H_.dev(f))
            torch.cuda.synchronize()
            assert np.array_equal(g.read(1, B.MDCNN_VIEW_OUT).reshape(H, W, C), f), f"frame {t}"
    finally:
        g.close()
