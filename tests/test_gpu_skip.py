"""Residual skips by themselves (calls per layer): channels in pieces of 16 bytes and one by one, views smaller than a block's
pieces, ragged last ones, more pieces than blocks' first turn, ring origins off zero; the lists and marks that go with them."""
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
