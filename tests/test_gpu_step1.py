"""The update mask of a pixel is decided by its largest channel, wherever among the lanes that share the pixel it lies: all numbers
of lanes per pixel, one channel of a pixel past the threshold, the others just below it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,C", [("f16", 8 << k) for k in range(8)] + [("f16", 24)] + [("f32", 4 << k) for k in range(8)])
def test_any_channel_decides(dtype, C):
    import gpu_harness as H_
    from inputs.nets import tiny_net
    H, W = 9, 13
    net = tiny_net(dtype, H, W, (C, 8), k=1, theta=0.5, seed=C, total_stride=1)
    rng = np.random.default_rng(C)
    x = rng.normal(0, 1, (H, W, C)).astype(np.float32)
    frames = [x]
    for t in range(3):
        x = x + rng.uniform(-0.2, 0.2, x.shape).astype(np.float32) * 0.5
        hit = np.argwhere(rng.random((H, W)) < 0.5)
        for k, (r, c) in enumerate(hit):
            x[r, c, (k * 7 + t * 3) % C] += 2.0
        frames.append(x)
    H_.teacher_forced(net, [f.astype(net.np_dtype) for f in frames], [(0, 0)] * 3 + [(1, -1)])
