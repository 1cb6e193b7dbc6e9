"""The blocks that publish the by-products of a 3 x 3 edge (source list, compute list, touched marks) read three flags of a row
as one word: windows narrower than a word, rows that end inside one, borders wider than the footprint, strides, the first and
last flags of a site."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(1, 1), (1, 5), (2, 3), (7, 1), (3, 2), (5, 64), (17, 31), (40, 66)])
@pytest.mark.parametrize("chans,stride", [((32, 32, 32), 1), ((3, 32), 1), ((3, 32), 2)])
def test_lists_and_marks_of_narrow_windows(H, W, chans, stride):
    import gpu_harness as H_
    from inputs.nets import tiny_net
    H, W = H * stride, W * stride
    net = tiny_net("f16", H, W, chans, k=3, stride=stride, theta=0.05, seed=H + W, total_stride=stride)
    rng = np.random.default_rng(H * 100 + W)
    x = rng.normal(0, 1, (H, W, chans[0])).astype(np.float32)
    frames = [x.astype(np.float16)]
    for _ in range(3):
        x = x.copy()
        x[rng.random((H, W)) < 0.2] += 0.5
        frames.append(x.astype(np.float16))
    H_.teacher_forced(net, frames, [(0, 0), (0, 0), (1, 0), (0, -1)])
