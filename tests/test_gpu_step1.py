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


@pytest.mark.parametrize("form", ["plain", "masked", "crops", "masked crops"])
@pytest.mark.parametrize("config,H,W,videos", [(5, 128, 128, 3), (4, 512, 512, 10)])
def test_launches_of_many_blocks(config, H, W, videos, form):
    """A video of a batch whose step-1 launches have more blocks than kAheadBlocks (6144 of one site, 4480 of several together) gives the bits
    it gives alone, where they have fewer: masks, residual skips, crops, camera shifts, frames that change nothing."""
    import gpu_harness as H_
    import torch
    from inputs import build_net
    from paper_2210_09887_amd.runtime import GpuBatch, GpuNet
    net = build_net(config, H=H, W=W)
    for s in net.sites:
        s.theta = s.theta or 0.05
    masked, crops = "masked" in form, "crops" in form
    rng = np.random.default_rng(config)
    x = rng.normal(0, 1, (H, W, net.sites[0].C)).astype(np.float32)
    T = net.total_stride
    one, many = GpuNet(net, crops=crops), GpuBatch(net, videos, crops=crops)
    try:
        for t, (dy, dx) in enumerate([(0, 0), (0, 0), (1, -1), (0, 0)]):
            if t != 3:
                x = x.copy()
                x[rng.random((H, W)) < 0.1] += 0.5
            box = (H // T // 4, t, H // T // 2, W // T - 4) if crops else (0, 0, H // T, W // T)
            cut = lambda a: H_.cut(net, a, box)
            f = H_.dev(cut(x.astype(net.np_dtype)))
            m = H_.dev(cut((rng.random((H, W)) < 0.3).astype(np.uint8))) if masked else None
            if crops:
                want = one.frame_crop(f, dy, dx, box, m)[0]
                got = many.frame_crop([f] * videos, [dy] * videos, [dx] * videos, [box] * videos, [m] * videos if masked else None)[0]
            else:
                want = [one.frame(f, dy, dx, m)[0]]
                got = [[o] for o in many.frame([f] * videos, [dy] * videos, [dx] * videos, [m] * videos if masked else None)[0]]
            torch.cuda.synchronize()
            for v, g in enumerate(got):
                assert all(torch.equal(a.reshape(-1), b.reshape(-1)) for a, b in zip(g, want)), f"frame {t}, video {v}"
    finally:
        one.close()
        many.close()
