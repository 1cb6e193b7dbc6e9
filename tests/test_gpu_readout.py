"""Readout within the launch of the last edge: what a frame call writes is what the view of the OUTPUT site holds afterwards, for
every convolution kernel, window sizes that are no multiple of a tile, frames that update everything, a few pixels, nothing."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [("f32", (16, 16), 3, 1, 33, 21), ("f32", (16, 32), 3, 2, 20, 34), ("f32", (32, 64), 3, 1, 19, 40), ("f32", (64, 16), 1, 1, 7, 9),
         ("f32", (40, 96), 1, 1, 30, 30), ("f32", (16, 32), 5, 1, 18, 18), ("f32", (3, 5), 3, 1, 9, 9),
         ("f16", (64, 64), 3, 1, 31, 45), ("f16", (128, 96), 3, 1, 17, 17), ("f16", (64, 512), 3, 1, 12, 30), ("f16", (32, 64), 3, 2, 30, 26),
         ("f16", (128, 256), 1, 1, 25, 18), ("f16", (32, 32), 3, 1, 24, 40), ("f16", (16, 32), 3, 1, 10, 10), ("f16", (32, 64), 5, 1, 15, 15)]


def check(net, batch=0):
    from gpu_harness import dev
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuBatch, GpuNet
    rng = np.random.default_rng(net.H * 100 + net.W)
    C = net.sites[0].C
    x = rng.normal(0, 1, (net.H, net.W, C)).astype(np.float32)
    frames, shifts = [x], [(0, 0), (0, 0), (0, 0), (0, 1), (-1, 0)]
    for t in range(4):
        x = x.copy()
        if t != 1:
            x[rng.random((net.H, net.W)) < 0.05] += 0.7
        frames.append(x)
    g = GpuBatch(net, batch) if batch else GpuNet(net)
    try:
        for t, (f, (dy, dx)) in enumerate(zip(frames, shifts)):
            fs = [dev((f + 0.1 * b).astype(net.np_dtype)) for b in range(max(batch, 1))]
            outs = g.frame(fs, [dy] * batch, [dx] * batch)[0] if batch else [g.frame(fs[0], dy, dx)[0]]
            torch.cuda.synchronize()
            for b, s in enumerate(g.streams if batch else [g]):
                got = s.split_outputs(outs[b])
                for o, i in zip(got, s.terminals):
                    want = s.read(i, B.MDCNN_VIEW_OUT)
                    assert np.array_equal(o.cpu().numpy().reshape(want.shape), want), f"frame {t} video {b} site {i}"
    finally:
        g.close()


@pytest.mark.parametrize("dtype,chans,k,stride,H,W", CASES)
def test_frame_output_is_the_view(dtype, chans, k, stride, H, W):
    from inputs.nets import tiny_net
    check(tiny_net(dtype, H * stride, W * stride, chans, k=k, stride=stride, theta=0.05, seed=H, total_stride=stride))


@pytest.mark.parametrize("dtype,C,h,w,up", [("f16", 64, 5, 7, 1), ("f16", 128, 6, 9, 2), ("f16", 64, 212, 210, 1), ("f16", 32, 9, 11, 1), ("f32", 64, 9, 11, 1)])
def test_upsampling_edges(dtype, C, h, w, up):
    from inputs.nets import NetSpec, _Builder
    f = 1 << up
    net = NetSpec("up", dtype, h * f, w * f, f)
    b = _Builder(net, np.random.default_rng(C + up), 0.1)
    x, s, y = b.site("in", 8, 1, "input", False, 0.05), b.site("low", C, f, theta=0.02), b.site("out", 32, 1, "output", False, 0.0)
    b.conv(x, s, 3, f)
    b.conv(s, y, 1, 1, pad=0, up=up)
    check(net)


@pytest.mark.parametrize("config,H,W,batch", [(5, 21, 30, 0), (5, 16, 16, 3), (3, 64, 96, 2), (4, 64, 64, 0)])
def test_networks(config, H, W, batch):
    from inputs import build_net
    check(build_net(config, H=H, W=W), batch)


def test_networks_in_turn_on_one_thread():
    """Networks of two to many sites, alone and in a batch, frame by frame in turn: what a call has read out is its own affair."""
    from gpu_harness import dev
    from inputs import build_net
    from inputs.nets import tiny_net
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuBatch, GpuNet
    nets = [build_net(4, H=64, W=64), tiny_net("f16", 31, 45, (64, 64), k=3, stride=1, theta=0.05, seed=1, total_stride=1),
            build_net(5, H=16, W=16), tiny_net("f32", 9, 9, (3, 5), k=3, stride=1, theta=0.05, seed=2, total_stride=1)]
    gs = [GpuNet(nets[0]), GpuNet(nets[1]), GpuBatch(nets[2], 3), GpuNet(nets[3])]
    rng = np.random.default_rng(8)
    try:
        for t in range(3):
            for net, g in zip(nets, gs):
                batch = len(getattr(g, "streams", []))
                fs = [dev(rng.normal(0, 1, (net.H, net.W, net.sites[0].C)).astype(net.np_dtype)) for _ in range(max(batch, 1))]
                outs = g.frame(fs, [0] * batch, [0] * batch)[0] if batch else [g.frame(fs[0], 0, 0)[0]]
                for b, s in enumerate(g.streams if batch else [g]):
                    for o, i in zip(s.split_outputs(outs[b]), s.terminals):
                        want = s.read(i, B.MDCNN_VIEW_OUT)
                        assert np.array_equal(o.cpu().numpy().reshape(want.shape), want), f"frame {t} {net.name} video {b} site {i}"
    finally:
        for g in gs:
            g.close()
