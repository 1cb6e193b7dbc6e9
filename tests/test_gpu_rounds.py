"""Independent launches of a frame put together (the default for networks with branches): the same bits as every launch by
itself (MDCNN_OPT_STREAMS = 1), over the tile shapes of the branches, more videos than a launch carries, frames in flight;
and upsampling edges, whose pixels are dealt to several blocks, against the oracle."""
import numpy as np
import pytest
import torch

from inputs import build_net, build_sequence
from inputs.nets import NetSpec, _Builder, random_dag_net
from test_gpu_f32 import frames_of
from test_gpu_streams import run, same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,batch", [(96, 96, 0), (512, 512, 0), (352, 480, 0), (96, 160, 7), (64, 96, 16)])
def test_rounds_do_not_change_a_bit(H, W, batch):
    net, seq = build_net(4, H=H, W=W, blocks=1), build_sequence(4, n_frames=3 if batch else 4, H=H, W=W)
    same(run(net, seq, 1, batch=batch), run(net, seq, 0, batch=batch))


# step 1 of a round asks for its values with the flags up to 512 blocks (one video of 512 x 512: about 480, two of 352 x 480: 620) and after them above
@pytest.mark.parametrize("H,W,batch", [(352, 480, 2), (352, 480, 3)])
def test_rounds_of_many_blocks(H, W, batch):
    net, seq = build_net(4, H=H, W=W, blocks=1), build_sequence(4, n_frames=3, H=H, W=W)
    same(run(net, seq, 1, batch=batch), run(net, seq, 0, batch=batch))


@pytest.mark.parametrize("seed", range(4))
def test_rounds_of_random_networks(seed):
    net = random_dag_net(seed, "f16", n_inner=9)
    class Seq:
        frames = frames_of(net, seed, 4)
        shifts = [(0, 0), (0, 1), (1, 0), (0, 0)]
        forced = None
    same(run(net, Seq, 1), run(net, Seq, 0))


def test_rounds_with_crops_and_frames_in_flight():
    from gpu_harness import dev
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuNet
    net, seq = build_net(4, H=128, W=192, blocks=2), build_sequence(4, n_frames=20, H=128, W=192)
    same(run(net, seq, 1, crops=True), run(net, seq, 0, crops=True))
    frames = [dev(f) for f in seq.frames]
    dy, dx = [int(s[0]) for s in seq.shifts], [int(s[1]) for s in seq.shifts]
    outs = []
    for streams in (1, 0):
        B.mdcnn_set_option(B.MDCNN_OPT_STREAMS, streams)
        g = GpuNet(net)
        try:
            if streams:
                got = [g.frame(f, y, x)[0].clone() for f, y, x in zip(frames, dy, dx)]
            else:
                got = [o.clone() for o in g.frames(frames, dy, dx)[0]]
            torch.cuda.synchronize()
        finally:
            B.mdcnn_set_option(B.MDCNN_OPT_STREAMS, 0)
            g.close()
        outs.append([o.flatten() for o in got])
    assert all(torch.equal(a, b) for a, b in zip(*outs))


@pytest.mark.parametrize("up,cin,cout", [(1, 64, 32), (2, 32, 64), (3, 128, 32), (4, 32, 32), (5, 64, 64)])
def test_upsampling_edges(up, cin, cout):
    import gpu_harness as G
    f = 1 << up
    net = NetSpec("up", "f16", 6 * f, 5 * f, f)
    b = _Builder(net, np.random.default_rng(up), 0.1)
    x, at = b.site("in", 16, 1, "input", False, 0.05), 1
    while at < f:                                  # down in steps of two and four
        step = 2 if (f // at).bit_length() % 2 == 0 else 4
        at *= step
        n = b.site(f"s{at}", cin if at == f else 32, at, theta=0.02)
        b.conv(x, n, step, step, pad=0)
        x = n
    y = b.site("out", cout, 1, "output", False, 0.0)
    b.conv(x, y, 1, 1, pad=0, up=up)
    G.teacher_forced(net, frames_of(net, up), [(0, 0), (0, 1), (0, 0)])
