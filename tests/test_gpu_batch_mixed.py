"""Videos of one batch that differ in what networks of equal shape may differ in: every video still gives the bits it
gives alone, with launches shared by several sites and videos (a network with parallel branches)."""
import copy
from dataclasses import replace

import numpy as np
import pytest
import torch

from inputs import build_net, build_sequence

pytestmark = pytest.mark.gpu

N_FRAMES = 5


def network():
    return build_net(4, H=128, W=96, widths=(32, 64, 64, 128), blocks=1)


def with_thresholds(net, factor):
    net = copy.copy(net)
    net.sites = [replace(s, theta=s.theta * factor) for s in net.sites]
    return net


def run_alone_and_together(specs, entry, make=None):
    """Per video its outputs and state from single calls, then from the batch call `entry` ('frame', 'frames', 'crop')."""
    import gpu_harness as H
    from paper_2210_09887_amd.runtime import GpuBatch, GpuNet
    from test_gpu_crops import rand_crops
    from test_gpu_frames import state_of
    make = make or (lambda b, spec, **kw: GpuNet(spec, **kw))
    net, n = specs[0], len(specs)
    seq = build_sequence(4, n_frames=N_FRAMES + n, H=net.H, W=net.W)
    X = [[seq.frames[b + t] for t in range(N_FRAMES)] for b in range(n)]
    path = [[(0, 0), (0, 1), (0, 0), (1, 0), (0, 0)]] * n
    crops = [rand_crops(net, N_FRAMES, 10 + b, full_first=False) if entry == "crop" else None for b in range(n)]

    def videos():
        gs = []
        for b, spec in enumerate(specs):
            g = make(b, spec, crops=entry == "crop", share_weights=gs[0] if gs else None)
            gs.append(g)
        return gs

    def result(gs, outs):
        torch.cuda.synchronize()
        got = [[o.cpu().numpy().copy() for o in row] for row in outs], [state_of(g, net) for g in gs]
        for g in reversed(gs):
            g.close()
        return got

    gs, outs = videos(), []
    for b, g in enumerate(gs):
        row = []
        for t in range(N_FRAMES):
            if entry == "crop":
                o = torch.cat([x.flatten() for x in g.frame_crop(H.dev(H.cut(net, X[b][t], crops[b][t])), *path[b][t], crops[b][t])[0]])
            else:
                o = g.frame(H.dev(X[b][t]), *path[b][t])[0].clone()
            row.append(o)
        outs.append(row)
    alone = result(gs, outs)

    gs = videos()
    gb = GpuBatch.__new__(GpuBatch)
    gb.streams = gs
    dys, dxs = [[[path[b][t][a] for b in range(n)] for t in range(N_FRAMES)] for a in (0, 1)]
    if entry == "frames":
        per_frame = gb.frames([[H.dev(X[b][t]) for b in range(n)] for t in range(N_FRAMES)], dys, dxs)[0]
    else:
        per_frame = []
        for t in range(N_FRAMES):
            if entry == "crop":
                o = gb.frame_crop([H.dev(H.cut(net, X[b][t], crops[b][t])) for b in range(n)], dys[t], dxs[t], [crops[b][t] for b in range(n)])[0]
                per_frame.append([torch.cat([x.flatten() for x in row]) for row in o])
            else:
                per_frame.append([o.clone() for o in gb.frame([H.dev(X[b][t]) for b in range(n)], dys[t], dxs[t])[0]])
    return alone, result(gs, [[per_frame[t][b] for t in range(N_FRAMES)] for b in range(n)])


def same(alone, together):
    for b, (u, v) in enumerate(zip(alone[0], together[0])):
        for t, (x, y) in enumerate(zip(u, v)):
            assert np.array_equal(x, y), f"video {b}, frame {t}: output differs"
    for b, (u, v) in enumerate(zip(alone[1], together[1])):
        for k, (x, y) in enumerate(zip(u, v)):
            assert np.array_equal(x, y), f"video {b}: state view {k} differs"


@pytest.mark.parametrize("entry", ["frame", "frames", "crop"])
def test_a_threshold_per_video(entry):
    net = network()
    alone, together = run_alone_and_together([with_thresholds(net, f) for f in (1.0, 0.25, 4.0)], entry)
    assert any(not np.array_equal(x, y) for x, y in zip(alone[1][0], alone[1][1]))      # the thresholds matter
    same(alone, together)


@pytest.mark.parametrize("keeping", [(0, 2), (1,)])
def test_pooling_output_kept_by_some_of_the_videos(keeping, monkeypatch):
    """Sites that keep a previous pooling output (here without a pooling edge) have their crop state further back in their
    memory: every video's own offset counts."""
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuNet
    nbytes = B.mdcnn_buffer_bytes
    net = network()
    sizes = []

    def make(b, spec, **kw):
        def sized(d):
            if d.kind == B.MDCNN_SITE_PREACT:
                d.pool_prev = int(b in keeping)
            return nbytes(d)
        with monkeypatch.context() as m:
            m.setattr(B, "mdcnn_buffer_bytes", sized)
            g = GpuNet(spec, **kw)
        sizes.append(sum(t.numel() for t in g.mem))
        return g

    alone, together = run_alone_and_together([net] * 3, "crop", make)
    assert len(set(sizes)) == 2                             # the layouts do differ
    same(alone, together)


@pytest.mark.parametrize("entry", ["frame", "frames"])
def test_weights_of_their_own(entry):
    """Videos that do not share their weights (the second runs another model of the same shape)."""
    from paper_2210_09887_amd.runtime import GpuNet
    net, other = network(), network()
    for e in other.edges:
        if e.w is not None:
            e.w = (e.w[..., ::-1] * np.float16(0.75)).astype(net.np_dtype)

    def make(b, spec, share_weights=None, **kw):
        return GpuNet(spec, share_weights=share_weights if b == 2 else None, **kw)

    alone, together = run_alone_and_together([net, other, net], entry, make)
    assert any(not np.array_equal(x, y) for x, y in zip(alone[1][0], alone[1][1]))
    same(alone, together)
