"""Upsampling 1x1 fp16 edges of 64 n channels against the oracle: every factor, ragged views, more 16-channel blocks than travel at once,
maps small enough to be requested at once and larger ones; edges into an OUTPUT site, and several into a site that keeps marks."""
import numpy as np
import pytest

from inputs.nets import NetSpec, _Builder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,h,w,up", [
    (64, 32, 5, 7, 1),             # 35 source pixels: a tile and a bit; 2 x 2 pixels, one part
    (128, 96, 3, 11, 2),           # four parts, three cout tiles
    (256, 32, 4, 8, 3),            # sixteen parts, one full tile
    (320, 64, 9, 5, 1),            # five 16-channel blocks to a wave
    (64, 64, 1, 1, 2),             # one source pixel
    (64, 32, 212, 210, 1),         # more than is requested at once
])
def test_upsampling_edges(cin, cout, h, w, up):
    import gpu_harness as G
    f = 1 << up
    net = NetSpec("up", "f16", h * f, w * f, f)
    b = _Builder(net, np.random.default_rng(cin + up), 0.1)
    x = b.site("in", 8, 1, "input", False, 0.05)
    m = b.site("mid", 16, 2, theta=0.02) if f > 4 else None      # (strides go up to four)
    s = b.site("low", cin, f, theta=0.02)
    y = b.site("out", cout, 1, "output", False, 0.0)
    if m:
        b.conv(x, m, 3, 2)
        b.conv(m, s, 3, 4)
    else:
        b.conv(x, s, 3, f)
    b.conv(s, y, 1, 1, pad=0, up=up)
    rng = np.random.default_rng(h + w)
    v = rng.normal(0, 1, (net.H, net.W, 8)).astype(np.float32)
    frames = [v.astype(np.float16)]
    for _ in range(2):
        v = v.copy()
        v[net.H // 3:net.H // 3 + 3, net.W // 4:net.W // 4 + 9] += 0.5
        frames.append(v.astype(np.float16))
    G.teacher_forced(net, frames, [(0, 0), (0, 0), (1, -1) if min(h, w) > 1 else (0, 0)])


@pytest.mark.parametrize("h,w", [(5, 7), (52, 40)])        # source pixels of the smaller map; requested at once, and later
def test_two_edges_into_a_site_with_marks(h, w):
    """A site fed by two upsampling edges of different factors and a 3x3 edge: pending values add up, and what an edge has marked as touched is
    there for the next and for the site's own step."""
    import gpu_harness as G
    net = NetSpec("up2", "f16", 4 * h, 4 * w, 4)
    b = _Builder(net, np.random.default_rng(h), 0.1)
    x = b.site("in", 8, 1, "input", False, 0.05)
    half = b.site("half", 64, 2, theta=0.3)
    low = b.site("low", 192, 4, theta=0.3)
    s = b.site("sum", 64, 1, theta=0.05)
    y = b.site("out", 32, 1, "output", False, 0.0)
    b.conv(x, half, 3, 2)
    b.conv(x, s, 3, 1)
    b.conv(half, low, 3, 2)
    b.conv(half, s, 1, 1, pad=0, up=1)
    b.conv(low, s, 1, 1, pad=0, up=2)
    b.conv(s, y, 1, 1, pad=0)
    rng = np.random.default_rng(w)
    v = rng.normal(0, 1, (net.H, net.W, 8)).astype(np.float32)
    frames = [v.astype(np.float16)]
    for _ in range(2):
        v = v.copy()
        v[net.H // 3:net.H // 3 + 3, net.W // 4:net.W // 4 + 9] += 0.5
        frames.append(v.astype(np.float16))
    G.teacher_forced(net, frames, [(0, 0), (0, 0), (1, -1)])
