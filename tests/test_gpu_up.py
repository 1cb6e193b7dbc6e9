"""Upsampling 1x1 fp16 edges of 64 n channels against the oracle: every factor, ragged views, more 16-channel blocks than travel at once,
maps small enough to be requested at once and larger ones; a second edge into the same site."""
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
