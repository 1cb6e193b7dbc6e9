"""3 x 3 stride-1 fp16 layers of 64 n input channels (conv_rect.h): every tile against the oracle, and the same bits whatever the
tile where the channels are split four ways - windows lower or narrower than a tile, ragged last tiles, numbers of cout tiles
that are no power of two, one to five chunks, frames in flight where they take other tiles than a frame alone.  The rule itself
takes tiles of 64 entries on small windows; the last two cases are the smallest for which it takes 96, of 32 and of 64 couts.
Stride 2 likewise (32 n input channels; 32, 64 or 128 couts to a tile by the number of tiles)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def frames_of(cin, H, W, n=3):
    rng = np.random.default_rng(cin * 1000 + H * 7 + W)
    x = rng.normal(0, 1, (H, W, cin)).astype(np.float32)
    out = [x.astype(np.float16)]
    for _ in range(n - 1):
        x = x.copy()
        y0, x0 = int(rng.integers(0, max(1, H - 8))), int(rng.integers(0, max(1, W - 17)))
        x[y0:y0 + 8, x0:x0 + 17] += rng.normal(0, 1, x[y0:y0 + 8, x0:x0 + 17].shape).astype(np.float32)
        x[rng.random((H, W)) < 0.02] += 0.5
        out.append(x.astype(np.float16))
    return out


@pytest.mark.parametrize("cin,cout,H,W,entries,couts", [
    (64, 64, 25, 41, 64, 32), (64, 32, 3, 90, 64, 32), (64, 192, 12, 12, 64, 32), (128, 96, 17, 29, 64, 32), (192, 64, 40, 9, 64, 32),
    (256, 192, 14, 15, 64, 32), (320, 64, 1, 30, 64, 32), (64, 96, 64, 73, 96, 32), (64, 192, 64, 73, 96, 64)])
def test_tiles_agree(cin, cout, H, W, entries, couts):
    import gpu_harness as H_
    from inputs.nets import tiny_net
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuNet
    assert B.mdcnn_rect_tiles(H + 2, W + 2, cin, cout)[:2] == (entries, couts)
    net = tiny_net("f16", H, W, (cin, cout), k=3, stride=1, theta=0.05, seed=cin + cout + H, total_stride=1)
    frames, shifts = frames_of(cin, H, W), [(0, 0), (0, 0), (0, -1)]
    outs = {}
    try:
        for sub in (0, 1, 2, 4):
            B.mdcnn_set_option(B.MDCNN_OPT_CONV_HALO_SUB, sub)
            H_.teacher_forced(net, frames, shifts)
            g = GpuNet(net)
            outs[sub] = [g.frame(H_.dev(f), dy, dx)[0].cpu().numpy().copy() for f, (dy, dx) in zip(frames, shifts)]
            g.close()
    finally:
        B.mdcnn_set_option(B.MDCNN_OPT_CONV_HALO_SUB, 0)
    for sub in (0, 1, 4):
        if cin > 64 or sub != 1:                   # (64 channels: the largest tile does not split them)
            for t, (a, b) in enumerate(zip(outs[sub], outs[2])):
                assert np.array_equal(a, b), f"split {sub}, frame {t}"


@pytest.mark.parametrize("cin,cout,H,W,alone,flying", [(64, 96, 55, 64, (64, 32), (96, 32)), (64, 256, 73, 52, (96, 64), (128, 64)),
                                                        (64, 96, 55, 97, (96, 32), (128, 32)), (512, 256, 73, 52, (96, 64), (64, 64)),
                                                        (192, 256, 76, 97, (160, 64), (128, 64))])
def test_frames_in_flight_take_other_tiles(cin, cout, H, W, alone, flying):
    import gpu_harness as H_
    from inputs.nets import tiny_net
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuNet
    assert (B.mdcnn_rect_tiles(H + 2, W + 2, cin, cout)[:2], B.mdcnn_rect_tiles(H + 2, W + 2, cin, cout, in_flight=True)[:2]) == (alone, flying)
    net = tiny_net("f16", H, W, (cin, cout, 32), k=3, stride=1, theta=0.05, seed=cin + cout + H, total_stride=1)
    frames = [H_.dev(f) for f in frames_of(cin, H, W, 6)]
    dy, dx = [0, 0, 1, 0, 0, -1], [0, 0, -1, 0, 1, 0]
    a, b = GpuNet(net), GpuNet(net)
    one = [a.frame(f, y, x)[0].clone() for f, y, x in zip(frames, dy, dx)]
    run, _ = b.frames(frames, dy, dx, depth=4)
    for t, (p, q) in enumerate(zip(one, run)):
        assert np.array_equal(p.cpu().numpy(), q.cpu().numpy()), f"frame {t}"
    a.close()
    b.close()


@pytest.mark.parametrize("cin,cout,H,W,videos,couts", [                              # couts of a tile, alone and in the batch
    (64, 96, 2, 46, 1, (32, 32)), (64, 64, 54, 38, 1, (32, 32)), (64, 64, 100, 126, 1, (64, 64)), (64, 128, 130, 252, 1, (128, 128)), (64, 256, 100, 120, 2, (128, 128)),
    (64, 128, 100, 120, 2, (64, 128)),
    (128, 32, 34, 2, 1, (32, 32)), (192, 192, 58, 90, 1, (64, 64)), (128, 128, 132, 260, 1, (128, 128)),
    (32, 32, 18, 30, 1, (32, 32)), (32, 64, 130, 92, 1, (64, 64)), (96, 192, 44, 62, 2, (32, 64))])
def test_stride_2(cin, cout, H, W, videos, couts):
    import gpu_harness as H_
    from inputs.nets import tiny_net
    from paper_2210_09887_amd import binding as B
    from paper_2210_09887_amd.runtime import GpuBatch, GpuNet
    net = tiny_net("f16", H, W, (cin, cout), k=3, stride=2, theta=0.05, seed=cin + cout + H, total_stride=2)
    by, bx = B.mdcnn_conv_border(3, 2, 1, H, H // 2), B.mdcnn_conv_border(3, 2, 1, W, W // 2)
    rule = getattr(B.lib(), "_ZN5mdcnn14rect_choice_s2Eiiiii")               # (an internal one, on the padded window)
    assert tuple(32 * rule(H // 2 + by[0] + by[1], W // 2 + bx[0] + bx[1], cin, cout, n) for n in (1, videos)) == couts
    frames, shifts = frames_of(cin, H, W), [(0, 0), (0, 0), (0, -1)]
    H_.teacher_forced(net, frames, shifts)
    if videos > 1:                                 # a video of a batch gives the bits it gives alone
        one, many = GpuNet(net), GpuBatch(net, videos)
        for f, (dy, dx) in zip(frames, shifts):
            want = one.frame(H_.dev(f), dy, dx)[0].cpu().numpy()
            outs, _ = many.frame([H_.dev(f)] * videos, [dy] * videos, [dx] * videos)
            for o in outs:
                assert np.array_equal(o.cpu().numpy().reshape(-1), want.reshape(-1))
        one.close()
        many.close()
