"""The convolution tile of the fp32 layers, against the oracle on ragged windows, partial chunks and cout tiles, odd numbers
of steps, strides and upsampling edges."""
import numpy as np
import pytest

from inputs.nets import NetSpec, _Builder, tiny_net

pytestmark = pytest.mark.gpu


def frames_of(net, seed, n=3):
    rng = np.random.default_rng(seed)
    x = rng.normal(0, 1, (net.H, net.W, net.sites[0].C)).astype(np.float32)
    out = [x.astype(net.np_dtype)]
    for _ in range(n - 1):
        x = x.copy()
        y0, x0 = int(rng.integers(0, max(1, net.H - 5))), int(rng.integers(0, max(1, net.W - 7)))
        x[y0:y0 + 5, x0:x0 + 7] += rng.normal(0, 1, x[y0:y0 + 5, x0:x0 + 7].shape).astype(np.float32)
        x[rng.random((net.H, net.W)) < 0.03] += 0.5
        out.append(x.astype(net.np_dtype))
    return out


@pytest.mark.parametrize("cin,cout,H,W,k,stride", [
    (96, 32, 8, 8, 3, 1),          # one tile and a bit: the 10 x 10 window in tiles of up to 32 pixels
    (8, 32, 5, 37, 3, 1),          # a quarter of a chunk: one wave multiplies
    (24, 96, 33, 18, 3, 1),        # three quarters of a chunk, three cout tiles
    (72, 16, 30, 22, 1, 1),        # half a cout tile
    (128, 128, 48, 40, 3, 2),      # stride 2
    (40, 64, 90, 100, 5, 1),       # 25 taps; a chunk and a quarter
    (480, 64, 11, 9, 3, 1),        # a long K loop
    (512, 64, 11, 9, 3, 2),
    (32, 32, 41, 29, 3, 1),        # one chunk: an odd number of steps
    (64, 72, 3, 75, 3, 1),         # two chunks, a quarter of a cout tile; a window narrower than a tile is high
    (96, 96, 3, 75, 3, 1),         # three chunks: an odd number, three cout tiles
    (128, 32, 8, 8, 3, 1),         # from here on the tiles of conv_f32s.h: 3x3, stride 1, 64 n channels, 32 m couts
    (512, 64, 11, 9, 3, 1),
    (64, 96, 3, 75, 3, 1),
])
def test_fp32_layers(cin, cout, H, W, k, stride):
    import gpu_harness as G
    H, W = H * stride, W * stride
    net = tiny_net("f32", H, W, (cin, cout), k=k, stride=stride, theta=0.05, seed=cin + cout, total_stride=stride)
    G.teacher_forced(net, frames_of(net, cin * 10 + cout), [(0, 0), (0, 0), (1, -1)])


def test_fp32_upsampling_edge():
    import gpu_harness as G
    net = NetSpec("up", "f32", 36, 52, 4)
    b = _Builder(net, np.random.default_rng(3), 0.1)
    x = b.site("in", 8, 1, "input", False, 0.05)
    s = b.site("low", 96, 4, theta=0.02)
    y = b.site("out", 32, 1, "output", False, 0.0)
    b.conv(x, s, 5, 4, pad=2)
    b.conv(s, y, 1, 1, pad=0, up=2)
    G.teacher_forced(net, frames_of(net, 1), [(0, 0), (0, 1), (0, 0)])


def kernel_of_last_site(net, X):
    """Which kind of kernel counted the products of a frame into the network's output site."""
    import gpu_harness as G
    from paper_2210_09887_amd.runtime import GpuNet
    g = GpuNet(net)
    try:
        g.frame(G.dev(X))
        t = g.totals()["per_site"]
        n = [int(t[k][-1]) for k in ("macs_mfma", "macs_plain")]
        assert sum(v > 0 for v in n) == 1, n
        return "mfma" if n[0] else "plain"
    finally:
        g.close()


@pytest.mark.parametrize("cin,cout,H,W,k,kernel", [
    (8, 16, 32, 64, 1, "plain"),        # 128 products per pixel: plain from 2048 pixels on
    (8, 16, 32, 63, 1, "mfma"),
    (8, 16, 126, 142, 3, "plain"),      # 1152 products, a padded window of 128 x 144
    (8, 16, 126, 141, 3, "mfma"),
    (128, 16, 128, 256, 1, "plain"),    # 2048 products: the most there may be, 32768 pixels
    (128, 16, 127, 258, 1, "mfma"),
    (8, 256, 181, 182, 1, "plain"),     # the most couts
    (72, 32, 200, 200, 1, "mfma"),      # 2304 products
])
def test_small_layers_on_large_windows(cin, cout, H, W, k, kernel):
    """Both sides of the line between k_conv_f32 and the plain kernel with its weights in LDS."""
    import gpu_harness as G
    net = tiny_net("f32", H, W, (cin, cout), k=k, theta=0.05, seed=cin + cout)
    frames = frames_of(net, cin + cout, 2)
    assert kernel_of_last_site(net, frames[0]) == kernel
    G.teacher_forced(net, frames, [(0, 0), (1, -1)])


@pytest.mark.parametrize("rows,kernel", [(64, "plain"), (63, "mfma")])
def test_small_upsampling_edges_on_large_views(rows, kernel):
    import gpu_harness as G
    net = NetSpec("up", "f32", 2 * rows, 256, 2)
    b = _Builder(net, np.random.default_rng(4), 0.1)
    x = b.site("in", 8, 1, "input", False, 0.05)
    s = b.site("low", 8, 2, theta=0.02)
    y = b.site("out", 16, 1, "output", False, 0.0)
    b.conv(x, s, 3, 2)
    b.conv(s, y, 1, 1, pad=0, up=1)
    frames = frames_of(net, 2)
    assert kernel_of_last_site(net, frames[0]) == kernel
    G.teacher_forced(net, frames, [(0, 0), (0, 1), (0, 0)])


def row_tiles(H, W, cin, cout, videos=1):
    """Row tiles of a tile that the library takes for 3x3 fp32 layers of 64 n channels on H x W views (an internal rule)."""
    from paper_2210_09887_amd import binding as B
    return getattr(B.lib(), "_ZN5mdcnn12split_choiceEiiiii")(H + 2, W + 2, cin, cout, videos)


@pytest.mark.parametrize("cin,cout,H,W,tiles", [
    (64, 32, 16, 16, 1),           # few tiles: one row tile each (2 x 14 pixels of an 18 x 18 window), one chunk of channels
    (192, 96, 37, 53, 1),          # the same with three chunks and three cout tiles, ragged in both directions
    (512, 32, 1, 1, 1),            # one pixel, eight chunks
    (64, 64, 64, 64, 2),           # two row tiles, one chunk
    (128, 64, 61, 75, 2),          # two chunks, ragged
    (64, 64, 96, 96, 3),           # three row tiles, one chunk: nothing staged ahead
    (128, 64, 95, 97, 3),          # three row tiles, two chunks
    (192, 64, 94, 99, 3),          # three chunks: the last in the first buffer
])
def test_fp32_layers_of_64_n_channels(cin, cout, H, W, tiles):
    """The tiles whose products are made of bf16 parts: every number of row tiles, dense frames (the first) and sparse ones."""
    import gpu_harness as G
    assert row_tiles(H, W, cin, cout) == tiles
    net = tiny_net("f32", H, W, (cin, cout), theta=0.05, seed=cin + cout)
    G.teacher_forced(net, frames_of(net, cin * 10 + cout), [(0, 0), (0, 0), (1, -1)])


def dense_frame(net, X):
    """Output of the first frame of a one-layer network, and the same in 64 bits."""
    import gpu_harness as G
    import torch
    from paper_2210_09887_amd.runtime import GpuNet
    g = GpuNet(net)
    try:
        out = g.split_outputs(g.frame(G.dev(X))[0])[0].double().cpu()
    finally:
        g.close()
    e, (cin, cout) = net.edges[0], (net.sites[0].C, net.sites[1].C)
    w = torch.from_numpy(e.w.reshape(3, 3, cout, cin).transpose(2, 3, 0, 1).copy()).double()
    ref = torch.nn.functional.conv2d(torch.from_numpy(X).double().permute(2, 0, 1)[None], w, torch.from_numpy(e.b).double(), padding=1)
    return out.reshape(net.H, net.W, cout), ref[0].permute(1, 2, 0)


@pytest.mark.parametrize("scale", [1.0, 1e-30, 1e30])
@pytest.mark.parametrize("cin,n", [(64, 64), (512, 16)])
def test_precision_of_split_products(cin, n, scale):
    """Against 64 bits: a sum of 9 cin products is rounded 9 cin / 64 times in each of four waves, to 2^-25 of a partial sum (of
    the sum's size or less) on average: at most 2^-25 sqrt(9 cin / 16 + 8), 2^-22.8 and 2^-21 here, where fp32 products, each of
    them rounded, come to 2^-22.1 and 2^-20.7.  (The ends of the range: test_precision_at_the_ends_of_the_range.)"""
    net = tiny_net("f32", n, n, (cin, 32), theta=0.0, seed=cin)
    net.edges[0].b[:] = 0
    X = (np.maximum(np.random.default_rng(cin).normal(0, 1, (n, n, cin)), 0) * scale).astype(np.float32)
    out, ref = dense_frame(net, X)
    assert float((out - ref).norm() / ref.norm()) < 2.0 ** -25 * (9 * cin / 16 + 8) ** 0.5


@pytest.mark.parametrize("n", [16, 64, 96])
def test_values_that_are_not_finite(n):
    """An infinity or NaN in the frame, and a finite value past what bf16 holds: what it reaches is what fp32 sums make of it, all else is
    untouched."""
    net = tiny_net("f32", n, n, (64, 64), theta=0.0, seed=n)
    X = np.random.default_rng(n).normal(0, 1, (n, n, 64)).astype(np.float32)
    X[3, 4, 5], X[9, 9, 60], X[n - 1, 2, 33], X[n - 2, n - 3, 7] = np.inf, np.nan, -np.inf, 3.4e38
    out, ref = dense_frame(net, X)
    big = ref.abs() > 1e30         # (sums with the large value: near the largest fp32, or past it)
    assert bool((out.isnan() == ref.isnan()).all())
    assert bool((out.isinf() & ~big == ref.isinf() & ~big).all()) and bool((out[ref.isinf()] == ref[ref.isinf()]).all())
    fin = ref.isfinite() & ~big
    assert int((~fin).sum()) <= 4 * 9 * 64 and float((out - ref)[fin].abs().max()) < 1e-4
    near = big & (ref.abs() < 3.4e38)
    assert float(((out - ref)[near] / ref[near]).abs().max()) < 1e-6


@pytest.mark.parametrize("bad", ["finite", "frame", "weight"])
@pytest.mark.parametrize("cin,n,videos,alone,together", [(64, 64, 2, 2, 3), (64, 96, 2, 3, 2), (64, 32, 4, 1, 2), (64, 32, 8, 1, 3), (128, 64, 2, 2, 3)])
def test_bits_in_a_batch(cin, n, videos, alone, together, bad):
    """A video of a batch gives the bits it gives alone where the batch takes other tiles: dense and sparse frames, and frames with a few
    sums that are not finite, from infinities, NaN and overflow in the frame or from a weight."""
    import gpu_harness as G
    from paper_2210_09887_amd.runtime import GpuBatch, GpuNet
    net = tiny_net("f32", n, n, (cin, 64), theta=0.05, seed=n + videos)
    assert (row_tiles(n, n, cin, 64), row_tiles(n, n, cin, 64, videos)) == (alone, together)
    frames = frames_of(net, n + videos)
    if bad == "weight":
        w = net.edges[0].w.reshape(9, 64, cin)
        w[2, 5, 7], w[4, 40, 63] = np.inf, np.nan
    if bad == "frame":
        for t, (y, x) in enumerate([(3, 4), (n // 2, n - 1), (n - 1, n // 3)]):
            frames[t][y, x, :5] += np.float32([np.inf, 0, 0, 0, 0])
            frames[t][n - 1 - y, n - 1 - x, 9] = [np.nan, 3.4e38, -np.inf][t]
    many = GpuBatch(net, videos)
    one = GpuNet(net)
    try:
        for f, (dy, dx) in zip(frames, [(0, 0), (0, 0), (1, -1)]):
            want = one.frame(G.dev(f), dy, dx)[0].cpu().numpy().reshape(-1)
            outs, _ = many.frame([G.dev(f)] * videos, [dy] * videos, [dx] * videos)
            for o in outs:
                o = o.cpu().numpy().reshape(-1)
                assert np.array_equal(o, want, equal_nan=True), f"{int((~((o == want) | (np.isnan(o) & np.isnan(want)))).sum())} values differ"
    finally:
        one.close()
        many.close()


@pytest.mark.parametrize("in_frame,in_weights", [(1e-34, 1.0), (1e-36, 1.0), (1.0, 1e-36), (1e-20, 1e-16), (1e35, 1e-36), (3e-38, 1e4), (1e-42, 1e10), (1e10, 1e-39), (1e37, 1.0)])
@pytest.mark.parametrize("cin,n", [(64, 64), (512, 16)])
def test_precision_at_the_ends_of_the_range(cin, n, in_frame, in_weights):
    """The bound of test_precision_of_split_products wherever the sums are normal numbers: the second and third part of a value below 2^-110
    would not be, and the matrix instruction takes what is not for zero.  At the upper end sums of 2^80 and more, which take a second pass."""
    net = tiny_net("f32", n, n, (cin, 32), theta=0.0, seed=cin)
    net.edges[0].b[:] = 0
    net.edges[0].w *= np.float32(in_weights)
    X = (np.maximum(np.random.default_rng(cin).normal(0, 1, (n, n, cin)), 0) * in_frame).astype(np.float32)
    out, ref = dense_frame(net, X)
    err = float((out - ref).norm() / ref.norm())
    assert err < 2.0 ** -25 * (9 * cin / 16 + 8) ** 0.5


@pytest.mark.parametrize("large", [1e32, 1e38])
@pytest.mark.parametrize("n", [16, 64, 96])
def test_small_sums_beside_large_values(n, large):
    """Values from 2^104 on with weights of zero: the second pass, which divides the rows by 2^40, loses all the others, and its sums are left to
    fp32 products.  The bound is theirs: a rounding per product, 9 cin / 4 in each of four waves, of 2^-25 of the sum on average."""
    net = tiny_net("f32", n, n, (64, 32), theta=0.0, seed=n)
    net.edges[0].b[:] = 0
    net.edges[0].w.reshape(9, 32, 64)[:, :, 7] = 0
    X = (np.maximum(np.random.default_rng(n).normal(0, 1, (n, n, 64)), 0) * 1e-28).astype(np.float32)
    X[2::5, 1::7, 7] = large
    out, ref = dense_frame(net, X)
    assert float((out - ref).norm() / ref.norm()) < 2.0 ** -25 * (9 * 64 / 4 + 8) ** 0.5


@pytest.mark.parametrize("tap", [0, 4])
def test_one_product(tap):
    """One live product to a sum.  Left out of it are the products of parts 1, 2 and 2, 1, at most 2^-25 of a unit pair's product each, and 2, 2,
    2^-34: half a unit of the last place and 2^-11 of one.  Rounding the sum takes another half, and each of the three sums of the smaller parts, at
    most 2^-7 of the whole, at most a unit of its own last place: 2^-5 in all."""
    net = tiny_net("f32", 32, 32, (64, 32), theta=0.0, seed=7)
    net.edges[0].b[:] = 0
    rng = np.random.default_rng(tap)
    w = rng.uniform(1, 2, 32).astype(np.float32)
    net.edges[0].w[:] = 0
    net.edges[0].w.reshape(9, 32, 64)[tap, :, 17] = w
    X = np.zeros((32, 32, 64), np.float32)
    X[:, :, 17] = rng.uniform(1, 2, (32, 32)).astype(np.float32)
    out, ref = dense_frame(net, X)
    ulp = 2.0 ** (ref.abs().clamp_min(1e-30).log2().floor() - 23)
    worst = float(((out - ref).abs() / ulp)[ref != 0].max())
    assert worst <= 1 + 2.0 ** -5 + 2.0 ** -11
