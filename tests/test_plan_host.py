"""Host-side check of the launch plan of a frame (mdcnn_frame_plan): whatever
streams the launches are put on, two launches that touch the same site, at
least one of them writing it, must be ordered - by running on one stream or
through the waits.  The launches and what they touch are derived here from the
network description alone; no GPU is needed (buffers wrap a fake address)."""
import pytest

from inputs import build_net
from inputs.nets import pool_net, random_dag_net
from paper_2210_09887_amd import binding as B

FAKE = 0x7F0000000000


def host_net(spec):
    """The library handles of `spec` without device memory (nothing is launched)."""
    dt = B.MDCNN_F16 if spec.dtype == "f16" else B.MDCNN_F32
    shape = [(spec.H // s.stride, spec.W // s.stride, s.C) for s in spec.sites]
    border = [[0, 0, 0, 0] for _ in spec.sites]
    pooled, edges = set(), []
    for e in spec.edges:
        Hs, Ws, _ = shape[e.src]
        pool = getattr(e, "pool", False)
        cd = B.mdcnn_conv_desc(e.k, e.stride, e.pad, spec.sites[e.src].C, spec.sites[e.dst].C, e.up, FAKE if e.k and not pool else None, None, int(pool))
        if pool:
            pooled.add(e.dst)
        elif e.k:
            oh, ow = (Hs + 2 * e.pad - e.k) // e.stride + 1, (Ws + 2 * e.pad - e.k) // e.stride + 1
            by, bx = B.mdcnn_conv_border(e.k, e.stride, e.pad, Hs, oh), B.mdcnn_conv_border(e.k, e.stride, e.pad, Ws, ow)
            border[e.dst] = [max(a, b) for a, b in zip(border[e.dst], [by[0], by[1], bx[0], bx[1]])]
        edges.append(cd)
    kinds = {"input": B.MDCNN_SITE_INPUT, "preact": B.MDCNN_SITE_PREACT, "output": B.MDCNN_SITE_OUTPUT}
    bufs = []
    for i, s in enumerate(spec.sites):
        d = B.mdcnn_buffer_desc()
        d.H, d.W, d.C, d.dtype, d.kind = shape[i][0], shape[i][1], shape[i][2], dt, kinds[s.kind]
        for j in range(4):
            d.border[j] = border[i][j]
        d.tile = spec.total_stride // s.stride
        d.pool_prev = int(i in pooled)
        d.truncation_free = int(bool(getattr(s, "trunc_free", False)))
        bufs.append(B.mdcnn_create_buffer(d, FAKE, B.mdcnn_buffer_bytes(d)))
    net = B.mdcnn_net_create(bufs, [e.src for e in spec.edges], [e.dst for e in spec.edges], edges)
    return net, bufs


def launches_of(spec):
    """[(sites read, sites written)] per launch in program order, as the frame call issues them:
    the delta launch of a site (which also adds a residual skip that is the first edge of the call
    into its destination), then one launch per remaining edge, or one compaction launch."""
    out = []
    for i, s in enumerate(spec.sites):
        if s.kind == "output":
            continue
        mine = [e for e in spec.edges if e.src == i]
        fused = None
        for n, e in enumerate(mine):
            if e.k == 0 and all(q.dst != e.dst for q in mine[:n]):
                fused = n
                break
        if not getattr(s, "trunc_free", False):              # (a truncation-free site has no delta launch)
            out.append((set(), {i} | ({mine[fused].dst} if fused is not None else set())))
        rest = [e for n, e in enumerate(mine) if n != fused]
        for e in rest:
            out.append(({i}, {e.dst}))
        if not rest:
            out.append(({i}, {i}))                          # compaction of the site's own list
    return out


def ordered_before(streams, waits):
    """reach[b] = set of launches that are certain to have finished when b starts."""
    reach, last_on = [], {}
    for b, (s, w) in enumerate(zip(streams, waits)):
        r = set()
        for a in ([last_on[s]] if s in last_on else []) + list(w):
            r |= reach[a] | {a}
        reach.append(r)
        last_on[s] = b
    return reach


NETS = {
    "resnet": lambda: build_net(3, H=64, W=64, widths=(32, 64, 64, 128)),
    "resnet_poolstem": lambda: build_net(3, H=64, W=64, widths=(32, 64, 64, 128), pool_stem=True),
    "hrnet": lambda: build_net(4, H=128, W=96, widths=(32, 64, 64, 128), blocks=2),
    "hrnet_full": lambda: build_net(4),
    "bottleneck": lambda: build_net(5, H=16, W=16, C=64, Cm=32),
    "cnn5": lambda: build_net(2, H=64, W=64),
    "pool": lambda: pool_net("f16", 16, 16, (8, 16, 8), 3, 2, 1),
}
NETS.update({f"dag{seed}": (lambda seed=seed: random_dag_net(seed, "f16" if seed % 2 else "f32")) for seed in range(12)})


@pytest.mark.parametrize("name", list(NETS))
@pytest.mark.parametrize("streams", [0, 1, 2, 3, 4])
def test_conflicting_launches_are_ordered(name, streams):
    spec = NETS[name]()
    net, bufs = host_net(spec)
    try:
        so, waits, used = B.mdcnn_frame_plan(net, streams)
        want = launches_of(spec)
        assert len(so) == len(want)
        assert used == max(so) + 1 and used <= (streams or 4)
        assert all(a < b for b, w in enumerate(waits) for a in w)          # only launches issued earlier are waited for
        assert all(so[a] != so[b] for b, w in enumerate(waits) for a in w)
        reach = ordered_before(so, waits)
        for b, (rb, wb) in enumerate(want):
            for a in range(b):
                ra, wa = want[a]
                if (wa & (rb | wb)) or (ra & wb):
                    assert a in reach[b], f"launches {a} and {b} touch {(wa & (rb | wb)) | (ra & wb)} unordered"
        if streams == 1:
            assert used == 1
    finally:
        B.mdcnn_net_destroy(net)
        for b in bufs:
            B.mdcnn_destroy_buffer(b)


def test_streams_are_used_where_the_network_has_branches():
    used = {}
    for name in ("resnet", "hrnet_full", "cnn5"):   # (random networks: whatever the plan decides)
        net, bufs = host_net(NETS[name]())
        used[name] = (B.mdcnn_frame_plan(net, 0)[2], B.mdcnn_frame_plan(net, 4)[2])
        B.mdcnn_net_destroy(net)
        for b in bufs:
            B.mdcnn_destroy_buffer(b)
    assert used["cnn5"] == (1, 1)                  # a chain
    assert used["resnet"][0] == 1 and used["resnet"][1] > 1      # three projection branches do not pay for the waits
    assert used["hrnet_full"] == (4, 4)            # four branches


@pytest.mark.parametrize("name", list(NETS))
@pytest.mark.parametrize("group,depth,mode", [(1, 4, 0), (2, 4, 0), (1, 2, 0), (3, 3, 0), (64, 4, 0), (1, 1, 0),
                                              (1, 4, 1), (2, 2, 1), (5, 3, 1), (64, 4, 1)])
def test_frames_in_flight_never_share_a_site(name, group, depth, mode):
    """mdcnn_frames keeps several frames in flight on several streams.  Whatever touches a site - its initialisation
    (which runs inside the first launch of another forward call, or ahead of the frame), forward calls, the readout -
    must be ordered against everything else that touches it, in the same and in the neighbouring frames: by being on
    the same stream or through the waits the library documents.  Three frames are laid out here as the library
    issues them and every pair of steps on a common site is checked."""
    spec = NETS[name]()
    net, bufs = host_net(spec)
    B.mdcnn_set_option(B.MDCNN_OPT_PIPE_GROUP, group)
    B.mdcnn_set_option(B.MDCNN_OPT_PIPE_MODE, mode)
    try:
        p = B.mdcnn_frames_plan(net, len(spec.sites), depth)
        first, wait, init, gos, soc, n_calls = (p[k] for k in ("first_call", "wait_call", "init_call", "group_of_site", "stream_of_call", "n_calls"))
        calls = [i for i, s in enumerate(spec.sites) if s.kind != "output"]
        assert n_calls == len(calls) and len(soc) == n_calls + 1
        assert first == list(range(0, n_calls, group))
        assert all(0 <= g < len(first) for g in gos)                          # every site is initialised once a frame
        assert init[0] == -1 and all(0 <= init[g] < first[g] for g in range(1, len(first)))
        if mode == 0:
            assert soc[0] == 0 and all(0 <= b - a <= 1 for a, b in zip(soc, soc[1:])) and soc[-1] < depth
            assert soc[-1] == min(depth, n_calls) - 1                         # every stream gets a run of calls
        stream = (lambda f, c: f % depth) if mode else (lambda f, c: soc[c])
        touched = [{i} | {e.dst for e in spec.edges if e.src == i} for i in calls]
        outputs = {i for i, s in enumerate(spec.sites) if s.kind == "output"}
        sites_of = [{i for i, gg in enumerate(gos) if gg == g} for g in range(len(first))]
        # steps in the order of issue: (frame, call or None for an initialisation, stream, sites, waits [(frame, call)])
        steps = []
        for f in range(3):
            for c in range(n_calls + 1):
                waits = []
                if 0 < c < n_calls and stream(f, c) != stream(f, c - 1):
                    waits.append((f, c - 1))
                for g in range(len(first)):
                    if init[g] == c or (c == 0 and init[g] == -1):
                        st = stream(f, c)
                        if f and wait[g] >= 0 and stream(f - 1, wait[g]) != st:
                            waits.append((f - 1, wait[g]))
                        assert init[g] == -1 or not (sites_of[g] & touched[c]), f"call {c} touches sites initialised in its own launch"
                        steps.append((f, None, st, sites_of[g], waits))
                        waits = []                                             # issued once; the call follows on the same stream
                steps.append((f, c, stream(f, c), touched[c] if c < n_calls else outputs, waits))
        index = {(f, c): k for k, (f, c, _, _, _) in enumerate(steps) if c is not None}
        reach = ordered_before([st for _, _, st, _, _ in steps], [[index[w] for w in ws] for _, _, _, _, ws in steps])
        for b, (fb, cb, _, sb, _) in enumerate(steps):
            for a in range(b):
                fa, ca, _, sa, _ = steps[a]
                if sa & sb:
                    assert a in reach[b], f"frame {fa} call {ca} and frame {fb} call {cb} touch {sa & sb} unordered"
        # within a frame a site is initialised before anything else touches it
        frame0 = [(c, t) for f, c, _, t, _ in steps if f == 0]
        for i in range(len(spec.sites)):
            assert [c for c, t in frame0 if i in t][0] is None, f"site {i} is used before it is initialised"
    finally:
        B.mdcnn_set_option(B.MDCNN_OPT_PIPE_GROUP, 0)
        B.mdcnn_set_option(B.MDCNN_OPT_PIPE_MODE, 1)
        B.mdcnn_net_destroy(net)
        for b in bufs:
            B.mdcnn_destroy_buffer(b)


@pytest.mark.parametrize("name", ["hrnet", "hrnet_full"] + [f"dag{seed}" for seed in range(1, 12, 2)])
@pytest.mark.parametrize("group,depth", [(0, 0), (1, 4), (2, 2), (5, 3), (64, 4), (1, 1)])
def test_rounds_of_frames_in_flight_never_share_a_site(name, group, depth):
    """Networks whose independent launches mdcnn_frames puts together do not follow mdcnn_frames_plan but the rounds of
    mdcnn_frames_rounds.  Every launch of the frame is in exactly one round, no two of a round touch a site that one of them
    writes, launches on one site keep their program order, and with four frames laid out as the library issues them
    (initialisation of a group, its rounds, the readout; frame f on stream f % depth) everything that touches a site is
    ordered."""
    spec = NETS[name]()
    net, bufs = host_net(spec)
    B.mdcnn_set_option(B.MDCNN_OPT_PIPE_GROUP, group)
    try:
        p = B.mdcnn_frames_rounds(net, len(spec.sites), depth)
        if p is None:
            assert not name.startswith("hrnet")
            return
        depth = depth or 4
        want = launches_of(spec)

        def touches(site, edge, skip):
            if edge == -1:
                return set(), {site} | ({spec.edges[skip].dst} if skip >= 0 else set())
            assert edge == -2 or spec.edges[edge].src == site
            return {site}, {site} if edge == -2 else {spec.edges[edge].dst}

        key = lambda t: (sorted(t[0]), sorted(t[1]))
        ops = [(r, touches(s, e, k)) for r, s, e, k in p["ops"]]
        assert sorted(key(t) for _, t in ops) == sorted(key(t) for t in want)
        assert len(p["ops"]) == len(set(p["ops"]))
        rounds = [r for r, _ in ops]
        assert rounds == sorted(rounds) and set(rounds) == set(range(p["n_rounds"])) and p["n_rounds"] < len(ops)
        for r in range(p["n_rounds"]):
            kinds = {e == -1 for q, _, e, _ in p["ops"] if q == r}
            assert len(kinds) == 1                                            # one kind of launch per round
        # program order of two launches that touch a site: the round of the earlier one comes first
        program = []                                                          # (round, touched) in program order
        left = list(ops)
        for t in want:
            hit = next(o for o in left if key(o[1]) == key(t))                # (equal ones come in the order of their rounds)
            left.remove(hit)
            program.append(hit)
        for b, (rb, (readb, writeb)) in enumerate(program):
            for ra, (reada, writea) in program[:b]:
                if (writea & (readb | writeb)) or (reada & writeb):
                    assert ra < rb, f"launch {b} and one before it touch {(writea & (readb | writeb)) | (reada & writeb)}: rounds {ra} and {rb}"
        first, wait, gos = p["first_round"], p["wait_round"], p["group_of_site"]
        assert first[0] == 0 and first == sorted(set(first)) and all(0 <= g < len(first) for g in gos)
        if group:
            assert first == list(range(0, p["n_rounds"], group))
        outputs = {i for i, s in enumerate(spec.sites) if s.kind == "output"}
        touched = [set().union(*(t[0] | t[1] for q, t in ops if q == r)) for r in range(p["n_rounds"])] + [outputs]
        steps = []                                                            # (frame, round or None, sites, waits)
        for f in range(4):
            for r in range(p["n_rounds"] + 1):
                if r in first and r < p["n_rounds"]:
                    g = first.index(r)
                    waits = [(f - 1, wait[g])] if f and wait[g] >= 0 and depth > 1 else []
                    steps.append((f, None, {i for i, gg in enumerate(gos) if gg == g}, waits))
                steps.append((f, r, touched[r], []))
        index = {(f, r): k for k, (f, r, _, _) in enumerate(steps) if r is not None}
        reach = ordered_before([f % depth for f, _, _, _ in steps], [[index[w] for w in ws] for _, _, _, ws in steps])
        for b, (fb, rb, sb, _) in enumerate(steps):
            for a in range(b):
                fa, ra, sa, _ = steps[a]
                if sa & sb:
                    assert a in reach[b], f"frame {fa} round {ra} and frame {fb} round {rb} touch {sa & sb} unordered"
        for i in range(len(spec.sites)):
            assert [r for f, r, t, _ in steps if f == 0 and i in t][0] is None, f"site {i} is used before it is initialised"
    finally:
        B.mdcnn_set_option(B.MDCNN_OPT_PIPE_GROUP, 0)
        B.mdcnn_net_destroy(net)
        for b in bufs:
            B.mdcnn_destroy_buffer(b)


def test_which_networks_run_in_rounds():
    for name, option, value, rounds in [("hrnet", None, 0, True), ("resnet", None, 0, False), ("cnn5", None, 0, False),
                                        ("hrnet", B.MDCNN_OPT_STREAMS, 1, False), ("hrnet", B.MDCNN_OPT_PIPE_MODE, 0, False)]:
        spec = NETS[name]()
        net, bufs = host_net(spec)
        try:
            if option is not None:
                B.mdcnn_set_option(option, value)
            assert (B.mdcnn_frames_rounds(net, len(spec.sites)) is not None) == rounds, (name, option)
        finally:
            B.mdcnn_set_option(B.MDCNN_OPT_STREAMS, 0)
            B.mdcnn_set_option(B.MDCNN_OPT_PIPE_MODE, 1)
            B.mdcnn_net_destroy(net)
            for b in bufs:
                B.mdcnn_destroy_buffer(b)
    spec = NETS["hrnet"]()
    net, bufs = host_net(spec)
    try:
        with pytest.raises(B.MdcnnError):
            B.mdcnn_frames_rounds(net, len(spec.sites), 5)
        with pytest.raises(B.MdcnnError):
            B.mdcnn_frames_rounds(net, len(spec.sites) - 1)
    finally:
        B.mdcnn_net_destroy(net)
        for b in bufs:
            B.mdcnn_destroy_buffer(b)


def test_rectangular_tiles_cover_the_window_within_their_limits():
    """mdcnn_conv_tiles (host only): the rectangles of the halo-staged and the fp32 kernels.  One holds no more pixels than allowed,
    its footprint no more than the staging buffer does, it is not larger than the window, and no other rectangle within the
    limits needs fewer tiles (brute force)."""
    import itertools
    import numpy as np
    rng = np.random.default_rng(3)
    cases = [(258, 258, 256, 352), (130, 130, 128, 192), (66, 66, 128, 192), (66, 66, 64, 128), (98, 74, 256, 352), (14, 11, 64, 128),
             (1, 300, 256, 352), (300, 1, 64, 128), (5, 5, 256, 512)]
    cases += [(int(rng.integers(1, 200)), int(rng.integers(1, 200)), int(rng.choice([64, 128, 256])), int(rng.choice([128, 192, 352, 384, 512]))) for _ in range(40)]
    for Hp, Wp, sub, cap in cases:
        th, tw, tiles = B.mdcnn_conv_tiles(Hp, Wp, 3, sub, cap)
        assert 1 <= th <= Hp and 1 <= tw <= Wp and th * tw <= sub and (th + 2) * (tw + 2) <= cap
        assert tiles == -(-Hp // th) * -(-Wp // tw)
        best = min(-(-Hp // a) * -(-Wp // b) for a, b in itertools.product(range(1, min(Hp, sub) + 1), range(1, min(Wp, sub) + 1))
                   if a * b <= sub and (a + 2) * (b + 2) <= cap)
        assert tiles == best, (Hp, Wp, sub, cap, th, tw, tiles, best)
    assert B.mdcnn_conv_tiles(66, 66, 3, 128, 192) == (11, 11, 36)
    assert B.mdcnn_conv_tiles(258, 258, 3, 256, 352)[2] == 280
    with pytest.raises(B.MdcnnError):
        B.mdcnn_conv_tiles(66, 66, 3, 128, 8)                                # nothing fits a staging buffer of 8 pixels
    with pytest.raises(B.MdcnnError):
        B.mdcnn_conv_tiles(66, 66, 3, 300, 192)                              # more pixels than a list segment


RECT_ROWS = {64: 10, 96: 10, 128: 12, 160: 14, 256: 20}                     # rows of 16 pixels a tile stages


def fewest_rect_tiles(Hp, Wp, entries):
    """Fewest rectangles of at most `entries` pixels, 14 columns and the staged rows less two that cover the window."""
    rows = RECT_ROWS[entries] - 2
    return min(-(-Hp // min(rows, entries // tw, Hp)) * -(-Wp // tw) for tw in range(1, min(14, Wp) + 1))


def test_rect_tiles_cover_the_window_within_their_limits():
    """mdcnn_rect_tiles (host only): the tiles of the layers of 64 n input channels."""
    import numpy as np
    rng = np.random.default_rng(5)
    windows = [(258, 258), (130, 130), (66, 66), (34, 34), (1, 1), (1, 300), (300, 1), (5, 5), (15, 14)]
    windows += [(int(rng.integers(1, 300)), int(rng.integers(1, 300))) for _ in range(60)]
    for Hp, Wp in windows:
        for cin, cout in [(64, 64), (64, 96), (128, 128), (256, 512), (512, 32)]:
            for videos, in_flight, shared in [(1, 0, 0), (1, 1, 0), (1, 0, 1), (8, 0, 0), (16, 1, 0)]:
                m, couts, th, tw, tiles = B.mdcnn_rect_tiles(Hp, Wp, cin, cout, videos, in_flight, shared)
                assert 1 <= th <= min(Hp, RECT_ROWS[m] - 2) and 1 <= tw <= min(Wp, 14) and th * tw <= m
                assert cout % couts == 0 and couts in (32, 64)
                assert tiles == -(-Hp // th) * -(-Wp // tw) * (cout // couts) == fewest_rect_tiles(Hp, Wp, m) * (cout // couts)
                assert m != 256 or cin == 64                                 # (larger tiles do not split the channels)
    for bad in [(0, 5, 64, 64), (5, 5, 96, 64), (5, 5, 64, 48), (5, 5, 0, 64), (5, 5, 64, 8192)]:
        with pytest.raises(B.MdcnnError):
            B.mdcnn_rect_tiles(*bad)


def test_rect_tiles_of_one_layer_split_its_channels_alike():
    """The split of the channels fixes the order of the sums: whatever the batch, whatever runs beside, it is the same."""
    for Hp, Wp in [(114, 114), (130, 130), (162, 162), (200, 190), (210, 215), (258, 258), (40, 700)]:
        for cout in (32, 64, 96, 128):
            split = {B.mdcnn_rect_tiles(Hp, Wp, 64, cout, v, f, s)[0] != 256 for v in (1, 2, 7, 16) for f in (0, 1) for s in (0, 1)}
            assert len(split) == 1, (Hp, Wp, cout)


@pytest.mark.parametrize("k", [1, 3, 5])
def test_gather_tiles_of_a_shared_launch_are_among_its_own(k):
    """mdcnn_gather_tile (host only): an edge asked for by a shared launch takes a tile that launch does not carry (256 x 64) only
    where it would alone as well - 224 blocks of it, about one per compute unit - and never a smaller one than alone."""
    for entries in [1, 64, 6144, 128 * 112, 192 * 192, 256 * 112, 256 * 223, 256 * 224, 258 * 258, 10 ** 6]:
        for cout in (32, 64, 96, 128, 192, 256, 320, 512):
            alone, shared = B.mdcnn_gather_tile(entries, k, cout), B.mdcnn_gather_tile(entries, k, cout, True)
            for pixels, couts in (alone, shared):
                assert cout % couts == 0 and 256 % pixels == 0
            assert shared[0] * shared[1] >= alone[0] * alone[1] and (k == 1 or shared == alone), (entries, cout)
            if (256, 64) in (alone, shared):
                assert alone == shared and -(-entries // 256) * (cout // 64) >= 224, (entries, cout)
    assert B.mdcnn_gather_tile(192 * 192, 1, 64, True) == (128, 64)
    for bad in [(0, 1, 64), (5, 0, 64), (5, 1, 48), (5, 1, 8192)]:
        with pytest.raises(B.MdcnnError):
            B.mdcnn_gather_tile(*bad)


def test_batches_in_flight_take_tiles_by_what_they_hold():
    """In a full GPU a launch costs its row tiles of 32 pixels and, per tile, weights and epilogue: no other size has fewer
    tiles and no more row tiles than the one taken."""
    def cost(Hp, Wp, m):                                                    # the rectangle as rect_tile picks it: fewest tiles, then the smaller footprint
        best = None
        for tw in range(1, min(14, Wp) + 1):
            th = min(m // tw, RECT_ROWS[m] - 2, Hp)
            down, across = -(-Hp // th), -(-Wp // tw)
            th = -(-Hp // down)
            key = (down * across, (th + 2) * (tw + 2))
            if best is None or key < best[0]:
                best = key, -(-th * tw // 32) * down * across
        return best[0][0], best[1]

    for view in range(96, 640, 16):
        for cin, stride in [(64, 4), (128, 8), (256, 16), (512, 32), (512, 16)]:
            w = view // stride + 2
            for videos in (8, 16):
                m, couts, _, _, tiles = B.mdcnn_rect_tiles(w, w, cin, cin, videos, True)
                of = {s: cost(w, w, s) for s in (64, 96, 128)}
                if m == 256 or any(t * (cin // couts) * videos * 3 <= 512 for t, _ in of.values()):
                    continue
                assert tiles == of[m][0] * (cin // couts)
                for s, (t, rows) in of.items():
                    assert not (t < of[m][0] and rows <= of[m][1]), (w, cin, videos, m, s)
    # weights: 512 channels on 34 x 34, 96 tiles of 128 instead of 160 of 64
    assert B.mdcnn_rect_tiles(34, 34, 512, 512, 8, True)[0] == 128


@pytest.mark.parametrize("view", [96, 128, 160, 192, 224, 256, 288, 320, 352])
def test_small_layers_in_flight_keep_their_blocks(view):
    """A launch among frames in flight has about a third of the 512 places of the GPU.  As long as its tiles of 64 entries fit
    those, larger ones only make it longer: no layer of a small view is put onto fewer blocks than it has places for."""
    for cin, stride in [(64, 2), (128, 4), (256, 8), (512, 16)]:
        window = view // stride + 2
        m, couts, _, _, tiles = B.mdcnn_rect_tiles(window, window, cin, cin, 1, True)
        small = fewest_rect_tiles(window, window, 64) * (cin // couts)
        if small <= 512 // 3:
            assert m == 64, (window, cin, m, tiles, small)
        else:
            assert tiles >= 512 // 6, (window, cin, m, tiles, small)
