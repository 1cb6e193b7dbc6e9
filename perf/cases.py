"""Performance cases: what a program that uses this library has it do, from one call on a tiny map to a batch of videos.

A case names one of the five workload networks of `inputs.nets` (single_conv, cnn5, resnet, hrnet, bottleneck), the size of
its view, and how the video reaches the library:

  live    one frame per pass, `GpuNet.frame`: a camera whose next frame is only there once the last one is done
  clip    `frames` consecutive frames that are in device memory already, one `GpuNet.frames` call
  crop    the same with a crop of its own per frame, `GpuNet.frames_crop`
  masked  the same with the input masks made by the library, `GpuNet.frames_masked`
  layers  one frame per pass through the layer-wise calls: shift, input mask, one forward call per site, readout
  batch   one frame of each of `videos` videos per pass, `GpuBatch.frame`
  batch_clip  `frames` frames of each of `videos` videos in one call, `GpuBatch.frames`

The scenes have the structure of `inputs.scenes` (a window that moves by whole tiles over a panorama of Gaussian blobs,
moving objects, sensor noise; forced masks of clustered 4 x 4 tiles for the bottleneck) and are made on the GPU from the seed.
A video starts over when its frames are used up; the jump back is one more camera shift.
"""
from __future__ import annotations

import functools
import random

import numpy as np
import torch

from inputs.nets import build_net, truncation_free
from inputs.scenes import clustered_tile_mask
from paper_2210_09887_amd import binding as B
from paper_2210_09887_amd.runtime import GpuBatch, GpuNet

CONFIG = {"single_conv": 1, "cnn5": 2, "resnet": 3, "hrnet": 4, "bottleneck": 5}
TILE = {"single_conv": 1, "cnn5": 4, "resnet": 8, "hrnet": 32, "bottleneck": 1}       # resnet with the pooling stem: 16
# share of a network's pixels that a frame updates on these scenes (resets included), for work() only
DENSITY = {"single_conv": 0.35, "cnn5": 0.2, "resnet": 0.55, "hrnet": 0.5}
LIVE_FRAMES = 12                                   # frames a live video has before it starts over


def _case(name, net, H, W, entry, dtype="f16", frames=1, videos=1, density=0.0, pool_stem=False, truncation_free=False):
    c = dict(net=net, H=H, W=W, entry=entry, dtype=dtype, frames=frames, videos=videos, density=density,
             pool_stem=pool_stem, truncation_free=truncation_free)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call there is: one layer on a 64 x 64 map, fp32; nothing but latency and launches
        _case("single_conv_live", "single_conv", 64, 64, "live", "f32"),
        # a small fp32 network behind a camera
        _case("cnn5_live", "cnn5", 256, 256, "live", "f32"),
        # one residual block of a larger model, the mask given by the caller, a fifth of the pixels updated
        _case("bottleneck_live", "bottleneck", 128, 128, "live", density=0.2),
        # the backbone behind a camera: the latency of a frame
        _case("resnet_live", "resnet", 512, 512, "live"),
        # the backbone on a decoded clip: the frame rate of one video
        _case("resnet_clip", "resnet", 512, 512, "clip", frames=30),
        # the backbone driven layer by layer with the mask front end, on a frame of no round size
        _case("resnet_layers_ragged", "resnet", 296, 424, "layers"),
        # the backbone with the usual pooling stem on HD frames of which a box is processed
        _case("resnet_pool_crop", "resnet", 720, 1280, "crop", frames=12, pool_stem=True),
        # the backbone kept in fp32, as a model is that was never converted
        _case("resnet_f32_live", "resnet", 256, 256, "live", "f32"),
        # many cameras on one GPU: the largest amount of work in one call
        _case("resnet_batch_clip", "resnet", 512, 512, "batch_clip", frames=4, videos=16),
        # the multi-resolution pose network behind a camera: many small layers
        _case("hrnet_live", "hrnet", 384, 288, "live"),
        # the same on a decoded clip
        _case("hrnet_clip", "hrnet", 384, 288, "clip", frames=24),
        # the same for eight people at a time
        _case("hrnet_batch", "hrnet", 384, 288, "batch", videos=8),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def size(lo, hi, tile):                        # a multiple of the tile, spread over the logarithm
        a, b = np.log(lo / tile), np.log(hi / tile)
        return tile * max(1, int(round(np.exp(rng.uniform(a, b)))))

    net = rng.choice(["single_conv", "cnn5", "bottleneck", "resnet", "resnet", "resnet", "hrnet", "hrnet"])
    if net == "single_conv":
        return _case(None, net, size(16, 256, 1), size(16, 256, 1), "live", "f32")
    if net == "cnn5":
        if rng.random() < 0.5:
            return _case(None, net, size(64, 512, 4), size(64, 512, 4), "clip", "f32", frames=rng.randint(4, 30))
        return _case(None, net, size(64, 512, 4), size(64, 512, 4), "live", "f32")
    if net == "bottleneck":
        return _case(None, net, size(32, 256, 1), size(32, 256, 1), "live", density=round(float(np.exp(rng.uniform(np.log(0.01), 0.0))), 3),
                     truncation_free=rng.random() < 0.5)
    if net == "hrnet":
        H, W = size(96, 512, 32), size(96, 512, 32)
        entry = rng.choice(["live", "clip", "batch", "batch_clip"])
        return _case(None, net, H, W, entry, frames={"clip": rng.randint(4, 24), "batch_clip": 2}.get(entry, 1),
                     videos=rng.randint(2, 16) if "batch" in entry else 1)
    if rng.random() < 0.15:
        return _case(None, net, size(64, 256, 8), size(64, 256, 8), "live", "f32")
    pool = rng.random() < 0.3
    tile = 16 if pool else 8
    H, W = size(96, 1024, tile), size(96, 1024, tile)
    entry = rng.choice(["live", "clip", "crop", "masked", "layers", "batch", "batch_clip"])
    budget = max(1, int(64 * 512 * 512 / (H * W)))                      # frames of the largest listed case
    if "batch" in entry:
        videos = max(1, min(rng.randint(2, 16), budget))
        return _case(None, net, H, W, entry, frames=max(1, min(4, budget // videos)), videos=videos, pool_stem=pool)
    return _case(None, net, H, W, entry, frames=max(1, min(rng.randint(4, 30), budget)), pool_stem=pool)


# -- the model: what a program loads once, the same for every seed -------------------------------------------------------
@functools.lru_cache(maxsize=8)
def _spec(net, H, W, dtype, pool_stem, trunc_free):
    kw = dict(pool_stem=True) if pool_stem else {}
    spec = build_net(CONFIG[net], **({} if net == "single_conv" else dict(H=H, W=W)), **kw)
    spec.H, spec.W = H, W
    if trunc_free:
        truncation_free(spec)
    if dtype != spec.dtype:                        # the fp16 model kept in fp32
        spec.dtype = dtype
        for e in spec.edges:
            if e.w is not None:
                e.w = e.w.astype(np.float32)
    return spec


def _spec_of(case):
    return _spec(case["net"], case["H"], case["W"], case["dtype"], case["pool_stem"], case["truncation_free"])


# -- scenes ------------------------------------------------------------------------------------------------------------
def _path(net, r, n):
    """Camera steps in tiles, one per frame; the first is filled in by _video."""
    if net == "single_conv":
        return [(2, 3)] * n
    if net == "cnn5":
        return [(0, 1)] * n
    if net == "resnet":
        return [(r.randint(-2, 2), r.randint(-2, 2)) for _ in range(n)]
    if net == "hrnet":                             # a pan every eighth frame, to and fro
        return [(0, 0) if t % 8 else (0, r.randint(1, 2) * (1 if t // 8 % 2 else -1)) for t in range(n)]
    return [(0, 0) if t % 10 else (0, 16) for t in range(n)]


def _blobs(r, C, H, W, n, sigma):
    """[C, H, W] float32: per channel the sum of n Gaussian blobs."""
    out = torch.zeros((C, H, W), device="cuda")
    ys = torch.arange(H, device="cuda", dtype=torch.float32)[None, :, None]
    xs = torch.arange(W, device="cuda", dtype=torch.float32)[None, None, :]
    p = torch.tensor([[[r.uniform(0, H), r.uniform(0, W), r.uniform(*sigma), r.uniform(-1, 1)] for _ in range(C)] for _ in range(n)], device="cuda")
    for cy, cx, sg, amp in p.permute(0, 2, 1)[..., None, None].unbind(0):      # [C, 1, 1] each
        out += torch.exp(-0.5 * ((ys - cy) / sg) ** 2) * (torch.exp(-0.5 * ((xs - cx) / sg) ** 2) * amp)
    return out


class _Video:
    """Frames in device memory, camera shifts, forced masks, crops."""

    def __init__(self, case, spec, seed, n):
        r = random.Random(seed)
        g = torch.Generator(device="cuda").manual_seed(r.randrange(1 << 31))
        net, H, W, tile, C = case["net"], spec.H, spec.W, spec.total_stride, spec.sites[0].C
        dt = torch.float16 if spec.dtype == "f16" else torch.float32
        noise = lambda *shape: torch.randn(shape, device="cuda", generator=g)
        steps = _path(net, r, n)
        steps[0] = (0, 0)
        lim_y, lim_x = max(1, H // tile - 1), max(1, W // tile - 1)
        steps = [(max(-lim_y, min(lim_y, a)), max(-lim_x, min(lim_x, b))) for a, b in steps]
        at = np.cumsum(np.array(steps), axis=0)
        at -= at.min(axis=0)
        self.shifts = [(-int(sum(s[0] for s in steps)), -int(sum(s[1] for s in steps)))] + steps[1:]     # [0]: the jump back
        span = (at.max(axis=0) + 1) * tile
        self.forced = None
        frames = torch.empty((n, H, W, C), dtype=dt, device="cuda")
        if net == "bottleneck":
            rng = np.random.default_rng(seed)
            canvas = 0.5 * noise(H + int(span[0]), W + int(span[1]), C)
            mh, mw = -(-H // 4) * 4, -(-W // 4) * 4
            masks = np.stack([clustered_tile_mask(rng, mh, mw, case["density"])[:H, :W] for _ in range(n)])
            self.forced = torch.from_numpy(np.ascontiguousarray(masks)).cuda()
            for t in range(n):
                y, x = (int(v) * tile for v in at[t])
                view = canvas[y:y + H, x:x + W]
                view += 0.1 * noise(H, W, C) * self.forced[t, :, :, None]
                frames[t] = view
        else:
            pano = _blobs(r, C, H + int(span[0]), W + int(span[1]), 40, (4.0, 12.0)).permute(1, 2, 0).contiguous()
            n_obj, sigma = {"single_conv": (0, 0.01), "cnn5": (3, 0.005), "resnet": (10, 0.005), "hrnet": (20, 0.005)}[net]
            objs = []
            for _ in range(n_obj):                 # textured or plain patches that move over the scene
                s = 24 if net == "cnn5" else r.randint(16, 64) if net == "resnet" else 20
                s = min(s, H, W)
                tex = _blobs(r, C, s, s, 6, (2.0, 6.0)).permute(1, 2, 0)
                objs.append((tex, s, r.uniform(0, H), r.uniform(0, W), r.uniform(-3, 3), r.uniform(-3, 3)))
            for t in range(n):
                y, x = (int(v) * tile for v in at[t])
                if net == "single_conv":           # one redrawn square per frame
                    k = min(8, H, W)
                    sy, sx = y + r.randint(0, H - k), x + r.randint(0, W - k)
                    pano[sy:sy + k, sx:sx + k] = 2 * torch.rand((k, k, C), device="cuda", generator=g) - 1
                view = pano[y:y + H, x:x + W].clone()
                for tex, s, oy, ox, vy, vx in objs:
                    py, px = int(oy + vy * t), int(ox + vx * t)
                    y0, x0, y1, x1 = max(py, 0), max(px, 0), min(py + s, H), min(px + s, W)
                    if y1 > y0 and x1 > x0:
                        view[y0:y1, x0:x1] = tex[y0 - py:y1 - py, x0 - px:x1 - px]
                frames[t] = view + sigma * noise(H, W, C)
        self.frames = [frames[t] for t in range(n)]
        self.crops = None
        if case["entry"] == "crop":                # a box of about 2/3 x 2/3 of the view that wanders over it
            Ht, Wt = H // tile, W // tile
            th, tw = max(1, round(2 * Ht / 3)), max(1, round(2 * Wt / 3))
            cy, cx = (Ht - th) // 2, (Wt - tw) // 2
            self.crops = []
            for t in range(n):
                if t and t % 4 == 0:
                    cy, cx = max(0, min(Ht - th, cy + r.randint(-1, 1))), max(0, min(Wt - tw, cx + r.randint(-1, 1)))
                self.crops.append((cy, cx, th, tw))
            self.frames = [f[c[0] * tile:(c[0] + c[2]) * tile, c[1] * tile:(c[1] + c[3]) * tile].contiguous() for f, c in zip(self.frames, self.crops)]


# -- the program -------------------------------------------------------------------------------------------------------
class _State:
    """A network (or a batch of them) with its videos, and one pass of the program's loop."""

    def __init__(self, case, seed):
        spec = _spec_of(case)
        self.entry, self.spec, self.t = case["entry"], spec, 0
        nv = case["videos"]
        self.one_by_one = self.entry in ("live", "layers", "batch")
        self.n = LIVE_FRAMES if self.one_by_one else case["frames"]
        self.videos = [_Video(case, spec, seed * 1009 + v, self.n) for v in range(nv)]
        self.net = GpuBatch(spec, nv) if "batch" in self.entry else GpuNet(spec, crops=self.entry == "crop")
        g = self.net.streams[0] if "batch" in self.entry else self.net
        if not self.one_by_one:                    # output buffers of a clip, kept by the program
            self.outs = torch.empty((self.n, nv, g.out.numel()), dtype=g.out.dtype, device="cuda")
            self.masks = torch.empty((self.n, spec.H, spec.W), dtype=torch.uint8, device="cuda") if self.entry == "masked" else None
            v = self.videos[0]
            self.dy, self.dx = [s[0] for s in v.shifts], [s[1] for s in v.shifts]
        if self.one_by_one:
            self.step()                            # the camera is running: its first frame has been through

    def __del__(self):
        if getattr(self, "net", None) is not None:
            self.net.close()

    def step(self):
        t, e, net, v = self.t, self.entry, self.net, self.videos[0]
        if self.one_by_one:
            self.t = (t + 1) % self.n
        if e == "live":
            out, reset = net.frame(v.frames[t], *v.shifts[t], None if v.forced is None else v.forced[t])
            return out, reset
        if e == "layers":
            reset = net.shift_camera(*v.shifts[t])
            mask = net.input_mask(v.frames[t], suppress=True, dilate=2)
            for i, s in enumerate(self.spec.sites):
                if s.kind != "output":
                    net.layer_forward(i, v.frames[t] if i == 0 else None, mask if i == 0 else None)
            for i in net.terminals:
                B.mdcnn_read_view(net.bufs[i], B.MDCNN_VIEW_OUT, net.out.data_ptr(), net.out.numel() * net.esize, net._stream())
            return net.out, mask, reset
        if e == "batch":
            outs, resets = net.frame([w.frames[t] for w in self.videos], [w.shifts[t][0] for w in self.videos], [w.shifts[t][1] for w in self.videos])
            return outs, resets
        if e == "batch_clip":
            _, resets = net.frames([[w.frames[f] for w in self.videos] for f in range(self.n)], [[w.shifts[f][0] for w in self.videos] for f in range(self.n)],
                                   [[w.shifts[f][1] for w in self.videos] for f in range(self.n)], outs=[list(row.unbind(0)) for row in self.outs.unbind(0)])
            return self.outs, np.array(resets)
        outs = list(self.outs[:, 0].unbind(0))
        if e == "crop":
            per, resets = net.frames_crop(v.frames, self.dy, self.dx, v.crops, outs=outs)
            n = sum(p.numel() for p in per[0])     # the crops of a video are of one size
            return self.outs[:, 0, :n], np.array(resets)
        if e == "masked":
            _, masks, resets = net.frames_masked(v.frames, self.dy, self.dx, outs=outs, masks=list(self.masks.unbind(0)), suppress=True, dilate=2)
            return self.outs, self.masks, np.array(resets)
        _, resets = net.frames(v.frames, self.dy, self.dx, None if v.forced is None else list(v.forced.unbind(0)), outs=outs)
        return self.outs, np.array(resets)


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    return state.step()


def work(case):
    """Per frame: the frame and the output once; of the state, the accumulated and the pending values of every inner site,
    read and written where a frame updates; the weights once per pass; two operations per weight and updated output."""
    spec = _spec_of(case)
    e = 2 if spec.dtype == "f16" else 4
    n = case["videos"] * (1 if case["entry"] in ("live", "layers", "batch") else case["frames"])
    d = case["density"] or DENSITY[case["net"]]
    if case["entry"] == "crop":
        d *= 4 / 9
    weights = sum(w.w.size for w in spec.edges if w.w is not None) * e
    per_frame = flops = 0
    for i, s in enumerate(spec.sites):
        h, w = spec.site_hw(i)
        per_frame += h * w * s.C * e * (2 + d if s.kind == "input" else 2 * d + 1 if s.kind == "output" else (2 if s.trunc_free else 4) * d)
    for ed in spec.edges:
        if ed.w is not None:
            h, w = spec.site_hw(ed.dst)
            flops += 2.0 * ed.w.size * (h >> ed.up) * (w >> ed.up) * d
    return {"bytes": float(n * per_frame + weights), "flops": float(n * flops)}


def tolerance(case):
    """fp16 state rounds every stored value; a sum taken in another order moves a value by a rounding, and now and then a
    pixel over its update threshold: what it would have passed on (at most about the threshold, 0.01 to 0.02) stays pending."""
    if case["dtype"] == "f16":
        return {"rel": 1e-2, "max": 0.3, "differ": 1e-4}
    return {"rel": 1e-4, "max": 0.05, "differ": 0.0}
