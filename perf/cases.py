"""Performance cases of the localization library: what its users have it do.

Each case is one call (or one training pass) through the Python binding's
public entry points on synthetic camera frames: full-frame localization in the
four arithmetic forms, the small and single-frame calls where latency counts,
uneven ROI batches, host frames through the pipelined path, the
dense-connection networks and training gradients.  Sizes follow the
repository's own benchmark workloads (128^2 to 2048^2 frames, ROI sides 128 to
1024, 16 x 128^2 training batches) and odd sizes between them.

    listed()             the fixed cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, network handle and output buffers on the GPU
    run(state)           one pass; its outputs
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    the outputs in 64-bit arithmetic (torch only)
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2410_02314_amd as dl
import smlm_synth as S

# weight seeds the repository's benchmark uses (their heads are calibrated)
NET_SEED = {"A": 1, "AU": 1, "B": 2, "BU": 2, "D": 3, "DU": 3, "DT": 3, "DUT": 3}
# The most pixels of a listed or drawn case whose emitter records are compared
# in the FP32-grade forms: whether a pixel is a detection is a comparison, and
# on frames much larger than this some pixel sits within rounding of it.
RECORD_PIXELS = 1 << 20


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: a graph-captured batch of small frames, replayed
        # over a buffer that the acquisition refills
        dict(name="tiny_graph_A_fp32", call="graph", net="A", precision="fp32", n=4, h=128, w=128, camera="scalar"),
        # one odd-sized camera frame as it arrives, emitters with uncertainties
        dict(name="frame_BU_fp32", call="localize", net="BU", precision="fp32", n=1, h=333, w=517, camera="scalar"),
        # full sCMOS frames, the exact form (the headline path)
        dict(name="full_B_fp32", call="maps", net="B", precision="fp32", n=4, h=2048, w=2048, camera="scmos"),
        # ragged frames in split BF16, the FP32-grade form on the BF16 cores
        dict(name="ragged_B_bf16x3", call="maps", net="B", precision="bf16x3", n=2, h=1187, w=1501, camera="scalar"),
        # full sCMOS frames in the two reduced-precision forms
        dict(name="full_B_bf16", call="maps", net="B", precision="bf16", n=4, h=2048, w=2048, camera="scmos"),
        dict(name="full_B_fp8", call="localize", net="B", precision="fp8", n=4, h=2048, w=2048, camera="scmos"),
        # regions of interest cut from frames, uneven sides
        dict(name="rois_A_fp32", call="rois", net="A", precision="fp32", n=40, h=1024, w=1024, camera="scalar"),
        # host frames, copies overlapped with compute, records back to the host
        dict(name="host_A_bf16", call="host", net="A", precision="bf16", n=4, h=512, w=512, camera="scalar"),
        # the dense-connection network, without and with the U-Net
        dict(name="dense_D_fp32", call="maps", net="D", precision="fp32", n=2, h=1024, w=1024, camera="scalar"),
        dict(name="ragged_DU_fp32", call="maps", net="DU", precision="fp32", n=1, h=701, w=903, camera="scalar"),
        # training: loss and every weight gradient of one batch
        dict(name="train_AU", call="train", net="AU", precision="fp32", n=16, h=128, w=128, camera="scalar"),
        dict(name="train_DUT", call="train", net="DUT", precision="fp32", n=8, h=128, w=128, camera="scalar"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    call = rng.choice(["maps", "maps", "maps", "localize", "graph", "rois", "host", "dense", "dense", "train"])
    if call == "train":
        return dict(call="train", net=rng.choice(["AU", "DT", "DUT"]), precision="fp32", n=_log_int(rng, 2, 16),
                    h=_log_int(rng, 48, 160), w=_log_int(rng, 48, 160), camera="scalar")
    if call == "dense":
        h, w = _log_int(rng, 64, 1400), _log_int(rng, 64, 1400)
        return dict(call="maps", net=rng.choice(["D", "DU"]), precision="fp32", n=max(1, _log_int(rng, 1, 2000000 // (h * w) + 1)),
                    h=h, w=w, camera="scalar")
    precision = rng.choice(["fp32", "fp32", "bf16x3", "bf16", "fp8"])
    # (split BF16 has no 10-output head at 48 channels)
    net = rng.choice(["A", "B", "B", "AU", "BU"] if precision != "bf16x3" else ["A", "B", "B", "AU"])
    # records of the FP32-grade forms are compared on smaller batches (see
    # RECORD_PIXELS); capturing a graph is for small ones too
    most = 8 << 20
    if call in ("localize", "host", "graph") and precision in ("fp32", "bf16x3") or call == "graph":
        most = RECORD_PIXELS // 4
    if call == "host":
        net = rng.choice(["A", "B"])
        most = min(most, 2 << 20)
    if call == "rois":
        return dict(call="rois", net=net, precision=precision, n=_log_int(rng, 2, 24), h=_log_int(rng, 160, 1024),
                    w=_log_int(rng, 160, 1024), camera="scalar")
    side = min(2048, int(math.sqrt(most)))
    h, w = _log_int(rng, 72, side), _log_int(rng, 72, side)
    n = _log_int(rng, 1, min(16, max(1, most // (h * w))))
    camera = "scmos" if call in ("maps", "localize") and rng.random() < 0.5 else "scalar"
    return dict(call=call, net=net, precision=precision, n=n, h=h, w=w, camera=camera)


HOST_BATCHES = 3


def _roi_shapes(case):
    """Uneven sides from 128 to the case's h and w, set by the case alone."""
    rng = random.Random(case["n"] * 1000003 + case["h"] * 1009 + case["w"])
    return [(_log_int(rng, 128, case["h"]), _log_int(rng, 128, case["w"])) for _ in range(case["n"])]


def _pixels(case):
    if case["call"] == "rois":
        return sum(h * w for h, w in _roi_shapes(case))
    return case["n"] * case["h"] * case["w"] * (HOST_BATCHES if case["call"] == "host" else 1)


# ------------------------------------------------------------------ inputs
def _render(n, h, w, seed, scmos=None, astig=False):
    """Seeded frames on the GPU: emitters at random positions, 1 per um^2 at
    100 nm pixels, pixel-integrated Gaussian (or astigmatic) spots, Poisson
    noise on spots and background, read noise, ADU.  Returns uint16 [n][h][w]
    and the emitters as (frame, x, y, z_nm, photons) columns, frame by frame.
    Spot photons are summed as integers (1e-4 photons), so the result does not
    depend on the order of the additions."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)

    def uniform(m, lo, hi):
        return torch.rand(m, generator=g, device=dev, dtype=torch.float64) * (hi - lo) + lo

    m = max(n, int(round(n * h * w * 0.01)))
    f = torch.sort((torch.rand(m, generator=g, device=dev, dtype=torch.float64) * n).floor())[0]
    x, y = uniform(m, 0.0, w), uniform(m, 0.0, h)
    if astig:
        z = uniform(m, -700.0, 700.0)
        ph = 3000.0 * torch.exp(0.5 * torch.randn(m, generator=g, device=dev, dtype=torch.float64))
        sx = 1.3 * torch.sqrt(1 + ((z - 250.0) / 400.0) ** 2)
        sy = 1.3 * torch.sqrt(1 + ((z + 250.0) / 400.0) ** 2)
    else:
        z = torch.zeros(m, device=dev, dtype=torch.float64)
        ph = uniform(m, 1000.0, 5000.0)
        sx = sy = torch.full((m,), 1.3, device=dev, dtype=torch.float64)
    R = 8 if astig else 6
    k = torch.arange(-R, R + 1, device=dev, dtype=torch.float64)
    rate = torch.zeros(n * h * w, dtype=torch.int64, device=dev)
    for at in range(0, m, 65536):
        e = slice(at, min(m, at + 65536))

        def axis(c, s):
            p = c.floor()[:, None] + k
            lo, hi = (p - c[:, None]) / s[:, None], (p + 1 - c[:, None]) / s[:, None]
            return p.long(), 0.5 * (torch.erf(hi / math.sqrt(2.0)) - torch.erf(lo / math.sqrt(2.0)))
        px, gx = axis(x[e], sx[e])
        py, gy = axis(y[e], sy[e])
        v = (ph[e][:, None, None] * gy[:, :, None] * gx[:, None, :] * 1e4).round().long()
        ok = ((py >= 0) & (py < h))[:, :, None] & ((px >= 0) & (px < w))[:, None, :]
        idx = (f[e].long()[:, None, None] * h + py[:, :, None]) * w + px[:, None, :]
        rate.index_add_(0, torch.where(ok, idx, 0).reshape(-1), torch.where(ok, v, 0).reshape(-1))
    frames = torch.empty((n, h, w), dtype=torch.int16, device=dev)
    for i in range(n):
        photons = torch.poisson(rate[i * h * w:(i + 1) * h * w].reshape(h, w).float() * 1e-4 + 100.0, generator=g)
        noise = torch.randn((h, w), generator=g, device=dev) * 1.5
        gain, offset = scmos if scmos is not None else (0.5, 100.0)
        adu = (photons / gain + offset + noise).round().clamp(0, 65535)
        frames[i] = adu.to(torch.int32).to(torch.int16)
    return frames.view(torch.uint16), (f, x, y, z, ph)


def _camera(case, seed):
    if case["camera"] != "scmos":
        return None
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed ^ 0x5C)
    shape = (case["h"], case["w"])
    gain = 0.5 * (1 + 0.05 * torch.randn(shape, generator=g, device="cuda:0").clamp(-4, 4))
    offset = 100.0 + 3.0 * torch.randn(shape, generator=g, device="cuda:0")
    return gain, offset


def _inputs(case, seed):
    """(frames or ROI list, camera maps, emitters): from the case and seed alone."""
    cam = _camera(case, seed)
    astig = case["net"][0] == "B"
    if case["call"] == "rois":
        shapes = _roi_shapes(case)
        side_h, side_w = case["h"], case["w"]
        # ROIs cut out of larger frames: rows keep the frame's stride
        nf = max(1, (len(shapes) + 7) // 8)
        frames, _ = _render(nf, side_h, side_w, seed, None, astig)
        rng = random.Random(seed)
        rois = []
        for i, (h, w) in enumerate(shapes):
            y, x = rng.randint(0, side_h - h), rng.randint(0, side_w - w)
            rois.append(frames[i % nf, y:y + h, x:x + w])
        return rois, None, None
    n = case["n"] * (HOST_BATCHES if case["call"] == "host" else 1)
    frames, em = _render(n, case["h"], case["w"], seed, cam, astig)
    return frames, cam, em


def _truth(em, n, h, w):
    f, x, y, z, ph = em
    off = torch.searchsorted(f, torch.arange(n + 1, device=f.device, dtype=f.dtype)).to(torch.int32)
    return torch.stack([x, y, z, ph], 1).float().contiguous(), off


def _host_cap(case):
    return max(1024, _pixels(case) // 48)


def prepare(case, seed):
    spec, weights = S.make_net(case["net"], NET_SEED[case["net"]])
    net = dl.Net(S.serialize_weights(spec, weights), precision=case["precision"])
    frames, cam, em = _inputs(case, seed)
    if cam is not None:
        net.set_camera_maps(cam[0].cpu().numpy(), cam[1].cpu().numpy())
    n, h, w, nh, call = case["n"], case["h"], case["w"], spec.head_outputs, case["call"]
    dev = torch.device("cuda:0")
    s = dict(call=call, net=net, frames=frames, nh=nh)
    if call == "maps":
        s["maps"] = torch.empty((n, nh, h, w), dtype=torch.float32, device=dev)
    elif call == "rois":
        s["maps"] = torch.empty(nh * _pixels(case), dtype=torch.float32, device=dev)
    elif call in ("localize", "graph"):
        cap = max(1024, n * h * w // 24)
        s["out"] = torch.zeros((cap, 8), dtype=torch.int32, device=dev)
        s["counts"] = torch.zeros(n + 1, dtype=torch.int32, device=dev)
        if call == "graph":
            s["graph"] = net.graph(frames, s["out"], s["counts"])
        elif nh == 10:
            s["unc"] = torch.zeros((cap, 5), dtype=torch.float32, device=dev)
    elif call == "host":
        host = frames.view(torch.int16).cpu().numpy().view(np.uint16)
        s["frames"] = host.reshape(HOST_BATCHES, n, h, w)
        # the program's own table of emitters, filled from each call's records
        s["place"] = np.zeros((_host_cap(case), 3), np.int32)
        s["values"] = np.zeros((_host_cap(case), 5), np.float32)
    elif call == "train":
        s["truth"], s["off"] = _truth(em, n, h, w)
        s["grad"] = torch.empty(net.nparams, dtype=torch.float32, device=dev)
        s["loss"] = torch.zeros(4, dtype=torch.float32, device=dev)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    net, call = s["net"], s["call"]
    if call == "maps":
        net.maps_device(s["frames"], s["maps"])
        return {"maps": s["maps"]}
    if call == "rois":
        net.maps_rois_device(s["frames"], s["maps"])
        return {"maps": s["maps"]}
    if call == "host":
        rec = net.localize_pipelined(s["frames"])
        m = min(len(rec), len(s["place"]))
        for i, k in enumerate(("frame", "row", "col")):
            s["place"][:m, i] = rec[k][:m]
        for i, k in enumerate(("x_px", "y_px", "z_nm", "photons", "prob")):
            s["values"][:m, i] = rec[k][:m]
        return {"place": s["place"], "values": s["values"], "count": len(rec)}
    if call == "train":
        net.train_grad(s["frames"], s["truth"], s["off"], s["grad"], s["loss"])
        return {"grad": s["grad"], "loss": s["loss"]}
    if call == "graph":
        s["graph"].launch()
    elif "unc" in s:
        net.localize_device_unc(s["frames"], s["out"], s["unc"], s["counts"])
    else:
        net.localize_device(s["frames"], s["out"], s["counts"])
    r = {"place": s["out"][:, :3], "values": s["out"].view(torch.float32)[:, 3:], "counts": s["counts"]}
    if "unc" in s:
        r["unc"] = s["unc"]
    return r


# ------------------------------------------------------------------ needed work
def work(case):
    spec = S.NETS[case["net"]]
    px = _pixels(case)
    flops = S.net_flops_per_px(spec) * px
    params = S.param_count(spec)
    if case["call"] == "train":
        return {"bytes": 2 * px + 2 * 4 * params, "flops": 3 * flops}
    out = 4 * spec.head_outputs * px if case["call"] in ("maps", "rois") else 32 * px // 100
    cam = 8 * case["h"] * case["w"] if case["camera"] == "scmos" else 0
    return {"bytes": 2 * px + out + cam + 4 * params, "flops": flops}


# ------------------------------------------------------------------ in 64 bits
def _conv(x, w, b, d):
    """3x3 convolution at dilation d with zero padding: nine products."""
    n, c, h, wd = x.shape
    xp = torch.nn.functional.pad(x, (d, d, d, d))
    y = b[None, :, None]
    for u in range(3):
        for v in range(3):
            y = y + torch.matmul(w[:, :, u, v], xp[:, :, u * d:u * d + h, v * d:v * d + wd].reshape(n, c, h * wd))
    return y.reshape(n, -1, h, wd)


def _point(x, w, b):
    n, c, h, wd = x.shape
    return (torch.matmul(w, x.reshape(n, c, h * wd)) + b[None, :, None]).reshape(n, -1, h, wd)


def _forward(x, spec, W):
    """Maps [n][nh][h][w] of network input x [n][1][h][w]."""
    a = torch.relu(_conv(x, W["stem.w"], W["stem.b"], 1))
    if not hasattr(spec, "layers"):
        for k, d in enumerate(spec.dilations):
            t = torch.relu(_conv(a, W[f"blk{k}.w1"], W[f"blk{k}.b1"], d))
            a = torch.relu(a + _conv(t, W[f"blk{k}.w2"], W[f"blk{k}.b2"], d))
        return _point(a, W["head.w"], W["head.b"])
    for k, d in enumerate(spec.dilations):
        cat = a
        for i in range(spec.layers):
            cat = torch.cat([cat, torch.relu(_conv(cat, W[f"blk{k}.l{i}.w"], W[f"blk{k}.l{i}.b"], d))], 1)
        a = torch.relu(_point(cat, W[f"blk{k}.t.w"], W[f"blk{k}.t.b"]))
    if spec.unet:
        def pool(v):
            h, w = v.shape[2:]
            v = torch.nn.functional.pad(v, (0, w % 2, 0, h % 2), value=-math.inf)
            return v.reshape(*v.shape[:2], v.shape[2] // 2, 2, v.shape[3] // 2, 2).amax((3, 5))

        def up(v, like):
            return v.repeat_interleave(2, 2).repeat_interleave(2, 3)[:, :, :like.shape[2], :like.shape[3]]
        d1 = torch.relu(_conv(pool(a), W["unet.d1.w"], W["unet.d1.b"], 1))
        d2 = torch.relu(_conv(pool(d1), W["unet.d2.w"], W["unet.d2.b"], 1))
        u1 = torch.relu(_conv(torch.cat([d1, up(d2, d1)], 1), W["unet.u1.w"], W["unet.u1.b"], 1))
        a = torch.relu(_conv(torch.cat([a, up(u1, a)], 1), W["unet.u0.w"], W["unet.u0.b"], 1))
    return _point(a, W["head.w"], W["head.b"])


def _network_input(frame, cam, spec):
    adu = (frame.view(torch.int16).to(torch.int32) & 0xFFFF).double()
    gain, offset = (c.double() for c in cam) if cam is not None else (0.5, 100.0)
    return (adu - offset) * gain * spec.in_scale


def _records(maps, frame, spec):
    """(place, values, unc) of one frame's maps, in raster order; None where a
    pixel's detection is too close a decision to be told by the maps alone."""
    l = maps[0]
    tau = math.log(0.3 / 0.7)
    p = torch.nn.functional.pad(l[None, None], (1, 1, 1, 1), value=-math.inf)[0, 0]
    h, w = l.shape
    near = torch.stack([p[u:u + h, v:v + w] for u in range(3) for v in range(3) if (u, v) != (1, 1)]).amax(0)
    close = (((l - near).abs() < 1e-5) & (l > tau)) | (((l - tau).abs() < 1e-5) & (l > near))
    if bool(close.any()):
        return None
    yx = ((l > tau) & (l > near)).nonzero()
    v = maps[:, yx[:, 0], yx[:, 1]]
    place = torch.cat([torch.full_like(yx[:, :1], frame), yx], 1)
    values = torch.stack([yx[:, 1] + 0.5 + v[1], yx[:, 0] + 0.5 + v[2], v[3] * spec.z_scale, v[4] * spec.ph_scale,
                          torch.sigmoid(v[0])], 1)
    unc = None
    if maps.shape[0] == 10:
        sp = torch.nn.functional.softplus(v[5:], threshold=100.0)
        unc = torch.stack([sp[0] + 0.01, sp[1] + 0.01, (sp[2] + 0.01) * spec.z_scale, (sp[3] + 0.01) * spec.ph_scale,
                           sp[4] / spec.in_scale], 1)
    return place, values, unc


def _loss(maps, truth, off):
    """[total, cross-entropy, count, localisation], each the mean over frames."""
    n, _, h, w = maps.shape
    sp = torch.nn.functional.softplus
    col = torch.arange(w, device=maps.device, dtype=torch.float64)[None, :].expand(h, w)
    row = torch.arange(h, device=maps.device, dtype=torch.float64)[:, None].expand(h, w)
    terms = []
    for i in range(n):
        m, t = maps[i], truth[off[i]:off[i + 1]]
        l, p = m[0], torch.sigmoid(m[0])
        occ = torch.zeros((h, w), dtype=torch.float64, device=maps.device)
        occ[t[:, 1].floor().long(), t[:, 0].floor().long()] = 1.0
        bce = (sp(l, threshold=100.0) - occ * l).mean()
        mu, var = p.sum(), (p * (1 - p)).sum() + 1e-4
        count = 0.5 * torch.log(2 * math.pi * var) + (len(t) - mu) ** 2 / (2 * var)
        mean = torch.stack([col + 0.5 + m[1], row + 0.5 + m[2], m[3], m[4]]).reshape(4, -1)
        sd = (sp(m[5:9], threshold=100.0) + 0.01).reshape(4, -1)
        logw = (-sp(-l, threshold=100.0) - torch.log(mu)).reshape(-1)
        loc = torch.zeros((), dtype=torch.float64, device=maps.device)
        if len(t):
            q = (-0.5 * ((t[:, :, None] - mean) / sd) ** 2 - torch.log(sd) - 0.5 * math.log(2 * math.pi)).sum(1)
            loc = -torch.logsumexp(q + logw, 1).sum()
        terms.append(torch.stack([bce + count + loc, bce, count, loc]))
    return torch.stack(terms).mean(0)


def exact(case, seed):
    spec, weights = S.make_net(case["net"], NET_SEED[case["net"]])
    call = case["call"]
    if case["precision"] == "fp8" or (call not in ("maps", "rois", "train") and case["precision"] == "bf16"):
        return None                       # FP8 activations, and BF16 detections, are their own forms' values
    W = {k: torch.from_numpy(v).cuda().double() for k, v in weights.items()}
    frames, cam, em = _inputs(case, seed)
    n, h, w = case["n"], case["h"], case["w"]
    if call == "rois":
        return {"maps": torch.cat([_forward(_network_input(r, None, spec)[None, None], spec, W).reshape(-1) for r in frames])}
    if call == "train":
        truth, off = _truth(em, n, h, w)
        t = truth.double() / torch.tensor([1.0, 1.0, spec.z_scale, spec.ph_scale], device=truth.device, dtype=torch.float64)
        off = off.tolist()
        names = [k for k, _ in S.tensor_layout(spec)]
        for k in names:
            W[k].requires_grad_(True)
        grad = torch.zeros(S.param_count(spec), dtype=torch.float64, device="cuda:0")
        loss = torch.zeros(4, dtype=torch.float64, device="cuda:0")
        for i in range(n):                # frame by frame: gradients are means over frames
            maps = _forward(_network_input(frames[i], cam, spec)[None, None], spec, W)
            li = _loss(maps, t[off[i]:off[i + 1]], [0, off[i + 1] - off[i]]) / n
            g = torch.autograd.grad(li[0], [W[k] for k in names], allow_unused=True)
            grad += torch.cat([(torch.zeros_like(W[k]) if x is None else x).reshape(-1) for k, x in zip(names, g)])
            loss += li.detach()
        return {"grad": grad, "loss": loss}
    n *= HOST_BATCHES if call == "host" else 1
    if call == "maps":
        return {"maps": torch.cat([_forward(_network_input(frames[i], cam, spec)[None, None], spec, W) for i in range(n)])}
    found = [_records(_forward(_network_input(frames[i], cam, spec)[None, None], spec, W)[0], i, spec) for i in range(n)]
    if any(f is None for f in found):
        return None
    values = torch.cat([f[1] for f in found])
    if call == "host":
        cap = _host_cap(case)
    else:
        cap = max(1024, n * h * w // 24)

    def filled(v):
        r = torch.zeros((cap, 5), dtype=torch.float64, device=v.device)
        r[:min(cap, len(v))] = v[:cap]
        return r
    if call == "host":
        return {"place": None, "values": filled(values), "count": None}
    r = {"place": None, "values": filled(values), "counts": None}
    if call == "localize" and spec.head_outputs == 10:
        r["unc"] = filled(torch.cat([f[2] for f in found]))
    return r
