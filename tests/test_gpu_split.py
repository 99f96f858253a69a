"""The FP32 form's convolution on FP16 halves (kernels_split.hip): one layer
against 64-bit sums over input magnitudes, tile edges and the values its
scaling rules treat apart.

Bound: each operand keeps 22 bits (2^-23 of the value) and the product of the
two low halves is dropped (2^-22), so a product is off by 3 2^-22 of itself at
most; 9 C of them are summed in FP32 in any order.  Where a tile mixes large and
small inputs, a value is also held to 2^-31 of the tile's largest.
"""
import numpy as np
import pytest
import torch

import smlm_synth as S

pytestmark = pytest.mark.gpu


def _layer(C, d, scale=1.0, seed=5, **cfg):
    import paper_2410_02314_amd as dl
    spec = S.NetSpec("X", C, (d,))
    w = S.he_normal_weights(spec, seed, bias_std=0.0)
    w["blk0.w1"] = (w["blk0.w1"] * scale).astype(np.float32)
    return w, dl.Net(S.serialize_weights(spec, w), precision="fp32", **cfg)


def _run(net, x):
    t = torch.from_numpy(x).cuda()
    out = torch.empty_like(t)
    net.debug_conv_layer(t, None, 0, 0, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _sums(x, w, d):
    """sum w x and sum |w x| in 64 bits, NHWC."""
    n, h, wd, C = x.shape
    xp = np.zeros((n, h + 2 * d, wd + 2 * d, C))
    xp[:, d:d + h, d:d + wd] = x
    y, m = np.zeros((n, h, wd, C)), np.zeros((n, h, wd, C))
    for u in range(3):
        for v in range(3):
            t = xp[:, u * d:u * d + h, v * d:v * d + wd]
            y += t @ w[:, :, u, v].T.astype(np.float64)
            m += np.abs(t) @ np.abs(w[:, :, u, v].T.astype(np.float64))
    return y, m


def _check(got, want, C, m, w, amax=0.0):
    bound = (3 * 2.0 ** -22 + 9 * C * 2.0 ** -24) * m + 2.0 ** -31 * amax * 9 * C * float(np.abs(w).max())
    over = np.abs(got - want) > bound
    worst = float(np.max(np.abs(got - want) / np.maximum(bound, 1e-300)))
    assert not over.any(), f"{int(over.sum())} values past the bound, worst {worst:.3g} of it"


@pytest.mark.parametrize("C,d,n,h,w", [(16, 1, 2, 9, 33), (32, 3, 1, 25, 97), (48, 1, 1, 8, 32), (48, 2, 1, 37, 70),
                                       (48, 1, 1, 1, 1), (32, 1, 3, 17, 31)])
@pytest.mark.parametrize("exp", [-100, -21, 0, 15, 70])
def test_layer_against_64_bit_sums(C, d, n, h, w, exp):
    x = (np.random.default_rng(C + h).standard_normal((n, h, w, C)) * 2.0 ** exp).astype(np.float32)
    wts, net = _layer(C, d)
    y, m = _sums(x, wts["blk0.w1"], d)
    got = _run(net, x)
    _check(got, np.maximum(y, 0), C, m, wts["blk0.w1"])
    _, net4 = _layer(C, d, tile_rows=4)
    same = np.array_equal(got, _run(net4, x))
    assert same or exp in (-21, 15)                # (tiles either side of a scaling step may differ)


@pytest.mark.parametrize("C", [32, 48])
def test_small_values_beside_large_ones(C):
    rng = np.random.default_rng(7)
    x = (rng.standard_normal((1, 24, 40, C)) * 2.0 ** rng.integers(-40, 14, (1, 24, 40, C))).astype(np.float32)
    wts, net = _layer(C, 1)
    y, m = _sums(x, wts["blk0.w1"], 1)
    _check(_run(net, x), np.maximum(y, 0), C, m, wts["blk0.w1"], float(np.abs(x).max()))


@pytest.mark.parametrize("C,value", [(48, np.inf), (32, -np.inf), (48, np.nan), (16, 2.0 ** 80)])
def test_infinities_nans_and_huge_values_propagate(C, value):
    x = np.random.default_rng(3).standard_normal((1, 20, 70, C)).astype(np.float32)
    x[0, 9, 33, 5] = value
    wts, net = _layer(C, 1)
    with np.errstate(invalid="ignore"):
        y, m = _sums(x, wts["blk0.w1"], 1)
    got = _run(net, x)
    with np.errstate(invalid="ignore"):
        want = np.where(np.isnan(y), 0.0, np.maximum(y, 0))       # ReLU takes NaN to 0
    fin = np.isfinite(want) & np.isfinite(m)
    assert (got[~fin] == want[~fin].astype(np.float32)).all()
    _check(got[fin], want[fin], C, m[fin], wts["blk0.w1"], 8.0)


@pytest.mark.parametrize("scale", [2.0 ** -70, 2.0 ** 62, 2.0 ** 90])
def test_weight_magnitudes(scale):
    x = np.random.default_rng(4).standard_normal((1, 12, 40, 32)).astype(np.float32)
    wts, net = _layer(32, 1, scale)
    y, m = _sums(x, wts["blk0.w1"], 1)
    _check(_run(net, x), np.maximum(y, 0), 32, m, wts["blk0.w1"])


@pytest.mark.parametrize("exps", [(-40, 0, 12), (12, -40, 0), (0, 16, 36), (-70, -70, -70), (-30, -70, 10)])
def test_channel_groups_of_different_magnitude(exps):
    """48 channels go group by group of 16: a later group that needs another
    power of two rescales the sums so far."""
    x = np.random.default_rng(9).standard_normal((1, 19, 75, 48))
    x = (x * np.repeat([2.0 ** e for e in exps], 16)).astype(np.float32)
    wts, net = _layer(48, 1)
    y, m = _sums(x, wts["blk0.w1"], 1)
    _check(_run(net, x), np.maximum(y, 0), 48, m, wts["blk0.w1"], float(np.abs(x).max()))


@pytest.mark.parametrize("C", [16, 32, 48])
def test_unbalanced_channels(C):
    """Channels scaled by powers of two where they are made and back where they
    are read, up to 2^60 apart: the same network, and its maps to the FP32
    path's 1e-4 of |o| + rms against the FP64 oracle; a single layer still runs
    with the weights as given, and a change to BF16 and back changes nothing."""
    import oracle
    import paper_2410_02314_amd as dl
    from tests.parity import map_rel_err
    spec = S.NetSpec("X", C, (1, 2), head_outputs=5)
    w = S.he_normal_weights(spec, 21, bias_std=0.05)
    frames = S.render_frames(1, 50, 70, "tiny", 22)
    ref = oracle.net_maps_batch(frames, spec, w)
    rng = np.random.default_rng(23)
    stream, hidden = (2.0 ** rng.integers(-30, 31, (n, C)).astype(np.float32) for n in (1, 2))
    stream = stream[0]
    w["stem.w"] *= stream[:, None, None, None]
    w["stem.b"] *= stream
    for k in (0, 1):
        h = hidden[k]
        w[f"blk{k}.w1"] *= h[:, None, None, None] / stream[None, :, None, None]
        w[f"blk{k}.b1"] *= h
        w[f"blk{k}.w2"] *= stream[:, None, None, None] / h[None, :, None, None]
        w[f"blk{k}.b2"] *= stream
    w["head.w"] /= stream[None, :]
    net = dl.Net(S.serialize_weights(spec, w), precision="fp32")
    fr = torch.from_numpy(frames).cuda()

    def maps():
        m = torch.full((1, 5, 50, 70), float("nan"), dtype=torch.float32, device="cuda")
        net.maps_device(fr, m)
        torch.cuda.synchronize()
        return m.cpu().numpy()

    a = maps()
    assert map_rel_err(a, ref).max() <= 1e-4
    x = (rng.standard_normal((1, 12, 40, C)) * stream).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    out = torch.empty_like(t)
    net.debug_conv_layer(t, None, 1, 0, out)
    torch.cuda.synchronize()
    y, m = _sums(x, w["blk1.w1"], 2)
    y, m = y + w["blk1.b1"], m + np.abs(w["blk1.b1"])
    top = np.abs(x).max() * np.abs(w["blk1.w1"]).max(axis=(1, 2, 3)) * 9 * C
    assert (np.abs(out.cpu().numpy() - np.maximum(y, 0)) <= 1e-4 * m + 2.0 ** -30 * top).all()
    net.set_config(precision="bf16")
    maps()
    net.set_config(precision="fp32")
    assert np.array_equal(maps(), a)
