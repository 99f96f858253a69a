"""Range of the FP16 pairs (split_common.h): small inputs beside large ones keep
their bits.

Bound: a tile's inputs share the power of two that brings the largest into
[2^14, 2^15).  A value down to 2^-28 of it keeps 22 bits (2^-23 of itself), and
the dropped product of the low halves is 2^-22 of the product: 3 2^-22 a product,
9 C of them added in FP32 in any order; smaller values are held to 2^-50 of the
largest.
"""
import dataclasses

import numpy as np
import pytest
import torch

import smlm_synth as S
from tests.test_gpu_split import _layer, _run, _sums

pytestmark = pytest.mark.gpu


def _check(got, x, w, d=1):
    C = x.shape[-1]
    y, m = _sums(x, w, d)
    bound = (3 * 2.0 ** -22 + 9 * C * 2.0 ** -24) * m + 2.0 ** -50 * float(np.abs(x).max()) * 9 * C * np.abs(w).max()
    worst = float(np.max(np.abs(got - np.maximum(y, 0)) / np.maximum(bound, 1e-300)))
    assert worst <= 1.0, f"worst {worst:.3g} of the bound"


@pytest.mark.parametrize("C", [16, 32, 48])
@pytest.mark.parametrize("top", [31.0, 33000.0, 4.0e6, 1.0e12])
def test_one_bright_value(C, top):
    """One value far above the others of its tile; while it is less than 2^28 above
    them, the sums that do not take it are as accurate as without it."""
    x = np.random.default_rng(51).standard_normal((1, 16, 64, C)).astype(np.float32)
    x[0, 5, 20, 3] = top
    wts, net = _layer(C, 1)
    got, w = _run(net, x), wts["blk0.w1"]
    _check(got, x, w)
    far = np.ones((16, 64), bool)
    far[4:7, 19:22] = False
    y, m = _sums(x, w, 1)
    err = np.abs(got - np.maximum(y, 0))[0][far]
    err = np.maximum(err - 2.0 ** -50 * top * 9 * C * np.abs(w).max() * (top > 2.0 ** 28), 0)
    assert np.sqrt(np.mean((err / m[0][far]) ** 2)) <= 2.0 ** -24      # (one FP32 rounding of sum |w x|)


@pytest.mark.parametrize("C,exp", [(32, -20), (48, -20), (48, -24)])
def test_a_faint_channel_read_alone(C, exp):
    """A channel far below the others which one output reads alone."""
    x = np.random.default_rng(52).standard_normal((1, 17, 40, C)).astype(np.float32)
    x[..., 5] *= np.float32(2.0 ** exp)
    wts, net = _layer(C, 1)
    w = wts["blk0.w1"]
    only = w[2].copy()
    w[2] = 0
    w[2, 5] = only[5]
    import paper_2410_02314_amd as dl
    net = dl.Net(S.serialize_weights(S.NetSpec("X", C, (1,)), wts), precision="fp32")
    got = _run(net, x)
    y, m = _sums(x, w, 1)
    err, ref = np.abs(got - np.maximum(y, 0))[..., 2], m[..., 2]
    assert (err <= (3 * 2.0 ** -22 + 9 * 2.0 ** -24) * ref).all(), float((err / ref).max())


@pytest.mark.parametrize("C", [16, 32, 48])
def test_faint_weights_on_a_bright_channel(C):
    """One output reads a bright channel with weights as far below its others."""
    import paper_2410_02314_amd as dl
    x = np.random.default_rng(55).standard_normal((1, 17, 40, C)).astype(np.float32)
    x[..., 5] *= np.float32(2.0 ** 22)
    wts, _ = _layer(C, 1)
    w = wts["blk0.w1"]
    w[2, 5] *= np.float32(2.0 ** -22)
    got = _run(dl.Net(S.serialize_weights(S.NetSpec("X", C, (1,)), wts), precision="fp32"), x)
    y, m = _sums(x, w, 1)
    err, ref = np.abs(got - np.maximum(y, 0))[..., 2], m[..., 2]
    assert np.sqrt(np.mean((err / ref) ** 2)) <= 2.0 ** -24, float((err / ref).max())


@pytest.mark.parametrize("spec", [S.DenseSpec("X", 32, (1,), 2, 16), S.DenseSpec("X", 16, (1,), 3, 16)])
def test_dense_layers_beside_a_bright_spot(spec):
    """Maps of a frame with one saturated pixel, away from it but in its tiles:
    the mean error is that of FP32 rounding (2^-20 of the maps' rms for the stem,
    three or four layers and the head)."""
    import oracle
    import paper_2410_02314_amd as dl
    w = S.he_normal_weights(spec, 53, bias_std=0.05)
    frames = np.random.default_rng(54).integers(0, 2, (1, 24, 64)).astype(np.uint16)
    frames[0, 3, 16] = 65535
    kw = dict(gain=1.0, offset=0.0, in_scale_override=1.0)
    net = dl.Net(S.serialize_weights(spec, w), precision="fp32", **kw)
    fr = torch.from_numpy(frames).cuda()
    m = torch.zeros((1, net.head_outputs, 24, 64), dtype=torch.float32, device="cuda")
    net.maps_device(fr, m)
    torch.cuda.synchronize()
    ref = oracle.net_maps_batch(frames, dataclasses.replace(spec, in_scale=1.0), w, gain=1.0, offset=0.0)
    far = np.zeros((24, 64), bool)
    far[:8, :32] = True                                     # the bright pixel's tile
    far[:, 10:23] = False
    err = (m.cpu().numpy().astype(np.float64) - ref)[0][:, far]
    rel = np.sqrt((err ** 2).mean(1)) / np.sqrt((ref[0][:, far] ** 2).mean(1))
    assert rel.max() <= 2.0 ** -20, rel
