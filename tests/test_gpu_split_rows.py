"""The FP32 form's tiles of 4 and of 8 rows give the same bits whatever the
inputs' magnitudes: tiles of 4 rows take the power of two of the tile of 8 rows
they are half of.  So a frame's maps do not depend on the batch around it, which
decides the rows, nor on the entry point.
"""
import numpy as np
import pytest
import torch

import smlm_synth as S
from tests.test_gpu_split import _layer, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,d,n,h,w", [(16, 1, 1, 1, 1), (16, 3, 2, 13, 101), (32, 1, 2, 9, 33), (32, 2, 1, 40, 70),
                                       (32, 1, 1, 21, 64), (48, 1, 1, 12, 65), (48, 2, 2, 37, 70)])
def test_layer(C, d, n, h, w):
    rng = np.random.default_rng(61)
    x = (rng.standard_normal((n, h, w, C)) * 2.0 ** rng.integers(-40, 14, (n, h, w, 1))).astype(np.float32)
    out = [_run(_layer(C, d, tile_rows=r)[1], x) for r in (4, 8)]
    assert np.array_equal(out[0], out[1])


def _maps(net, frames):
    fr = torch.from_numpy(frames).cuda()
    m = torch.full((len(frames), net.head_outputs, *frames.shape[1:]), float("nan"), dtype=torch.float32, device="cuda")
    net.maps_device(fr, m)
    torch.cuda.synchronize()
    return m.cpu().numpy()


@pytest.mark.parametrize("C,dil,nh", [(16, (1, 2), 10), (32, (1, 2, 4), 5), (32, (2, 16), 10), (48, (1, 4), 5)])
@pytest.mark.parametrize("scale", [2.0 ** -20, 1.0, 2.0 ** 9])
def test_frame_in_any_batch(C, dil, nh, scale):
    """One frame alone (tiles of 4 rows to 32 channels), with either tile, in a
    batch of many tiles, and as a region of interest replayed by a graph."""
    import paper_2410_02314_amd as dl
    spec = S.NetSpec("X", C, dil, head_outputs=nh)
    w = S.he_normal_weights(spec, 62, bias_std=0.05)
    for k in w:
        if k.endswith("b") or ".b" in k:
            w[k] = (w[k] * scale).astype(np.float32)
    blob = S.serialize_weights(spec, w)
    rng = np.random.default_rng(63)
    h, wd = 70, 130
    frames = rng.integers(0, 3, (40, h, wd)).astype(np.uint16)
    spots = rng.random(frames.shape) < 0.002
    frames[spots] = (2 ** rng.integers(3, 16, int(spots.sum()))).astype(np.uint16)
    cfg = dict(precision="fp32", gain=1.0, offset=0.0, in_scale_override=scale)
    alone = _maps(dl.Net(blob, **cfg), frames[:1])
    assert not np.isnan(alone).any()
    for rows in (4, 8):
        assert np.array_equal(_maps(dl.Net(blob, tile_rows=rows, **cfg), frames[:1]), alone)
    net = dl.Net(blob, **cfg)
    assert np.array_equal(_maps(net, frames)[:1], alone)
    fr = torch.from_numpy(frames[:1]).cuda()
    out = torch.zeros((h * wd, 8), dtype=torch.int32, device="cuda")
    counts = torch.zeros(3, dtype=torch.int32, device="cuda")
    net.localize_device(fr, out, counts)
    torch.cuda.synchronize()
    eager = out[:int(counts[1])].cpu().numpy().copy()
    g = net.graph_rois_dynamic(2, 128, 256, 128 * 256, out, counts)
    g.launch_rois([fr[0]])
    torch.cuda.synchronize()
    assert np.array_equal(out[:int(counts[1])].cpu().numpy(), eager)
