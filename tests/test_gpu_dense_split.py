"""The dense networks' layers on the FP16 pairs (kernels_dsplit.hip) at the
sizes and values their code treats apart, against the FP64 oracle.

Bound: each operand keeps 22 bits and the product of the two low halves is
dropped, 3 2^-22 of a product at most; the deepest net here has 29
convolutions after one another, so 29 x 3 2^-22 = 2.1e-5 of |o| + rms with
He-normal weights (which keep the magnitudes), inside the FP32 path's 1e-4.
Where a tile mixes large and small channels a value is also held to 2^-31 of
the tile's largest: 2^-19 of a channel 2^12 below it.
"""
import numpy as np
import pytest
import torch

import oracle
import smlm_synth as S
from tests.parity import map_rel_err

pytestmark = pytest.mark.gpu
TOL = 1e-4


def _maps(spec, w, frames, **cfg):
    import paper_2410_02314_amd as dl
    net = dl.Net(S.serialize_weights(spec, w), **cfg)
    n, h, wd = frames.shape
    maps = torch.full((n, net.head_outputs, h, wd), float("nan"), dtype=torch.float32, device="cuda")
    net.maps_device(torch.from_numpy(frames).cuda(), maps)
    torch.cuda.synchronize()
    return maps.cpu().numpy()


# (C, growth, layers, dilations, U-Net): weights resident and streamed (more
# than 160 KB of them), one and two blocks of outputs, one and two of the
# transition, one layer a block, dilations with and without a phase layout
@pytest.mark.parametrize("C,G,L,dil,unet", [(32, 32, 8, (1, 2, 4), 0), (32, 16, 8, (2, 3), 2), (16, 16, 1, (4, 1), 0),
                                            (16, 32, 6, (5, 16), 0), (32, 32, 1, (8,), 2), (16, 16, 8, (3,), 0)])
@pytest.mark.parametrize("queue", [0, 1, 2])
def test_forms(C, G, L, dil, unet, queue):
    spec = S.DenseSpec("X", C, dil, layers=L, growth=G, unet=unet)
    w = S.he_normal_weights(spec, 11, bias_std=0.05)
    frames = S.render_frames(2, 45, 83, "tiny", 17)
    got = _maps(spec, w, frames, tile_queue=queue)
    assert map_rel_err(got, oracle.net_maps_batch(frames, spec, w)).max() <= TOL


@pytest.mark.parametrize("e", [-100, -80, -40, 16, 40, 80, 100])
@pytest.mark.parametrize("unet", [0, 2])
def test_magnitudes(e, unet):
    """The first block's values 2^e times as large, its transition's weights
    2^-e times: other exponents of the tiles and weights, and (from 2^75, below
    2^-60) the plain FP32 tiles; the maps stay what they were."""
    spec = S.DenseSpec("X", 32, (2, 1), layers=2, growth=16, unet=unet)
    w = S.he_normal_weights(spec, 12)
    frames = S.render_frames(1, 40, 70, "tiny", 18)
    ref = oracle.net_maps_batch(frames, spec, w)
    w["stem.w"] = w["stem.w"] * np.float32(2.0 ** e)
    w["blk0.t.w"] = w["blk0.t.w"] * np.float32(2.0 ** -e)
    assert map_rel_err(_maps(spec, w, frames), ref).max() <= TOL


@pytest.mark.parametrize("e0,e1", [(12, 0), (0, 12), (-12, 0), (0, -12), (30, 30)])
def test_planes_of_different_magnitude(e0, e1):
    """A layer's input plane 2^e times another's: the sums change their exponent
    at the plane that needs it."""
    spec = S.DenseSpec("X", 16, (2, 1), layers=3, growth=16)
    w = S.he_normal_weights(spec, 13)
    frames = S.render_frames(1, 40, 70, "tiny", 19)
    ref = oracle.net_maps_batch(frames, spec, w)
    for b in (0, 1):
        for i, e in ((0, e0), (1, e1)):
            w[f"blk{b}.l{i}.w"] = w[f"blk{b}.l{i}.w"] * np.float32(2.0 ** e)
            lo = 16 + 16 * i
            for name in [f"blk{b}.l{k}.w" for k in range(i + 1, 3)] + [f"blk{b}.t.w"]:
                w[name][:, lo:lo + 16] *= np.float32(2.0 ** -e)
    assert map_rel_err(_maps(spec, w, frames), ref).max() <= TOL


@pytest.mark.parametrize("dil", [(2,), (4, 1), (8, 3, 2)])
@pytest.mark.parametrize("n,h,w", [(1, 164, 150), (3, 70, 101)])
def test_unet_wider_than_the_blocks(dil, n, h, w):
    """One layer of 16 channels a block: the U-Net's level-0 concatenation (64
    channels) is wider than a block's (48), in either of the two buffers."""
    import paper_2410_02314_amd as dl
    from tests.parity import compare_emitters
    spec = S.DenseSpec("X", 32, dil, layers=1, growth=16, unet=2)
    wts = S.he_normal_weights(spec, 53, bias_std=0.1)
    frames = S.render_frames(n, h, w, "tiny", 54)
    ref, ref_maps = oracle.localize(frames, spec, wts, return_maps=True)
    assert map_rel_err(_maps(spec, wts, frames), ref_maps).max() <= TOL
    net = dl.Net(S.serialize_weights(spec, wts))
    out = torch.zeros((n * h * w, 8), dtype=torch.int32, device="cuda")
    counts = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    net.localize_device(torch.from_numpy(frames).cuda(), out, counts)
    torch.cuda.synchronize()
    rec = dl.emitters_from_device(out, int(counts[-1]))
    assert len(ref) > 10 and compare_emitters(rec, ref, ref_maps)["non_exempt_mismatch"] == 0
