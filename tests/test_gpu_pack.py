"""Weights as FP16 pairs, packed on the device (k_pack_pairs): every conv shape
the networks have -- channel groups of 16 and 32, 1x1 transitions over part of
their inputs, more convs than one launch takes -- against the FP64 oracle, at the
FP32 form's 1e-4 of |o| + rms; a net whose channels are balanced when packed, and
back, gives the maps it gave before.
"""
import numpy as np
import pytest
import torch

import oracle
import smlm_synth as S
from tests.parity import map_rel_err

pytestmark = pytest.mark.gpu


def _maps(net, frames):
    m = torch.full((len(frames), net.head_outputs, *frames.shape[1:]), float("nan"), dtype=torch.float32, device="cuda")
    net.maps_device(torch.from_numpy(frames).cuda(), m)
    torch.cuda.synchronize()
    return m.cpu().numpy()


@pytest.mark.parametrize("spec", [S.NetSpec("X", 16, (1, 3)), S.NetSpec("X", 32, (2,), head_outputs=10), S.NetSpec("X", 48, (1, 2) * 4),
                                  S.DenseSpec("X", 16, (1, 2), 1, 32), S.DenseSpec("X", 32, (1, 2) * 4, 4, 16),
                                  S.DenseSpec("X", 32, (1, 2, 1, 2, 1, 2, 1), 4, 16, unet=2), S.DenseSpec("X", 16, (2,), 3, 32, unet=2)])
def test_maps_against_the_oracle(spec):
    import paper_2410_02314_amd as dl
    w = S.he_normal_weights(spec, 81, bias_std=0.05)
    frames = S.render_frames(2, 23, 45, "tiny", 82)
    net = dl.Net(S.serialize_weights(spec, w), precision="fp32")
    assert map_rel_err(_maps(net, frames), oracle.net_maps_batch(frames, spec, w)).max() <= 1e-4


@pytest.mark.parametrize("exp,row", [(40, None), (16, 0), (16, 7)])
def test_a_channel_read_faintly(exp, row):
    """Hidden channel 3 is 2^exp above the others and read with weights as far
    below, in every row (balanced when packed) or in all but one, whichever it is
    (packed as it is: within the 2^28 that a tile's pairs span)."""
    import paper_2410_02314_amd as dl
    spec = S.NetSpec("X", 32, (1,))
    w = S.he_normal_weights(spec, 83, bias_std=0.05)
    s = np.float32(2.0 ** exp)
    w["blk0.w1"][3] *= s
    w["blk0.b1"][3] *= s
    ordinary = w["blk0.w2"][row, 3].copy() if row is not None else None
    w["blk0.w2"][:, 3] /= s
    if row is not None:
        w["blk0.w2"][row, 3] = ordinary
        w["head.w"][:, row] /= s
    frames = S.render_frames(1, 23, 45, "tiny", 84)
    assert map_rel_err(_maps(dl.Net(S.serialize_weights(spec, w), precision="fp32"), frames),
                       oracle.net_maps_batch(frames, spec, w)).max() <= 1e-4
