"""Gated FP32 runs and what earlier calls left in the handle's workspace: a
layer's active tiles also read points no layer computed in this run.  Such
points must not reach the kept tiles, neither as values nor through the power
of two that a tile's inputs share.

Tolerance against the ungated run: the products of a kept pixel are the same, a
tile's power of two may differ, which changes an operand by 2^-36 of the tile's
largest input at most and so a sum's last bit now and then; 1e-6 of |o| + rms is
twelve such bits.
"""
import numpy as np
import pytest
import torch

import smlm_synth as S

pytestmark = pytest.mark.gpu

H, W = 512, 768
KEEP = np.array([[1, 0, 0], [0, 0, 0]], bool)          # the only bright tile of the frame


def _frames():
    f = S.render_frames(2, H, W, "sparse", 4047)
    f = np.minimum(f, 400)
    f[:, 100:110, 60:70] = 3000
    return f


def _maps(net, frames):
    fr = torch.from_numpy(frames).cuda()
    m = torch.zeros((len(frames), net.head_outputs, H, W), dtype=torch.float32, device="cuda")
    net.maps_device(fr, m)
    torch.cuda.synchronize()
    return m.cpu().numpy()


@pytest.mark.parametrize("name,seed", [("A", 1), ("B", 2)])
@pytest.mark.parametrize("rows", [0, 4])
@pytest.mark.parametrize("before", ["scaled", "fp8", "bf16"])
def test_kept_tiles_do_not_depend_on_earlier_calls(name, seed, rows, before):
    _check(*S.make_net(name, seed), rows, before)


@pytest.mark.parametrize("C,dil", [(16, (64, 40)), (48, (3, 64))])
def test_radius_of_more_than_half_a_gate_tile(C, dil):
    spec = S.NetSpec("X", C, dil)
    _check(spec, S.he_normal_weights(spec, 4048, bias_std=0.1), 0, "scaled")


def _check(spec, w, rows, before):
    import paper_2410_02314_amd as dl
    from tests.parity import map_rel_err
    from tests.test_gpu_gated import brightness_gate
    blob = S.serialize_weights(spec, w)
    frames = _frames()
    theta = brightness_gate(6.0).astype(np.float32)
    cfg = dict(precision="fp32", flags=dl.DL_FLAG_GATE, tile_rows=rows)
    kept = np.repeat(np.repeat(KEEP, 256, 0), 256, 1)

    def gated(net):
        net.set_config(**cfg)
        net.set_gate(theta, 0.05)
        m = _maps(net, frames)
        k = torch.zeros(2 * 6, dtype=torch.uint8, device="cuda")
        net.gate_keep_map(k)
        torch.cuda.synchronize()
        assert np.array_equal(k.cpu().numpy().reshape(2, 2, 3).astype(bool), np.stack([KEEP, KEEP]))
        return m[:, :, kept]

    fresh = gated(dl.Net(blob, **cfg))
    net = dl.Net(blob, **cfg)
    gated(net)                                             # (the workspace has its size)
    if before == "scaled":
        net.set_config(precision="fp32", tile_rows=rows, in_scale_override=0.01 * 2.0 ** 45)
    else:
        net.set_config(precision=before)
    net.set_gate(None)
    _maps(net, frames)
    after = gated(net)
    assert np.array_equal(after, fresh)
    full = _maps(dl.Net(blob, precision="fp32", tile_rows=rows), frames)[:, :, kept]
    assert map_rel_err(after[..., None], full[..., None]).max() <= 1e-6
