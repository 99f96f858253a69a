"""A residual block's two BF16 layers in one kernel (kernels_block.hip) against
the two layers run one after the other: products, their order and roundings are
the same, so the maps are equal bit for bit.  tile_rows = 4 takes the two layers.
"""
import numpy as np
import pytest
import torch

import smlm_synth as S

pytestmark = pytest.mark.gpu


def _maps(spec, w, frames, **cfg):
    import paper_2410_02314_amd as dl
    net = dl.Net(S.serialize_weights(spec, w), precision="bf16", **cfg)
    n, h, wd = frames.shape
    maps = torch.full((n, net.head_outputs, h, wd), float("nan"), dtype=torch.float32, device="cuda")
    net.maps_device(torch.from_numpy(frames).cuda(), maps)
    torch.cuda.synchronize()
    return maps.cpu().numpy()


# one pixel, one row, tiles' edges (8 x 64 points of a dilation's lattice and the
# rim of one and two), several frames and tiles per workgroup, every layout
@pytest.mark.parametrize("C", [16, 32, 48])
@pytest.mark.parametrize("heads", [5, 10])
@pytest.mark.parametrize("n,h,w,dil", [(2, 1, 1, (1, 2)), (1, 1, 200, (1,)), (3, 9, 65, (1, 3)), (1, 8, 64, (1, 1)),
                                       (2, 33, 131, (2, 4)), (1, 150, 259, (16, 1)), (4, 300, 333, (1,))])
def test_equals_two_layers(C, heads, n, h, w, dil):
    spec = S.NetSpec("X", C, dil, head_outputs=heads)
    wts = S.he_normal_weights(spec, 31, bias_std=0.05)
    frames = S.render_frames(n, h, w, "tiny", 32)
    a, b = _maps(spec, wts, frames), _maps(spec, wts, frames, tile_rows=4)
    assert not np.isnan(a).any() and np.array_equal(a, b)
