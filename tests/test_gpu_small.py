"""Small batches: detection in bands of 2 rows, FP32 tiles of 4 rows.  Both only
split the work differently, so a frame gives the same bits alone (the small
split) and in a batch that takes the other one.
"""
import numpy as np
import pytest
import torch

import smlm_synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(1, 1), (2, 64), (3, 65), (8, 256), (9, 257), (33, 1030)])
def test_detection_bands(h, w):
    import paper_2410_02314_amd as dl
    spec, wts = S.make_net("A", 1)
    net = dl.Net(S.serialize_weights(spec, wts))
    n = 129 // ((h + 7) // 8) + 1            # more than 128 bands of 8 rows
    rng = np.random.default_rng(41)
    x = rng.integers(-3, 4, (n, h, w)).astype(np.float32)        # many plateaus
    x[rng.random(x.shape) < 0.05] = -np.inf
    t = torch.from_numpy(x).cuda()

    def detect(v):
        d = torch.full(v.shape, 7, dtype=torch.uint8, device="cuda")
        net.debug_detect(v, -1.5, d)
        torch.cuda.synchronize()
        return d.cpu().numpy()

    both = detect(t)
    for f in range(0, n, max(1, n // 6)):
        assert np.array_equal(detect(t[f:f + 1].contiguous())[0], both[f])


@pytest.mark.parametrize("C", [16, 32])
@pytest.mark.parametrize("n,h,w,dil", [(1, 1, 1, (1,)), (2, 5, 33, (1, 2)), (1, 60, 131, (4, 1)), (5, 90, 70, (1, 3)),
                                       (1, 140, 190, (1, 16))])
def test_tile_rows(C, n, h, w, dil):
    import paper_2410_02314_amd as dl
    spec = S.NetSpec("X", C, dil)
    blob = S.serialize_weights(spec, S.he_normal_weights(spec, 42, bias_std=0.05))
    fr = torch.from_numpy(S.render_frames(n, h, w, "tiny", 43)).cuda()
    out = []
    for rows in (0, 8):
        net = dl.Net(blob, precision="fp32", tile_rows=rows)
        maps = torch.full((n, net.head_outputs, h, w), float("nan"), dtype=torch.float32, device="cuda")
        net.maps_device(fr, maps)
        torch.cuda.synchronize()
        out.append(maps.cpu().numpy())
    assert not np.isnan(out[0]).any() and np.array_equal(out[0], out[1])
