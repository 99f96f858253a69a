"""Load offsets of the FP32 pair kernels (halo_start and halo_point of
csrc/conv_common.h, 32 bits) against 64-bit arithmetic, on the host: every
sampled tile's points that lie in the frame, for frames up to the 2 GiB of
activations that the library accepts, however flat, in plain rows and in phase
layouts."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

DRIVER = r"""
#include "conv_common.h"
#include <cstdio>
#include <cstdlib>
#include <set>
using namespace dloc;

static std::set<int> some(int n) { return {0, n > 1 ? 1 : 0, n / 2, n > 1 ? n - 2 : 0, n - 1}; }

int main(int argc, char **argv)
{
    const int C = std::atoi(argv[1]), d = std::atoi(argv[2]), h = std::atoi(argv[3]), w = std::atoi(argv[4]);
    const bool phase = std::atoi(argv[5]);
    const int64_t layout = phase ? d : 1;
    if (act_points(h, w, (int)layout) * C * 4 >= (int64_t)1 << 31) return 3;      // (not accepted)
    const int TC = 32, hd = (h + d - 1) / d, wd = (w + d - 1) / d;
    const uint32_t stride = 64;
    long points = 0;
    for (int TR : {4, 8})
        for (int ry : some((h + TR * d - 1) / (TR * d)))
            for (int rx : some((w + TC * d - 1) / (TC * d)))
                for (int py : some(d))
                    for (int px : some(d)) {
                        const int y0 = ry * TR * d + py, x0 = rx * TC * d + px;
                        if (y0 >= h || x0 >= w) continue;
                        const int a0 = phase ? ((py * d + px) * hd + ry * TR) * wd + rx * TC : y0 * w + x0;
                        const int rs = phase ? wd : d * w, cs = phase ? 1 : d;
                        for (int ii = 0; ii < TR + 2; ++ii)
                            for (int jj = 0; jj < TC + 2; ++jj) {
                                const int y = y0 + d * (ii - 1), x = x0 + d * (jj - 1);
                                if (y < 0 || y >= h || x < 0 || x >= w) continue;
                                const int64_t pt = phase ? ((int64_t)((y % d) * d + x % d) * hd + y / d) * wd + x / d
                                                         : (int64_t)y * w + x;
                                const uint32_t got = halo_start(a0, rs, cs, stride) + halo_point(ii, jj, rs, cs, stride);
                                if (got != (uint64_t)pt * stride || got >= 0x7FFFFFFFu - 64) {
                                    std::printf("tile (%d, %d), point (%d, %d): %u, want %lld\n", y0, x0, ii, jj, got,
                                                (long long)(pt * stride));
                                    return 1;
                                }
                                ++points;
                            }
                    }
    std::printf("ok %ld points\n", points);
    return points > 0 ? 0 : 2;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("offsets")
    (d / "driver.hip").write_text(DRIVER)
    csrc = os.path.join(ROOT, "paper_2410_02314_amd", "csrc")
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17", "-O1",
                           "-I", os.path.join(ROOT, "include"), "-I", csrc, str(d / "driver.hip"), "-o", str(d / "driver")],
                          stderr=subprocess.DEVNULL)
    return str(d / "driver")


@pytest.mark.parametrize("C,d,h,w", [(16, 64, 513, 58300), (16, 16, 129, 235000), (16, 64, 1, 1 << 20), (48, 64, 1, 1 << 20),
                                     (32, 64, 15, 1 << 20), (48, 1, 3344, 3344), (48, 3, 10, 1 << 20), (32, 5, 4095, 4095),
                                     (16, 1, 31, 1 << 20), (32, 2, 77, 131), (16, 64, 1, 1), (48, 63, 1 << 20, 10)])
def test_offsets_of_a_frames_points(driver, C, d, h, w):
    ran = 0
    for phase in (0, 1):
        if phase and (d == 1 or d & (d - 1)):
            continue
        r = subprocess.run([driver, str(C), str(d), str(h), str(w), str(phase)], capture_output=True, text=True, timeout=60)
        assert r.returncode in (0, 3), r.stdout
        ran += r.returncode == 0
    assert ran


@pytest.mark.gpu
@pytest.mark.parametrize("C", [16, 48])
def test_flattest_frame_against_the_oracle(C):
    """1 x 2^20 pixels at dilation 64: the rows above and below a tile lie 2^26
    points away."""
    import numpy as np
    import torch

    import oracle
    import paper_2410_02314_amd as dl
    import smlm_synth as S
    from tests.parity import map_rel_err
    spec = S.NetSpec("X", C, (64,))
    w = S.he_normal_weights(spec, 71, bias_std=0.05)
    frames = np.random.default_rng(72).integers(90, 700, (1, 1, 1 << 20)).astype(np.uint16)
    net = dl.Net(S.serialize_weights(spec, w), precision="fp32")
    m = torch.full((1, 5, 1, 1 << 20), float("nan"), dtype=torch.float32, device="cuda")
    net.maps_device(torch.from_numpy(frames).cuda(), m)
    torch.cuda.synchronize()
    assert map_rel_err(m.cpu().numpy(), oracle.net_maps_batch(frames, spec, w)).max() <= 1e-4
