"""Layer projection at the edges of the kernel's tiles and over its two ways of reading a layer.

Bars: positions, weights and sums are FP64 and the result is rounded once to FP32, so a value is
within 2^-24 of its magnitude plus the FP64 rounding of the screen coordinates (2^-52 of a
coordinate below 4096 samples, so 1e-12 samples) times the slope between neighbouring samples.
"""
import numpy as np
import pytest

from oracle import openloop as OO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# pupil sides around the 64-column tiles (in pairs) and the 128 rows of a block row of 8 XCDs; layers
# coarser and finer than the pupil (at most one sample per pixel: rows shared; finer: rows read apart)
@pytest.mark.parametrize("n,spacings", [(1, (0.05,)), (3, (0.05, 0.02)), (63, (0.05, 0.1)), (64, (0.02,)),
                                        (65, (0.0499, 0.0501)), (129, (0.05, 0.013, 0.2)), (200, (0.05,) * 16)])
def test_projection_tiles(torch_dev, n, spacings):
    from paper_1408_0698_amd import shwfs
    dx, rng = 0.05, np.random.default_rng(n)
    layers, host = [], []
    for k, sp in enumerate(spacings):
        alt = 0.0 if k == 0 else 900.0 * k
        cols = int(n * dx / sp) + 24
        scr = rng.normal(size=(cols + 3, cols + 5)).astype(np.float32)
        c = (cols - 1) / 2.0
        layers.append((torch_dev.from_numpy(scr).cuda()[:, :cols + 2], sp, alt, c + 0.3, c + 1.7))
        host.append((scr[:, :cols + 2], sp, alt, c + 0.3, c + 1.7))
    targets = [(0.0, 0.0, 0.0), (2e-6, -1e-6, 90e3), (-1e-6, 3e-6, 88e3)] * 4
    tilt = rng.normal(size=(len(targets), 2)) * 1e-6
    out = torch_dev.full((len(targets), n, n + 3), float("nan"), device="cuda")
    shwfs.project_layers(layers, n, dx, targets, out[:, :, :n], tilt=torch_dev.from_numpy(tilt).cuda())
    torch_dev.cuda.synchronize()
    got = out.cpu().numpy()
    for t, (tx, ty, h) in enumerate(targets):
        want = OO.project(host, n, dx, (tx, ty), h, tilt[t])
        bar = 2.0 ** -24 * np.abs(want) + 1e-12 * 20.0 * len(spacings) + 1e-12
        assert np.all(np.abs(got[t, :, :n] - want) <= bar)
    assert np.isnan(got[:, :, n:]).all()


def test_projection_keeps_infinite_samples(torch_dev):
    """An infinite sample gives infinity where its weight is not 0 and NaN where it is (0 x infinity)."""
    from paper_1408_0698_amd import shwfs
    scr = torch_dev.zeros((40, 40), device="cuda")
    scr[20, 20] = float("inf")
    out = torch_dev.empty((1, 8, 8), device="cuda")
    shwfs.project_layers([(scr, 0.05, 0.0, 19.75, 19.75)], 8, 0.05, [(0.0, 0.0, 0.0)], out)
    got = out[0].cpu().numpy()     # pixel centres at 19.75 + (j - 3.5): 16.25, 17.25, ...
    want = np.zeros((8, 8), np.float32)
    want[3:5, 3:5] = np.inf        # 19.25 and 20.25 on both axes
    assert np.array_equal(got, want)


@pytest.mark.parametrize("n_s", [2, 3, 31, 64, 65, 130, 256])
def test_uplink_sample_groups(torch_dev, n_s):
    """Sample counts around one group of 4 x 1024 samples per block."""
    from paper_1408_0698_amd import shwfs
    rng = np.random.default_rng(n_s)
    scr = rng.normal(size=(80, 90)).astype(np.float32)
    layers = [(torch_dev.from_numpy(scr).cuda(), 0.05, h, 44.0, 39.0) for h in (0.0, 5000.0)]
    lgs = [(0.3, -0.2, 1e-6, 2e-6, 90e3), (0.0, 0.0, 0.0, 0.0, 80e3)]
    out = torch_dev.empty((2, 2), device="cuda", dtype=torch_dev.float64)
    shwfs.uplink_tilt(layers, lgs, 1.1, n_s, out)
    got = out.cpu().numpy()
    for k, (lx, ly, tx, ty, h) in enumerate(lgs):
        want = OO.uplink_tilt([(scr, 0.05, a, 44.0, 39.0) for a in (0.0, 5000.0)], (lx, ly), (tx, ty), h, 1.1, n_s)
        # FP64 sums of at most 65536 terms of magnitude |OPD| < 10 over a lever of about d / 4
        assert np.abs(got[k] - np.array(want)).max() <= 1e-9
