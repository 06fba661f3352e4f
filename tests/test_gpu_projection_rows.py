"""Layer projection where rounding moves the screen row by two.

With one screen sample per pupil pixel and an origin one rounding step below a half-integer, the FP64
screen coordinate rounds down before a power of two and up after it, so that two neighbouring pupil rows lie
two screen rows apart.  Bars as for the projection's tiles: 2^-24 of the value plus 1e-12 samples of
coordinate rounding times the slope between samples (below 20 for unit-variance screens).
"""
import math

import numpy as np
import pytest

from oracle import openloop as OO

pytestmark = pytest.mark.gpu

DX = 4.875e-2


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _advanced(y0, step, times):
    for _ in range(times):
        y0 += step
    return y0


# pupil side, row origin; a drifting screen's origin (five steps of 0.2) and the nearest value below a
# half-integer; the two rows may share a wavefront (rows 4 k .. 4 k + 3) or not
@pytest.mark.parametrize("n,y0", [(800, _advanced(401.5, 0.2, 5)), (800, _advanced(500.5, 0.2, 5)), (400, _advanced(500.5, 0.2, 5)),
                                  (80, _advanced(500.5, 0.2, 5)), (80, math.nextafter(63.5, 0.0)), (800, math.nextafter(1023.5, 0.0))])
@pytest.mark.parametrize("axes", ["row", "both"])
def test_projection_row_steps(torch_dev, n, y0, axes):
    from paper_1408_0698_amd import shwfs
    rows = np.floor(y0 + (np.arange(n) + 0.5 - 0.5 * n))
    assert np.diff(rows).max() == 2     # the case is there
    rng = np.random.default_rng(n)
    x0 = y0 if axes == "both" else y0 + 0.3
    scr = rng.normal(size=(int(y0 + n / 2) + 3, int(x0 + n / 2) + 4)).astype(np.float32)
    out = torch_dev.empty((2, n, n), device="cuda")
    targets = [(0.0, 0.0, 0.0), (1e-6, 2e-6, 90e3)]
    shwfs.project_layers([(torch_dev.from_numpy(scr).cuda(), DX, 0.0, x0, y0)], n, DX, targets, out)
    got = out.cpu().numpy()
    for t, (tx, ty, h) in enumerate(targets):
        want = OO.project([(scr, DX, 0.0, x0, y0)], n, DX, (tx, ty), h, None)
        assert np.all(np.abs(got[t] - want) <= 2.0 ** -24 * np.abs(want) + 1e-12 * 20.0 + 1e-12)
