"""DM surfaces and residuals at the edges of the kernels' tiles, against FP64 NumPy.

Surface bar: a value is a sum of at most (patch / pitch + 1)^2 products c e_x e_y, formed in two
passes of at most patch / pitch + 1 FMAs each with two FP32 exponentials (2 ulp each); each term
thus carries at most 2 (patch / pitch + 1) + 6 roundings of 2^-24 of the sum of the terms' magnitudes.
Residual: n_dm FP32 subtractions, each rounded once, in the order of the mirrors.
"""
import numpy as np
import pytest

from oracle import dm as OD

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# (pupil, pitch, patch): ragged tiles, a pitch that leaves one actuator per patch, more grid rows and
# columns per tile than one chunk holds (16 x 32), patches larger than the surface
@pytest.mark.parametrize("n,pitch,patch", [(64, 10, 64), (66, 7, 20), (130, 1, 34), (100, 2, 90), (34, 40, 64),
                                           (90, 13, 1024), (2, 1, 2)])
def test_surface_tiles(torch_dev, n, pitch, patch):
    from paper_1408_0698_amd import shwfs
    coupling = 0.3
    dm = shwfs.DmPlan(n, 0.05, 0.0, pitch, 0.0, coupling, patch)
    act = OD.actuators(n, 0.05, 0.0, pitch, 0.0)
    c = np.random.default_rng(n + pitch).normal(size=len(act)).astype(np.float32)
    out = torch_dev.full((dm.size, dm.size), float("nan"), device="cuda")
    dm.surface(torch_dev.from_numpy(c).cuda(), out)
    torch_dev.cuda.synchronize()
    got = out.cpu().numpy()
    want = OD.dm_surface(dm.size, act, c.astype(np.float64), pitch, coupling, patch)
    mag = OD.dm_surface(dm.size, act, np.abs(c).astype(np.float64), pitch, coupling, patch)
    bar = (2 * (patch / pitch + 1) + 6) * 2.0 ** -24 * mag + 1e-37
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - want) <= bar)


# pupil sides around multiples of 4 (four pixels per lane) and of the 256-quad tiles, unaligned window
# origins, odd pitches of screen and result, outputs past one launch's 80, repeated and distinct windows
@pytest.mark.parametrize("n,n_out,n_dm", [(1, 3, 1), (3, 2, 2), (4, 1, 0), (31, 81, 3), (32, 160, 4), (33, 7, 1),
                                          (130, 30, 3)])
def test_residual_tiles(torch_dev, n, n_out, n_dm):
    from paper_1408_0698_amd import shwfs
    rng = np.random.default_rng(n * 1000 + n_out)
    rows, cols = n + 9, n + 14
    scr = rng.normal(size=(rows, cols + 3)).astype(np.float32)
    surfs = [rng.normal(size=(n + 5 + d, n + 5 + d)).astype(np.float32) for d in range(n_dm)]
    scr_o = [(int(rng.integers(0, rows - n + 1)), int(rng.integers(0, cols - n + 1))) for _ in range(n_out)]
    kinds = [[(int(rng.integers(0, 6 + d)), int(rng.integers(0, 6 + d))) for d in range(n_dm)] for _ in range(3)]
    dm_o = [kinds[int(rng.integers(0, 3))] for _ in range(n_out)]
    big = torch_dev.full((n_out, n + 2, n + 5), float("nan"), device="cuda")
    out = big[:, :n, :n]
    d_scr = torch_dev.from_numpy(scr).cuda()
    shwfs.residual_opd(d_scr[:, :cols], [torch_dev.from_numpy(s).cuda() for s in surfs], n, scr_o, dm_o, out)
    torch_dev.cuda.synchronize()
    got = big.cpu().numpy()
    for k, ((r, c), od) in enumerate(zip(scr_o, dm_o)):
        want = scr[r:r + n, c:c + n]
        for s, (a, b) in zip(surfs, od):
            want = want - s[a:a + n, b:b + n]
        assert np.array_equal(got[k, :n, :n], want)
    assert np.isnan(got[:, n:]).all() and np.isnan(got[:, :, n:]).all()   # nothing outside the windows


def test_large_residual_equals_small(torch_dev):
    """Results above 64 MB are written past the caches: the same values as output by output."""
    from paper_1408_0698_amd import shwfs
    n, n_out = 601, 50
    gen = torch_dev.Generator(device="cuda").manual_seed(3)
    scr = torch_dev.randn((700, 701), generator=gen, device="cuda")
    sf = torch_dev.randn((640, 640), generator=gen, device="cuda")
    scr_o = [(k, 2 * k) for k in range(n_out)]
    dm_o = [[(k % 3, 5 * (k % 7))] for k in range(n_out)]
    out = torch_dev.empty((n_out, n, n), device="cuda")
    shwfs.residual_opd(scr, [sf], n, scr_o, dm_o, out)
    one = torch_dev.empty((1, n, n), device="cuda")
    for k in range(n_out):
        shwfs.residual_opd(scr, [sf], n, scr_o[k:k + 1], dm_o[k:k + 1], one)
        assert torch_dev.equal(one[0], out[k])
