"""Control-matrix product around its tiles: 1, 2 or 4 rows a wavefront, 4 wavefronts a block, 256-column steps
taken several at a time, chunks of 4096 columns, a ragged last chunk; many modes with few slopes (row blocks
past 65535).

Bar: FP32 products summed per lane over at most 16 four-term steps, over 64 lanes, then over the
chunks in order: (64 + 6 + n_chunks) roundings of 2^-24 of the sum of the terms' magnitudes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# the last two groups have blocks enough for 2 and for 4 rows a wavefront
@pytest.mark.parametrize("n_modes,n_slopes",
                         [(m, s) for m in (1, 7, 8, 9, 31, 33, 63)
                          for s in (1, 4, 255, 257, 511, 513, 767, 4095, 4101, 4096 * 17 + 130)]
                         + [(8185 + e, 2 * 4096 + s) for e in (0, 7, 8) for s in (-3, 1, 514)]
                         + [(32753 + e, s) for e in (0, 15, 16) for s in (1, 126, 4095)])
def test_tiles(torch_dev, n_modes, n_slopes):
    from paper_1408_0698_amd import shwfs
    rng = np.random.default_rng(n_modes * 131 + n_slopes)
    ld = (n_slopes + 3) // 4 * 4 + 4
    cm = np.full((n_modes, ld), np.nan, np.float32)          # what lies beside the matrix is not used
    cm[:, :n_slopes] = rng.normal(size=(n_modes, n_slopes))
    s = rng.normal(size=n_slopes).astype(np.float32)
    plan = shwfs.ReconPlan(n_modes, n_slopes)
    coefs = torch_dev.zeros(n_modes, device="cuda")
    delta = torch_dev.full((n_modes + 1,), 7.0, device="cuda")
    plan.step(torch_dev.from_numpy(cm).cuda(), torch_dev.from_numpy(s).cuda(), 0.5, coefs, delta[:n_modes])
    torch_dev.cuda.synchronize()
    a = cm[:, :n_slopes].astype(np.float64)
    want, mag = a @ s.astype(np.float64), np.abs(a) @ np.abs(s.astype(np.float64))
    got = delta.cpu().numpy()
    bar = (70 + n_slopes // 4096 + 1) * 2.0 ** -24 * mag
    assert np.all(np.abs(got[:n_modes] - want) <= bar) and got[n_modes] == 7.0
    assert np.array_equal(coefs.cpu().numpy(), np.float32(0.5) * got[:n_modes])


def test_more_row_blocks_than_a_second_grid_dimension_holds(torch_dev):
    from paper_1408_0698_amd import shwfs
    n = (1 << 22) - 5
    plan = shwfs.ReconPlan(n, 3)
    gen = torch_dev.Generator(device="cuda").manual_seed(1)
    cm = torch_dev.randint(-8, 9, (n, 4), generator=gen, device="cuda").float()
    s = torch_dev.tensor([1.0, 2.0, -3.0], device="cuda")
    coefs = torch_dev.zeros(n, device="cuda")
    plan.step(cm, s, 1.0, coefs)
    assert torch_dev.equal(coefs, cm[:, 0] + 2 * cm[:, 1] - 3 * cm[:, 2])    # whole numbers: exact
