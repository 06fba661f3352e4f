"""Calibrations whose pairs of one group of modes have more lanes than a launch may (2^32)."""
import numpy as np
import pytest

from gen import configs as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_many_sensors(torch_dev):
    from paper_1408_0698_amd import calib, shwfs
    cfg = G.CFG1.replace(pupil_n=130, n_subap=13, flags=0)
    n_wfs, n_modes, cells = 4096, 256, 8 * 8      # a 64-pixel patch reaches 8 x 8 sub-apertures of 10 pixels at most
    assert n_modes * n_wfs * cells * 80 > 2 ** 32
    torch_dev.cuda.empty_cache()
    if torch_dev.cuda.mem_get_info()[0] < 16 << 30:
        pytest.skip("not enough free GPU memory")
    dm = shwfs.DmPlan(130, cfg.pupil_dx_m, 0.0, 6, 0.0, 0.3, 64)
    acts = np.arange(n_modes, dtype=np.int32)
    assert dm.n_act >= n_modes
    # sensors alike but for the first and the last
    launch = G.launch_positions(cfg, 2)
    plan = shwfs.WfsPlan(cfg, n_wfs, [launch[0]] * (n_wfs - 1) + [launch[1]])
    im = calib.interaction_matrix(plan, dm, acts, 50e-9, 0, 0).view(n_wfs, -1, n_modes)
    two = calib.interaction_matrix(shwfs.WfsPlan(cfg, 2, launch), dm, acts, 50e-9, 0, 0).view(2, -1, n_modes)
    assert (two != 0).any(dim=1).all()
    assert torch_dev.equal(im[-1], two[1])
    assert torch_dev.equal(im[:-1], two[:1].expand(n_wfs - 1, -1, -1))


def test_large_matrix(torch_dev):
    """A matrix of more groups of four elements than lanes: zeros to its last row and column."""
    from paper_1408_0698_amd import calib, shwfs
    cfg = G.CFG1.replace(pupil_n=130, n_subap=13, flags=0)
    n_wfs = 4096
    launch = G.launch_positions(cfg, 1)
    plan = shwfs.WfsPlan(cfg, n_wfs, launch * n_wfs)
    rows = 2 * plan.n_valid * n_wfs
    n_modes = 4 * (2 ** 32 // rows + 1)
    assert rows * (n_modes // 4) > 2 ** 32
    torch_dev.cuda.empty_cache()
    if torch_dev.cuda.mem_get_info()[0] < 4 * rows * n_modes + (16 << 30):
        pytest.skip("not enough free GPU memory")
    dm = shwfs.DmPlan(130, cfg.pupil_dx_m, 0.0, 10, 0.0, 0.3, 2)
    every = calib.interaction_matrix(shwfs.WfsPlan(cfg, 1, launch), dm, np.arange(dm.n_act, dtype=np.int32), 50e-9, 0, 0)
    seen = int((every != 0).any(dim=0).nonzero()[0])   # an actuator that a valid sub-aperture sees
    acts = np.full(n_modes, -1, np.int32)              # off the mirror: columns of zeros
    acts[0] = acts[-1] = seen
    stale = torch_dev.full((rows, n_modes), 7.0, device="cuda")   # what the matrix's memory may hold
    del stale
    im = calib.interaction_matrix(plan, dm, acts, 50e-9, 0, 0)
    for k in (0, -1):
        assert torch_dev.equal(im[:, k].reshape(n_wfs, -1), every[:, seen].expand(n_wfs, -1))
    for r in range(0, rows, 65536):
        assert int(torch_dev.count_nonzero(im[r:r + 65536, 1:-1])) == 0
    del im
    torch_dev.cuda.empty_cache()
