"""The direct calibration kernel gives the same bits as whole frames: influence functions, measurement of every
sub-aperture and push-pull difference.  Both form the samples by one expression and run the same transforms."""
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


# patches off and on sub-aperture edges, smaller than a sub-aperture, reaching most of the pupil; several sensors
@pytest.mark.parametrize("n_subap,n_wfs,pitch,patch", [(13, 2, 10, 64), (16, 3, 9, 6), (20, 1, 33, 100), (40, 1, 10, 64)])
def test_direct_equals_whole_frames(torch_dev, n_subap, n_wfs, pitch, patch):
    from paper_1408_0698_amd import calib, shwfs
    cfg = G.CFG1.replace(pupil_n=10 * n_subap, n_subap=n_subap, flags=0)
    plan = shwfs.WfsPlan(cfg, n_wfs, G.launch_positions(cfg, n_wfs))
    dm = shwfs.DmPlan(cfg.pupil_n, cfg.pupil_dx_m, 0.0, pitch, 0.0, 0.3, patch)
    n, N, amp = min(dm.n_act, 150), cfg.pupil_n, 50e-9
    acts = np.arange(dm.n_act - n, dm.n_act, dtype=np.int32)
    n_slopes = n_wfs * 2 * plan.n_valid
    opd = torch_dev.empty((2 * n, N, N), device="cuda")
    dm.influence_opd(torch_dev.from_numpy(np.repeat(acts, 2)).cuda(),
                     torch_dev.from_numpy(np.tile(np.array([amp, -amp], np.float32), n)).cuda(), 0, 0, N, opd)
    sl = torch_dev.empty((2 * n, n_wfs, 2, plan.n_valid), device="cuda")
    plan.measure(opd.unsqueeze(1).expand(-1, n_wfs, -1, -1), sl)
    want = torch_dev.empty((n_slopes, n), device="cuda")
    shwfs.push_pull(sl.view(2 * n, n_slopes), n, 1.0 / (2.0 * amp), want)
    got = torch_dev.full((n_slopes, n), float("nan"), device="cuda")
    assert shwfs.interaction_matrix(plan, dm, acts, amp, 0, 0, 1.0 / (2.0 * amp), got)
    assert (want != 0).any()
    assert torch_dev.equal(got, want)
    assert torch_dev.equal(calib.interaction_matrix(plan, dm, acts, amp, 0, 0), want)
