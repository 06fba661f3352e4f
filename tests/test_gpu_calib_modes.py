"""The interaction matrix computed only where the modes reach, against the whole-frame path.

Both form the same slopes from the same wavefronts with the same kernel code; an OPD sample may
round differently by the FP32 contraction of dx^2 + dy^2 (1 ulp of the exponent, below 2^-20 of the
amplitude for a 64-pixel patch), which moves a slope by less than 1e-6 detector pixels.
"""
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


def _whole(torch, plan, dm, acts, amp, r0, c0):
    """The matrix from whole frames (influence frames, measurement, push-pull)."""
    from paper_1408_0698_amd import shwfs
    n, N = len(acts), plan.cfg.pupil_n
    n_slopes = plan.n_wfs * 2 * plan.n_valid
    im = torch.empty((n_slopes, n), device="cuda")
    act = torch.from_numpy(np.repeat(np.asarray(acts, np.int32), 2)).cuda()
    a = torch.from_numpy(np.tile(np.array([amp, -amp], np.float32), n)).cuda()
    opd = torch.empty((2 * n, N, N), device="cuda")
    dm.influence_opd(act, a, r0, c0, N, opd)
    sl = torch.empty((2 * n, plan.n_wfs, 2, plan.n_valid), device="cuda")
    plan.measure(opd.unsqueeze(1).expand(-1, plan.n_wfs, -1, -1), sl)
    shwfs.push_pull(sl.view(2 * n, n_slopes), n, 1.0 / (2.0 * amp), im)
    return im


# (n_subap, n_wfs, altitude, pitch, patch): patches that start on and off sub-aperture edges, end
# inside one, are smaller than one, mirrors larger than the pupil, actuators off the pupil; one more
# block than a whole number of pairs
@pytest.mark.parametrize("n_subap,n_wfs,alt,pitch,patch", [(13, 2, 0.0, 10, 64), (13, 1, 0.0, 7, 20), (16, 3, 3000.0, 9, 6),
                                                           (21, 1, 0.0, 5, 2), (20, 1, 0.0, 33, 100)])
def test_modes_equal_whole_frames(torch_dev, n_subap, n_wfs, alt, pitch, patch):
    from paper_1408_0698_amd import calib, shwfs
    cfg = G.CFG1.replace(pupil_n=10 * n_subap, n_subap=n_subap, flags=0)
    plan = shwfs.WfsPlan(cfg, n_wfs, G.launch_positions(cfg, n_wfs))
    dm = shwfs.DmPlan(cfg.pupil_n, cfg.pupil_dx_m, alt, pitch, 30.0, 0.3, patch)
    r0, c0 = (dm.size - cfg.pupil_n) // 2, (dm.size - cfg.pupil_n) // 3
    rng = np.random.default_rng(n_subap + pitch)
    acts = rng.choice(dm.n_act, min(dm.n_act, 37), replace=False).astype(np.int32)
    acts[:2] = [0, dm.n_act - 1]
    acts[-1] = dm.n_act          # off the grid: its column is 0
    amp = 50e-9
    direct = torch_dev.full((plan.n_wfs * 2 * plan.n_valid, len(acts) + 3), float("nan"), device="cuda")
    assert shwfs.interaction_matrix(plan, dm, acts, amp, r0, c0, 1.0 / (2.0 * amp), direct[:, :len(acts)])
    whole = _whole(torch_dev, plan, dm, acts, amp, r0, c0)
    torch_dev.cuda.synchronize()
    got, want = direct.cpu().numpy(), whole.cpu().numpy()
    assert np.isnan(got[:, len(acts):]).all()
    got = got[:, :len(acts)]
    assert np.abs(got - want).max() * 2 * amp <= 2e-6
    assert np.array_equal(got == 0, want == 0)          # the same sub-apertures are touched
    assert np.all(got[:, -1] == 0)
    assert torch_dev.equal(calib.interaction_matrix(plan, dm, acts, amp, r0, c0), direct[:, :len(acts)])


def test_many_modes_in_several_launches(torch_dev):
    from paper_1408_0698_amd import calib, shwfs
    cfg = G.CFG1.replace(pupil_n=130, n_subap=13, flags=0)
    plan = shwfs.WfsPlan(cfg, 1, G.launch_positions(cfg, 1))
    dm = shwfs.DmPlan(130, cfg.pupil_dx_m, 0.0, 4, 0.0, 0.3, 20)
    acts = np.arange(dm.n_act, dtype=np.int32)
    assert len(acts) > 800
    im = calib.interaction_matrix(plan, dm, acts, 50e-9, 0, 0)
    for k in (0, 799, 800, len(acts) - 1):
        assert torch_dev.equal(im[:, k], calib.interaction_matrix(plan, dm, acts[k:k + 1], 50e-9, 0, 0)[:, 0])


def test_other_plans_take_whole_frames(torch_dev):
    """Noise, another launch variant, another shape and a patch across the pupil: refused by the direct
    kernel, and calibrated through whole frames as before; a window off the surface raises as before."""
    from paper_1408_0698_amd import calib, shwfs
    base = G.CFG1.replace(pupil_n=130, n_subap=13, flags=0)
    dm = shwfs.DmPlan(130, base.pupil_dx_m, 0.0, 10, 0.0, 0.3, 64)
    acts = np.array([40, 60], np.int32)
    for cfg, variant, mirror in ((base.replace(flags=1), None, dm), (base, 12, dm), (G.CFG1_R2.replace(pupil_n=130, n_subap=13, flags=0), None, dm),
                                 (base, None, shwfs.DmPlan(130, base.pupil_dx_m, 0.0, 10, 0.0, 0.3, 128))):
        plan = shwfs.WfsPlan(cfg, 1, G.launch_positions(cfg, 1))
        if variant is not None:
            plan.set_variant(variant)
        im = torch_dev.empty((2 * plan.n_valid, 2), device="cuda")
        assert not shwfs.interaction_matrix(plan, mirror, acts, 50e-9, 0, 0, 1e7, im)
        assert torch_dev.equal(calib.interaction_matrix(plan, mirror, acts, 50e-9, 0, 0), _whole(torch_dev, plan, mirror, acts, 50e-9, 0, 0))
    plan = shwfs.WfsPlan(base, 1, G.launch_positions(base, 1))
    with pytest.raises(shwfs.ShwError):
        calib.interaction_matrix(plan, dm, acts, 50e-9, 1, 0)
