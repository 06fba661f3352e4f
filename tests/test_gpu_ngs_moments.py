"""Noise-free 8-pixel NGS sub-apertures: slopes from the field's line moments, with and without images.

Bars: those of the sensor (images 1e-4 of the sub-aperture's maximum, slopes 1e-3 px) are far above
the FP32 error: a line moment has 28 products of unit phasors with weights below 1, so a slope is
within about 16 lines x 60 roundings x 2^-24 x 4 px / sqrt(16) < 1e-4 px; 1e-4 is asserted.
"""
import numpy as np
import pytest

from gen import configs as G
from gen import screens as S
from oracle import wfs as OW

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _run(torch, plan, opd, images, **kw):
    f = opd.shape[0]
    sl = torch.full((f, plan.n_wfs, 2, plan.n_valid), float("nan"), device="cuda")
    im = torch.full((f, plan.n_wfs, plan.n_valid, plan.cfg.det_n, plan.cfg.det_n), float("nan"), device="cuda") if images else None
    fl = torch.full((f, plan.n_wfs, plan.n_valid), 7, dtype=torch.uint8, device="cuda")
    plan.measure(opd, sl, im, fl, **kw)
    torch.cuda.synchronize()
    return sl, im, fl


# sub-aperture counts around the 8 of a wavefront and the 32 of a block, both detectors, photometry
@pytest.mark.parametrize("n_subap,n_wfs,frames,det,photons", [(1, 1, 1, 8, 0.0), (2, 1, 2, 8, 0.0), (3, 1, 1, 16, 0.0),
                                                              (3, 3, 3, 8, 250.0), (5, 2, 3, 16, 100.0), (10, 1, 3, 8, 0.0)])
def test_slopes_and_images(torch_dev, n_subap, n_wfs, frames, det, photons):
    from paper_1408_0698_amd import shwfs
    cfg = G.CFG0.replace(pupil_n=8 * n_subap, n_subap=n_subap, det_n=det, photons_per_subap=photons, obstruction=0.0 if n_subap < 4 else 0.14)
    plan = shwfs.WfsPlan(cfg, n_wfs)
    n = cfg.pupil_n
    opd = S.random_opd((frames, n_wfs, n, n), 120e-9, n_subap * 10 + det)
    # rows at 4-byte alignment inside a wider buffer
    buf = torch_dev.zeros((frames, n_wfs, n, n + 3), device="cuda")
    d = buf[..., 1:n + 1]
    d.copy_(torch_dev.from_numpy(opd))
    sl, im, fl = _run(torch_dev, plan, d, True)
    bare, _, fl2 = _run(torch_dev, plan, d, False)
    assert torch_dev.equal(sl, bare) and torch_dev.equal(fl, fl2) and not fl.any()
    want = OW.Sensor(cfg, n_wfs).measure(opd)
    assert np.abs(sl.cpu().numpy() - want["slopes"]).max() <= 1e-4
    scale = np.abs(want["images"]).max(axis=(-1, -2), keepdims=True)
    assert (np.abs(im.cpu().numpy() - want["images"]) / scale).max() <= 1e-5


def test_work_list_mixes_items_with_and_without_images(torch_dev):
    from paper_1408_0698_amd import shwfs
    plan = shwfs.WfsPlan(G.CFG0)
    opd = torch_dev.from_numpy(S.ngs8m_opd(5)[:, None]).cuda()
    ref, im, _ = _run(torch_dev, plan, opd, True)
    sl = torch_dev.full_like(ref, float("nan"))
    got = torch_dev.full_like(im, float("nan"))
    shwfs.measure_batch([(plan, opd[k], sl[k], got[k] if k % 2 else None, k, k) for k in range(5)])
    torch_dev.cuda.synchronize()
    assert torch_dev.equal(sl, ref)
    for k in range(5):
        assert torch_dev.equal(got[k], im[k]) if k % 2 else torch_dev.isnan(got[k]).all()


def test_a_bad_sample_empties_its_sub_aperture_only(torch_dev):
    """An OPD that is not a number leaves nothing above the threshold: slopes 0 and flag 1, as with an image."""
    from paper_1408_0698_amd import shwfs
    plan = shwfs.WfsPlan(G.CFG0)
    opd = torch_dev.from_numpy(S.ngs8m_opd(1)[:, None]).cuda()
    ref, _, _ = _run(torch_dev, plan, opd, False)
    opd[0, 0, 43, 12] = float("nan")      # sub-aperture row 5, column 1
    sl, im, fl = _run(torch_dev, plan, opd, True)
    idx, _ = shwfs.geometry(G.CFG0)
    k = idx.index(51)
    assert fl[0, 0, k] == 1 and fl.sum() == 1 and sl[0, 0, :, k].tolist() == [0.0, 0.0]
    assert torch_dev.isnan(im[0, 0, k]).all()
    ref[0, 0, :, k] = 0.0
    assert torch_dev.equal(sl, ref)
