"""Layer projections of more target-layer pairs than one launch's table holds (120): the kernel then makes the
maps itself, for up to 93 targets a launch, and gives the same bits as targets projected one at a time."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# pairs at the table's end and one past it, targets at the end of one launch and past it, 16 layers
@pytest.mark.parametrize("n,n_layers,n_targets", [(20, 1, 120), (20, 1, 121), (70, 7, 17), (70, 7, 18), (33, 16, 7), (33, 16, 8),
                                                  (130, 16, 40), (9, 2, 93), (9, 2, 94), (9, 3, 187)])
def test_many_targets(torch_dev, n, n_layers, n_targets):
    from paper_1408_0698_amd import shwfs
    dx, rng = 0.05, np.random.default_rng(n * n_targets)
    layers = []
    for k in range(n_layers):
        spacing = (0.05, 0.03, 0.07)[k % 3]
        side = int(n * dx / spacing) + 40
        scr = torch_dev.from_numpy(rng.normal(size=(side, side + 3)).astype(np.float32)).cuda()
        layers.append((scr, spacing, 300.0 * k, side / 2.0 + rng.uniform(-1, 1), side / 2.0 + rng.uniform(-1, 1)))
    targets = [(4e-5 * math.cos(k), 4e-5 * math.sin(k), 0.0 if k % 4 == 3 else 80e3 + 100.0 * k) for k in range(n_targets)]
    tilt = torch_dev.from_numpy(rng.normal(size=(n_targets, 2)) * 1e-6).cuda()
    out = torch_dev.full((n_targets, n + 1, n + 2), float("nan"), device="cuda")
    shwfs.project_layers(layers, n, dx, targets, out[:, :, :n], tilt=tilt)
    one = torch_dev.empty((1, n, n), device="cuda")
    for t, g in enumerate(targets):
        shwfs.project_layers(layers, n, dx, [g], one, tilt=tilt[t:t + 1])
        assert torch_dev.equal(out[t, :n, :n], one[0])
    assert out[:, n:].isnan().all() and out[:, :, n:].isnan().all()
