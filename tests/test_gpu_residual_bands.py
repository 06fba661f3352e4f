"""Residuals of pupils with more groups of four pixels than one launch counts (2^30): bands of rows.

Pixels are small whole numbers, so every difference is exact.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _pattern(torch, n, rows, r0, r1, c0=0):
    y = torch.arange(r0, r1, device="cuda", dtype=torch.float32)[:, None]
    x = torch.arange(c0, c0 + n, device="cuda", dtype=torch.float32)[None, :]
    return (y % rows) * 4096.0 + x % 4096.0


# one band more than a launch takes, with a mirror; more groups than 31 bits, so that an index of one launch
# would wrap
@pytest.mark.parametrize("n,n_dm", [(65_600, 1), (92_700, 0)])
def test_residual_bands(torch_dev, n, n_dm):
    from paper_1408_0698_amd import shwfs
    torch, step = torch_dev, 4096
    assert (n + 3) // 4 * n > (2 ** 31 if n_dm == 0 else 2 ** 30)
    need = 4 * n * n * (2 + n_dm)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip("not enough free GPU memory")
    screen = torch.empty((n, n), device="cuda")
    surfs = [torch.empty((n, n), device="cuda") for _ in range(n_dm)]
    out = torch.full((1, n, n), float("nan"), device="cuda")
    for r in range(0, n, step):
        e = min(n, r + step)
        screen[r:e] = _pattern(torch, n, 977, r, e)
        for s in surfs:
            s[r:e] = _pattern(torch, n, 31, r, e, 5)
    shwfs.residual_opd(screen, surfs, n, [(0, 0)], [[(0, 0)] * n_dm], out)
    for r in range(0, n, step):
        e = min(n, r + step)
        want = _pattern(torch, n, 977, r, e)
        for _ in surfs:
            want -= _pattern(torch, n, 31, r, e, 5)
        assert torch.equal(out[0, r:e], want)
    del screen, surfs, out
    torch.cuda.empty_cache()
