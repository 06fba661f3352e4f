"""Residuals of more outputs than the host orders at a time (1024), and a call without memory to spare."""
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A call on made-up addresses, which fails at its first launch for want of a GPU, with the address space
# closed 64 MB above what the process has: the list of 6 million outputs must not need memory of its own.
NO_MEMORY = """
import ctypes as C, resource
from paper_1408_0698_amd import shwfs as s
n, fake = 6_000_000, C.c_void_p(0x1000)
so = (C.c_int32 * (2 * n))()
def call(n_out):
    return s._lib.shw_residual_opd(fake, 2048, 2048, 2048, 0, None, None, 800, n_out, so, None, fake, 800, 640000, None)
first = call(1)
have = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (have + (64 << 20),) * 2)
assert first != 0 and call(n) == first
"""


def test_long_list_without_memory():
    import torch
    if torch.cuda.is_available():
        pytest.skip("only where no launch can reach a GPU")
    r = subprocess.run([sys.executable, "-c", NO_MEMORY], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("n_out", [1024, 1025, 2200])
def test_groups_of_outputs(n_out):
    import torch
    from paper_1408_0698_amd import shwfs
    n, rng = 9, np.random.default_rng(n_out)
    scr = rng.normal(size=(n + 5, n + 6)).astype(np.float32)
    surf = rng.normal(size=(n + 4, n + 4)).astype(np.float32)
    so, do = rng.integers(0, 6, (n_out, 2)).tolist(), rng.integers(0, 5, (n_out, 1, 2)).tolist()
    out = torch.full((n_out, n, n), float("nan"), device="cuda")
    shwfs.residual_opd(torch.from_numpy(scr).cuda(), [torch.from_numpy(surf).cuda()], n, so, do, out)
    want = np.stack([scr[r:r + n, c:c + n] - surf[p:p + n, q:q + n] for (r, c), ((p, q),) in zip(so, do)])
    assert np.array_equal(out.cpu().numpy(), want)   # one FP32 subtraction
