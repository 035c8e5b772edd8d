"""GPU parity of the solve with several right-hand sides where its route
changes: the blocked solves of one, two and four wavefronts per column (orders
up to 256, or more right-hand sides than the chip holds pipelines for) and
the pipelined one that takes right-hand sides in pairs, the last one alone.
Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import ctx, note, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,n,nrhs", [(2, 1, 2), (2, 64, 5), (3, 65, 2), (4, 128, 3), (2, 129, 4),
                                       (4, 256, 2), (2, 257, 2), (3, 300, 5), (4, 289, 3),
                                       (2, 320, 110)])
def test_getrs_several_rhs(nc, n, nrhs):
    note(f"getrs nc={nc} n={n} nrhs={nrhs}")
    import torch
    rng = np.random.default_rng(100 * n + nrhs)
    # any factors will do; small ones below a dominant diagonal keep x finite
    LU = np.where(np.eye(n, dtype=bool)[..., None], 1.0, 2.0 ** -10) * W.wellcond(n, nc, rng)
    ipiv = np.array([rng.integers(j, n) for j in range(n)], dtype=np.int64)
    B = W.random_expansions(n, nrhs, nc, rng, exp_sigma=2.0)
    B[0, n // 2] = 0.0
    want = O.getrs(LU, ipiv, B)
    dB = to_dev(B)
    ctx().getrs(to_dev(LU), torch.from_numpy(ipiv).cuda(), dB)
    ctx().sync_check()
    assert np.isfinite(want).all() and np.array_equal(to_host(dB), want)
