"""getrf where a panel's rows fit one workgroup (up to 32) and just above, as
the whole matrix and as the last panel, with ties and zero columns,
bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import ctx, note, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,n,b", [(2, 1, 32), (4, 2, 32), (3, 31, 32), (4, 32, 32), (2, 33, 32),
                                    (4, 34, 32), (2, 64, 32), (4, 65, 32), (3, 96, 64), (2, 32, 5)])
@pytest.mark.parametrize("kind", ["random", "ties", "zero"])
def test_small_panels(nc, n, b, kind):
    import paper_2609_29554_amd as Z
    note(f"getrf small panels nc={nc} n={n} b={b} {kind}")
    A = W.graded(n, nc, 30.0, np.random.default_rng(n + nc))
    if kind == "ties":
        A[:, :, 0] = np.where(A[:, :, 0] < 0, -1.0, 1.0)
        A[:, :, 1:] = 0.0
        A[np.arange(n), np.arange(n), 0] = 3.0
    if kind == "zero":
        A[n // 2] = 0.0
    LU, ipiv, info, _ = O.getrf(A, b, O.METHOD_OZAKI, O.make_plan(53 * nc, b))
    src = to_dev(A)
    dA = src.clone()
    opts = Z.make_opts(block=b, method=Z.METHOD_OZAKI, backend=Z.BE_INT8)
    for _ in range(2):
        dA.copy_(src)
        dip, dinfo = ctx().getrf(dA, block=b, method=Z.METHOD_OZAKI, opts=opts)
        ctx().sync_check()
        assert int(to_host(dinfo)[0]) == info
        assert np.array_equal(to_host(dip), ipiv)
        assert np.array_equal(to_host(dA), LU)


@pytest.mark.parametrize("nc,n,b", [(2, 100, 85), (2, 100, 86), (3, 290, 256), (2, 345, 340),
                                    (2, 345, 341), (4, 150, 130)])
def test_wide_panels(nc, n, b):
    """Widths at which the rows of a workgroup change, and few rows a workgroup."""
    note(f"wide panel nc={nc} n={n} b={b}")
    rng = np.random.default_rng(n + b)
    A = W.graded(n, nc, 20.0, rng)
    want, ipiv, info, _ = O.getrf(A, b, O.METHOD_OZAKI)
    dA = to_dev(A)
    ip, inf = ctx().getrf(dA, block=b)
    ctx().sync_check()
    assert int(inf) == info and np.array_equal(to_host(ip), ipiv)
    assert np.array_equal(to_host(dA), want)


def test_tags_start_over():
    """Refused factorisations of order 2^20, b = 1, use up a quarter of the
    panels' tags each, so that the words are cleared between the others."""
    import ctypes as C
    import torch
    import paper_2609_29554_amd as Z
    rng = np.random.default_rng(11)
    c = Z.Context(0)
    cases = []
    for nc, n, b in ((2, 150, 64), (4, 70, 32)):
        A = W.graded(n, nc, 20.0, rng)
        cases.append((to_dev(A), b) + O.getrf(A, b, O.METHOD_OZAKI)[:3])
    small = torch.zeros(16, dtype=torch.float64, device="cuda")
    ipiv = torch.zeros(16, dtype=torch.int64, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    o = Z.make_opts(block=1, method=Z.METHOD_NAIVE)
    for rep in range(6):
        note(f"tags start over rep={rep}")
        for dA, b, want, ip, inf in cases:
            X = dA.clone()
            p, i = c.getrf(X, block=b)
            c.sync_check()
            assert int(i) == inf and np.array_equal(to_host(p), ip)
            assert np.array_equal(to_host(X), want)
        st = Z.lib().ozII_getrf(c._h, 2, 1 << 20, small.data_ptr(), 1 << 20, ipiv.data_ptr(),
                                info.data_ptr(), C.byref(o))
        assert st == Z.EUNSUPPORTED   # no panel of so many rows; nothing is factored
    c.close()
