"""Calls that need no ordering between streams, and calls under graph capture:
solves that overlap on several streams of one handle, and solves captured on a
handle with and without their scratch.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as O
import oracle.limb_lu as OLU
import workloads as W
from tests.gpu_util import note, to_dev, to_host
from tests.test_gpu_limb_lu import _dev, _host, _matrix, _same

pytestmark = pytest.mark.gpu


def _system(nc, n, nrhs, seed):
    rng = np.random.default_rng(seed)
    LU = np.where(np.eye(n, dtype=bool)[..., None], 1.0, 2.0 ** -10) * W.wellcond(n, nc, rng)
    ipiv = np.array([rng.integers(j, n) for j in range(n)], dtype=np.int64)
    B = W.random_expansions(n, nrhs, nc, rng, exp_sigma=2.0)
    return LU, ipiv, B, O.getrs(LU, ipiv, B)


def test_getrs_overlapping_streams():
    import torch
    import paper_2609_29554_amd as Z
    c = Z.Context(0)
    shapes = [(2, 300, 4), (4, 270, 2), (2, 513, 3), (3, 290, 5)]
    sys_ = [_system(nc, n, r, 10 * n + r) for nc, n, r in shapes]
    dev = [(to_dev(LU), torch.from_numpy(ip).cuda(), to_dev(B)) for LU, ip, B, _ in sys_]
    out = [[torch.empty_like(B) for _ in range(4)] for _, _, B in dev]
    streams = [torch.cuda.Stream() for _ in shapes]
    torch.cuda.synchronize()
    note("getrs on four streams at once")
    for rep in range(4):
        for (LU, ip, B), x, s in zip(dev, out, streams):
            with torch.cuda.stream(s):
                x[rep].copy_(B)
                c.getrs(LU, ip, x[rep])
    torch.cuda.synchronize()
    c.sync_check()
    for (_, _, _, want), x in zip(sys_, out):
        for y in x:
            assert np.array_equal(to_host(y), want)


@pytest.mark.parametrize("warm", [False, True])
def test_getrs_captured(warm):
    """On a fresh handle, and after the same call outside the capture."""
    import torch
    import paper_2609_29554_amd as Z
    note(f"captured getrs warm={warm}")
    c = Z.Context(0)
    LU, ip, B, want = _system(2, 300, 3, 5)
    dLU, dip, dB = to_dev(LU), torch.from_numpy(ip).cuda(), to_dev(B)
    X = torch.empty_like(dB)
    if warm:
        c.getrs(dLU, dip, dB.clone())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        X.copy_(dB)
        c.getrs(dLU, dip, X)
    other = _system(2, 400, 2, 6)
    o = [to_dev(other[0]), torch.from_numpy(other[1]).cuda(), to_dev(other[2])]
    for _ in range(3):
        g.replay()
        y = o[2].clone()
        c.getrs(o[0], o[1], y)  # beside the replay or after it
        torch.cuda.synchronize()
        assert np.array_equal(to_host(X), want)
        assert np.array_equal(to_host(y), other[3])
        X.zero_()
    c.sync_check()


def _limb_system(nl, n, nrhs):
    F, ip, _ = OLU.getrf(_matrix(nl, n, 3 * n + nl), n, "native")
    B = W.random_limbs(n, nrhs, nl, np.random.default_rng(n), exp_sigma=2.0, zero_frac=0.05)
    return F, ip.copy(), B, OLU.getrs(F, ip, B)


def test_getrs_limbs_overlapping_streams():
    import torch
    import paper_2609_29554_amd as Z
    c = Z.Context(0)
    sys_ = [_limb_system(nl, n, r) for nl, n, r in [(4, 60, 1), (8, 45, 3), (17, 30, 2), (4, 70, 2)]]
    dev = [(_dev(F), torch.from_numpy(ip).cuda(), _dev(B)) for F, ip, B, _ in sys_]
    out = [[tuple(torch.empty_like(t) for t in B) for _ in range(4)] for _, _, B in dev]
    streams = [torch.cuda.Stream() for _ in sys_]
    torch.cuda.synchronize()
    note("getrs_limbs on four streams at once")
    for rep in range(4):
        for (F, ip, B), x, s in zip(dev, out, streams):
            with torch.cuda.stream(s):
                for d, t in zip(x[rep], B):
                    d.copy_(t)
                c.getrs_limbs(F, ip, x[rep])
    torch.cuda.synchronize()
    for (_, _, _, want), x in zip(sys_, out):
        for y in x:
            _same(_host(y), want)


@pytest.mark.parametrize("warm", [False, True])
def test_getrs_limbs_captured(warm):
    """Captured on a fresh handle and after a call outside the capture; a larger
    solve replaces the handle's scratch between the replays."""
    import torch
    import paper_2609_29554_amd as Z
    note(f"captured getrs_limbs warm={warm}")
    c = Z.Context(0)
    F, ip, B, want = _limb_system(5, 40, 2)
    dF, dip, dB = _dev(F), torch.from_numpy(ip).cuda(), _dev(B)
    X = tuple(torch.empty_like(t) for t in dB)
    if warm:
        c.getrs_limbs(dF, dip, _dev(B))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for d, t in zip(X, dB):
            d.copy_(t)
        c.getrs_limbs(dF, dip, X)
    for nl, n in ((5, 55), (9, 60), (16, 64)):
        o = _limb_system(nl, n, 1)
        y = _dev(o[2])
        c.getrs_limbs(_dev(o[0]), torch.from_numpy(o[1]).cuda(), y)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        _same(_host(X), want)
        _same(_host(y), o[3])
        for t in X:
            t.zero_()


@pytest.mark.parametrize("nl,n,b,leaf,warm", [
    (4, 40, 40, 0, 40),    # captured with the packed leaf
    (4, 40, 40, 0, 5),     # not allocated at that size: on the planes
    (9, 24, 24, 7, 24), (9, 24, 24, 7, 3),
    (2, 90, 80, 0, 90), (2, 90, 80, 0, 4),   # leaf wider than 64 columns
])
def test_getrf_limbs_captured(nl, n, b, leaf, warm):
    """Larger factorisations replace the handle's scratch between the replays."""
    import torch
    import paper_2609_29554_amd as Z
    note(f"captured getrf_limbs nl={nl} n={n} b={b} leaf={leaf} warm={warm}")
    c = Z.Context(0)
    c.getrf_limbs(_dev(_matrix(nl, warm, 1)), block=b, method=Z.METHOD_NAIVE, leaf=leaf)
    A = _matrix(nl, n, 7)
    want, ip, inf = OLU.getrf(A, b, "native", leaf=leaf)
    dA = _dev(A)
    X = tuple(torch.empty_like(t) for t in dA)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for d, t in zip(X, dA):
            d.copy_(t)
        ipiv, info = c.getrf_limbs(X, block=b, method=Z.METHOD_NAIVE, leaf=leaf)
    for m in (n + 20, n + 40, n + 60):
        O2 = _matrix(nl, m, m)
        y = _dev(O2)
        c.getrf_limbs(y, block=m, method=Z.METHOD_NAIVE, leaf=0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        _same(_host(X), want)
        assert np.array_equal(to_host(ipiv)[:n], ip) and int(info) == inf
        _same(_host(y), OLU.getrf(O2, m, "native")[0])
        for t in X:
            t.zero_()
