"""Calls that need no ordering between streams, and calls under graph capture:
solves that overlap on several streams of one handle, and solves captured on a
handle that has none of their scratch yet.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from tests.gpu_util import note, to_dev, to_host

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
