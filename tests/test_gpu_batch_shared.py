"""The batched Ozaki-II LU with idle workgroups helping those still factoring
(few systems) and with none idle at first (more systems than workgroups), bit
for bit against the oracle: trailing blocks and panels at the edges of a task,
a zero column, widths that are no multiple of anything, and replays of a
captured graph; orders above the threads of a workgroup."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from gpu_util import ctx, note, to_host
from test_gpu_batch_ozaki import _check, _device, _expected

pytestmark = pytest.mark.gpu


def _systems(sizes, seed):
    rng = np.random.default_rng(seed)
    out = []
    for nc, n in sizes:
        A = W.graded(n, nc, float(rng.uniform(20, 60)), rng)
        if n % 7 == 3:
            A[n // 2, :, :] = 0.0
        out.append((nc, A, W.rhs_ones(A)))
    return out


@pytest.mark.parametrize("b,sizes", [
    (64, [(2, 128), (3, 129), (4, 130), (2, 192), (4, 193), (2, 257)]),
    (7, [(2, 71), (3, 72), (4, 80), (2, 143)]),
    (1, [(2, 66), (4, 67)]),
    (70, [(4, 135), (2, 200), (3, 207)]),
    (256, [(2, 322)]),
])
def test_few(b, sizes):
    import paper_2609_29554_amd as Z
    note(f"shared batch b={b}")
    systems = _systems(sizes, b)
    exp = _expected(systems, b)
    dev = _device(systems)
    ctx().batch_prepare(dev, Z.make_opts(block=b, method=Z.METHOD_OZAKI))
    ctx().batch_run()
    ctx().sync_check()
    _check(dev, exp, systems)


def test_more_than_workgroups():
    import torch
    import paper_2609_29554_amd as Z
    note("shared batch, 600 systems, graph replays")
    base = _systems([(2, 130), (4, 97), (3, 66), (2, 33), (4, 10)], 5)
    exp = _expected(base, 32)
    systems = base * 120
    src, work = _device(systems), _device(systems)
    c = ctx()
    c.batch_prepare(work, Z.make_opts(block=32, method=Z.METHOD_OZAKI))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.batch_run()
    for _ in range(3):
        for (a0, b0, _, _), (a, b, _, _) in zip(src, work):
            a.copy_(a0)
            b.copy_(b0)
        g.replay()
        torch.cuda.synchronize()
        _check(work, exp * 120, systems)


@pytest.mark.parametrize("nc,n,b", [(2, 1024, 0), (3, 1025, 0), (2, 1030, 0), (2, 1024, 64),
                                    (4, 513, 32), (3, 600, 128)])
def test_several_rows_per_thread(nc, n, b):
    """Orders above the threads of a workgroup: the factors and solution of
    getrf / getrs at the same block (b = 0: unblocked, native update)."""
    import torch
    import paper_2609_29554_amd as Z
    note(f"batch against getrf nc={nc} n={n} b={b}")
    g = torch.Generator(device="cuda").manual_seed(n + nc)
    A = torch.zeros(n, n, nc, dtype=torch.float64, device="cuda")
    A[..., 0] = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64)
    A[..., 1] = A[..., 0] * 2.0 ** -56 * torch.rand(n, n, generator=g, device="cuda", dtype=torch.float64)
    B = torch.zeros(1, n, nc, dtype=torch.float64, device="cuda")
    B[..., 0] = torch.randn(1, n, generator=g, device="cuda", dtype=torch.float64)
    LU, X = A.clone(), B.clone()
    ip = torch.zeros(n, dtype=torch.int64, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    c = ctx()
    opts = Z.make_opts(block=b, method=Z.METHOD_OZAKI, backend=Z.BE_INT8) if b else None
    c.batch_prepare([(LU, X, ip, info)], opts)
    c.batch_run()
    c.sync_check()
    wLU, wX = A.clone(), B.clone()
    if b:
        wip, winfo = c.getrf(wLU, block=b, method=Z.METHOD_OZAKI, opts=opts)
    else:
        wip, winfo = c.getrf(wLU, block=1, method=Z.METHOD_NAIVE)
    c.getrs(wLU, wip, wX)
    c.sync_check()
    assert torch.equal(ip, wip) and int(info) == int(winfo) == 0
    assert torch.equal(LU, wLU)
    assert torch.equal(X, wX)


def test_largest_order_shared():
    """The largest accepted QD system, its first block shared too."""
    test_several_rows_per_thread(4, 1024, 64)
