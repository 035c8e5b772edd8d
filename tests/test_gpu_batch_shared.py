"""The batched Ozaki-II LU with idle workgroups helping those still factoring
(few systems) and with none idle at first (more systems than workgroups), bit
for bit against the oracle: trailing blocks and panels at the edges of a task,
a zero column, widths that are no multiple of anything, and replays of a
captured graph."""
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
