"""Shared exponents (S1) of both operands, found in one launch or, on small
products, inside the producer: at the sizes where the split of the outputs
over workgroups changes (1, 4 or 16 outputs each; scans inside the producer)
and where an output's entries do not fill the threads that share it.  The
exponents and the limb products equal the oracle's."""
import numpy as np
import pytest

import oracle as O
import oracle.limbs as OL
import workloads as W
from tests.gpu_util import ctx, note, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc,M,N,K", [
    (4, 1, 1, 1), (2, 17, 33, 5), (4, 16, 31, 64), (3, 40, 15, 129), (2, 511, 513, 300),
    (4, 515, 1030, 70), (3, 4099, 3, 65), (2, 3, 4097, 1000), (4, 600, 600, 700),
])
def test_exponents_of_both_operands(nc, M, N, K):
    note(f"exponents nc={nc} {M}x{N}x{K}")
    rng = np.random.default_rng(1000 * nc + M + N + K)
    A = W.random_expansions(M, K, nc, rng, exp_sigma=30.0)
    B = W.random_expansions(K, N, nc, rng, exp_sigma=30.0)
    A[:, M // 2] = 0.0                # a zero row of A, a zero column of B
    B[N // 2] = 0.0
    A[0, M - 1, 0] = 0.0              # a zero leading component
    C = np.zeros((N, M, nc))
    st = ctx().gemm_stages(0, to_dev(A), to_dev(B), to_dev(C))
    ctx().sync_check()
    assert np.array_equal(to_host(st["ea"]), O.exponents(A, True))
    assert np.array_equal(to_host(st["eb"]), O.exponents(B, False))


@pytest.mark.parametrize("nc,M,N,K", [(2, 5, 16390, 40), (3, 16385, 4, 33), (4, 4096, 5, 70),
                                      (2, 2, 16383, 65)])
def test_exponents_of_many_outputs(nc, M, N, K):
    """Eight outputs each from 4096, sixteen from 16384 on."""
    test_exponents_of_both_operands(nc, M, N, K)


@pytest.mark.parametrize("nl,M,N,K", [(1, 4100, 3, 200), (2, 5, 600, 700), (1, 513, 2, 3)])
def test_limb_product_rows(nl, M, N, K):
    """Sampled rows of A against all of B (row exponents are per row)."""
    note(f"limb exponents nl={nl} {M}x{N}x{K}")
    rng = np.random.default_rng(77 + M + N + K)
    A = W.random_limbs(M, K, nl, rng, exp_sigma=30.0, zero_frac=0.3)
    B = W.random_limbs(K, N, nl, rng, exp_sigma=30.0, zero_frac=0.3)
    C = W.random_limbs(M, N, nl, rng)
    rows = np.unique(np.r_[0, M - 1, rng.integers(0, M, 3)])
    cols = np.unique(np.r_[0, N - 1, rng.integers(0, N, 3)])
    sub = tuple(np.ascontiguousarray(x[..., rows]) for x in A)
    subB = tuple(np.ascontiguousarray(x[..., cols, :]) for x in B)
    want, _ = OL.ozgemm(0, sub, subB, tuple(np.ascontiguousarray(x[..., cols, :][..., rows]) for x in C),
                        O.make_plan(64 * nl, K))
    d = lambda X: (to_dev(X[0].view(np.int64)), to_dev(X[1]), to_dev(X[2]))  # noqa: E731
    out = d(C)
    ctx().gemm_limbs(0, d(A), d(B), out)
    ctx().sync_check()
    got = (to_host(out[0]).view(np.uint64), to_host(out[1]), to_host(out[2]))
    for g, w in zip(got, want):
        assert np.array_equal(g[..., cols, :][..., rows], w)
