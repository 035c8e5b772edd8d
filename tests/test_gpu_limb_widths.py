"""GPU parity of the limb arithmetic, LU and solve where their kernels change
form: limb counts at the edges of the matrix-core product's sizes, divisions
in one and two registers of digits, the division by stored reciprocals in the
solve, pivots decided below the top limb, U12 leaves held in registers and in
memory, and interchanges of more than one batch of 256.  Bit for bit against
the oracle."""
import random

import numpy as np
import pytest

import oracle.lfloat as LF
import oracle.limb_lu as OLU
import workloads as W
from tests.gpu_util import ctx, note
from tests.test_gpu_limb_lu import (_arith_cases, _dev, _host, _lu, _matrix, _pack_vec, _same)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nl", [4, 15, 16, 17, 32, 33, 48, 57, 63])
@pytest.mark.parametrize("op", ["add", "mul", "div"])
def test_arith_at_size_edges(nl, op):
    note(f"limbs_arith edge nl={nl} op={op}")
    p = 64 * nl
    cs = _arith_cases(op, nl, 60, 77 * nl + len(op))
    rng = random.Random(nl)
    ones, half = (1 << p) - 1, 1 << (p - 1)
    sp = [half, half + 1, ones, ones - 1, half | 1 << 63, ones ^ (1 << 64) - 1,
          int("80" * (8 * nl), 16), int("7f" * (8 * nl), 16) | half, int("81" * (8 * nl), 16)]
    cs += [((x, 0, 0), (y, rng.randrange(-2, 3), rng.randrange(2))) for x in sp for y in sp]
    A = _pack_vec([a for a, _ in cs], nl)
    B = _pack_vec([b for _, b in cs], nl)
    want = OLU.from_lf(LF.vec(op, OLU.to_lf(A), OLU.to_lf(B)))
    dA, dB = _dev(A), _dev(B)
    dC = _dev(tuple(np.zeros_like(x) for x in A))
    ctx().limbs_arith(op, dA, dB, dC)
    ctx().sync_check()
    _same(_host(dC), want)


@pytest.mark.parametrize("nl,n,nrhs,kind", [(4, 40, 2, "random"), (17, 20, 1, "random"),
                                            (49, 18, 1, "powers"), (64, 17, 2, "random"),
                                            (1, 300, 1, "random"), (8, 33, 1, "zero")])
def test_solve(nl, n, nrhs, kind):
    note(f"getrs_limbs nl={nl} n={n} {kind}")
    A = _matrix(nl, n, 3 * n + nl)
    F, ip, _ = OLU.getrf(A, n, "native")
    F = tuple(x.copy() for x in F)
    if kind == "powers":                          # power-of-two and all-ones diagonals
        for k in range(0, n, 2):
            F[0][:, k, k] = 0 if k % 4 == 0 else np.uint64(2 ** 64 - 1)
            F[0][nl - 1, k, k] = np.uint64(1 << 63) if k % 4 == 0 else np.uint64(2 ** 64 - 1)
    if kind == "zero":                            # an exactly zero u_kk
        F[0][:, 5, 5] = 0
        F[1][5, 5] = OLU.EXP32_ZERO
        F[2][5, 5] = 0
    B = W.random_limbs(n, nrhs, nl, np.random.default_rng(n), exp_sigma=2.0, zero_frac=0.05)
    if kind == "powers":                          # exact quotients and ties
        B[0][:, 0, ::3] = F[0][:, n - 1, n - 1][:, None]
    want = OLU.getrs(F, ip, B)
    import torch
    dB = _dev(B)
    ctx().getrs_limbs(_dev(F), torch.from_numpy(ip.copy()).cuda(), dB)
    ctx().sync_check()
    _same(_host(dB), want)


@pytest.mark.parametrize("nl,n", [(1, 270), (4, 600)])
def test_solve_any_interchanges(nl, n):
    """Interchanges with any row, those above the batch of 256 included."""
    note(f"getrs_limbs interchanges nl={nl} n={n}")
    rng = np.random.default_rng(n)
    F = tuple(x.copy() for x in W.random_limbs(n, n, nl, rng, exp_sigma=0.0, zero_frac=0.0))
    for x in F:                                    # the unit matrix
        x[...] = 0
    F[1][...] = OLU.EXP32_ZERO
    d = np.arange(n)
    F[0][nl - 1, d, d] = np.uint64(1 << 63)
    F[1][d, d] = 1
    ip = rng.integers(0, n, n)
    ip[[n - 1, n - 3, 10]] = [3, 255, n - 2]
    B = W.random_limbs(n, 2, nl, rng, exp_sigma=2.0, zero_frac=0.05)
    order = np.arange(n)
    for j in range(n):
        order[[j, ip[j]]] = order[[ip[j], j]]
    import torch
    dB = _dev(B)
    ctx().getrs_limbs(_dev(F), torch.from_numpy(ip).cuda(), dB)
    ctx().sync_check()
    _same(_host(dB), tuple(x[..., order] for x in B))


@pytest.mark.parametrize("nl,n,b,leaf,method", [(5, 45, 45, 0, "native"), (17, 24, 24, 8, "native"),
                                                (4, 50, 50, 33, "ozaki"), (33, 12, 6, 3, "ozaki"),
                                                (2, 80, 16, 0, "native")])
def test_lu_with_tied_pivots(nl, n, b, leaf, method):
    """Entries that share exponent and top limb (or are equal) in every column."""
    note(f"getrf_limbs ties nl={nl} n={n} b={b} leaf={leaf} {method}")
    A = _matrix(nl, n, 11 * n + nl)
    live = A[0][nl - 1] != 0
    A[1][live] = 0
    A[0][nl - 1][live] = np.uint64(1 << 63)       # equal exponents and top limbs
    for x in A:
        x[..., :, n // 2] = x[..., :, n // 3]     # two equal rows
    got, ipiv, info = _lu(A, b, method, leaf)
    want, ip, inf = OLU.getrf(A, b, method, leaf=leaf)
    _same(got, want)
    assert np.array_equal(ipiv[:n], ip) and info == inf


