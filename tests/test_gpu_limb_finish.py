"""The last steps of the limb product, bit for bit against the oracle, on both
sides of the rule that chooses between one pass and separate kernels, at the
edges of a workgroup's 32 elements, with products that
cancel against C exactly or down to the last bits, and zeros on either side."""
import numpy as np
import pytest

import oracle as O
import oracle.limbs as OL
import workloads as W
from tests.gpu_util import ctx, note
from tests.test_gpu_limbs import _dev, _host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nl,M,N,K,mode,be", [
    (1, 16, 16, 5, 0, 0), (1, 257, 1, 5, 0, 0), (1, 768, 1, 3, 1, 0), (1, 769, 1, 3, 1, 0),
    (2, 31, 33, 9, 0, 0), (2, 33, 32, 9, 0, 0), (2, 96, 32, 4, 1, 0), (2, 97, 32, 4, 1, 0),
    (3, 65, 3, 70, 1, 0), (3, 33, 5, 12, 1, 1), (31, 32, 2, 6, 1, 0), (32, 63, 2, 6, 0, 0),
    (63, 33, 2, 4, 1, 0), (64, 1, 1, 1, 1, 0), (64, 64, 1, 3, 1, 1), (65, 5, 3, 4, 1, 0),
])
@pytest.mark.parametrize("near", [False, True])
def test_finish(nl, M, N, K, mode, be, near):
    import paper_2609_29554_amd as Z
    note(f"limb finish nl={nl} {M}x{N}x{K} mode={mode} be={be} near={near}")
    rng = np.random.default_rng(nl * 1000 + M + mode)
    A, B, C0 = (W.random_limbs(r, c, nl, rng, exp_sigma=3.0, zero_frac=0.1)
                for r, c in ((M, K), (K, N), (M, N)))
    opts = Z.make_opts(backend=Z.BE_F64MOD) if be else None
    pl = O.make_plan(64 * nl, K, **({"backend": O.BACKEND_F64MOD} if be else {}))
    if near:      # C: the rounded product, exactly or one unit away, or a far smaller number
        C0, _ = OL.ozgemm(0, A, B, C0, pl)
        C0 = tuple(x.copy() for x in C0)
        odd = rng.random((N, M)) < 0.5
        C0[0][0][odd & (C0[1] != OL.EXP_ZERO)] ^= np.uint64(1)
        far = rng.random((N, M)) < 0.2
        C0[1][far & (C0[1] != OL.EXP_ZERO)] -= 64 * nl + rng.integers(0, 3)
    want, _ = OL.ozgemm(mode, A, B, C0, pl)
    dA, dB, dC = _dev(A), _dev(B), _dev(C0)
    ctx().gemm_limbs(mode, dA, dB, dC, opts)
    ctx().sync_check()
    for g, w_, name in zip(_host(dC), want, ("limbs", "exp", "sign")):
        assert np.array_equal(g, w_), name
