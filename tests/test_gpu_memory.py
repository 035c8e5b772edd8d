"""Scratch of a handle where the GPU's memory is nearly all taken: the packed
panel leaf of an earlier limb LU makes room for a product's workspace, and a
limb LU that cannot have the leaf runs without."""
import pytest

from tests.gpu_util import note

pytestmark = pytest.mark.gpu


def test_panel_leaf_makes_room():
    import torch
    import paper_2609_29554_amd as Z
    n, nl, nc, M, K = 2048, 64, 4, 4096, 2048
    leaf_bytes = 8 * n * n * (nl + 1)            # 2.2 GB
    S, _, _, nmod, _ = Z.plan_query(53 * nc, K)
    ws_bytes = S * nmod * (2 * M * K + M * M)    # 2.3 GB with S = 2: two digit groups
    assert S == 2
    spare = 1 << 30
    assert spare < ws_bytes < spare + leaf_bytes - (64 << 20)
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.zeros(K, M, nc, dtype=torch.float64, device="cuda")
    A[..., 0] = torch.rand(K, M, generator=g, device="cuda", dtype=torch.float64)
    B = torch.zeros(M, K, nc, dtype=torch.float64, device="cuda")
    B[..., 0] = torch.rand(M, K, generator=g, device="cuda", dtype=torch.float64)
    with Z.Context(0) as c:
        want = c.gemm(0, A, B, torch.empty(M, M, nc, dtype=torch.float64, device="cuda"))
        c.sync_check()
    got = torch.zeros_like(want)
    zero = (torch.zeros(nl, n, n, dtype=torch.int64, device="cuda"),
            torch.zeros(n, n, dtype=torch.int32, device="cuda"),
            torch.zeros(n, n, dtype=torch.uint8, device="cuda"))
    hog = None
    with Z.Context(0) as c:
        try:
            note("limb LU of a zero matrix, then the memory is taken")
            _, info = c.getrf_limbs(zero, block=n, method=Z.METHOD_NAIVE)
            c.sync_check()
            assert int(info) == 1
            torch.cuda.empty_cache()
            free, _ = torch.cuda.mem_get_info()
            try:
                hog = torch.empty(free - spare, dtype=torch.uint8, device="cuda")
            except torch.OutOfMemoryError:
                pytest.skip("the free memory cannot be taken in one piece")
            free, _ = torch.cuda.mem_get_info()
            note(f"{free} bytes left, the product takes {ws_bytes}")
            assert free < ws_bytes
            c.gemm(0, A, B, got)
            c.sync_check()
            note("limb LU without its leaf")
            _, info = c.getrf_limbs(zero, block=n, method=Z.METHOD_NAIVE)
            c.sync_check()
            assert int(info) == 1
        finally:
            hog = None
            torch.cuda.empty_cache()
    assert torch.equal(got, want)
