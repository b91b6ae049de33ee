"""FP32 GEMM vertices on k-tiled planes over many and few queries: the number
of blocks chooses the tile (128 x 128, 64 x 256, 256 x 64 where they fill the
chip, 64 x 64 where they do not, 32 x 128 and 128 x 32 for skinny results), and
every query is right at the tiles' edges, with an infinity in one operand too.

Bound: as for one vertex, 8 sqrt(12 ceil(K / 16) + 8) 2^-23 of |A| |B|."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


# (M, N, K, queries): each of the six tiles, full and with remainders
@pytest.mark.parametrize("M,N,K,Q", [
    (129, 127, 144, 64), (128, 256, 160, 128), (64, 257, 160, 128), (300, 64, 144, 128),
    (129, 127, 144, 3), (65, 33, 528, 2), (320, 190, 208, 7),
    (20, 200, 8320, 1), (140, 24, 8320, 1), (31, 129, 144, 128), (129, 32, 160, 128), (1, 130, 272, 70),
])
def test_tiles(M, N, K, Q):
    import torch
    g = torch.Generator(device="cuda").manual_seed(M * N + K + Q)
    A = torch.randn((Q, M, K), generator=g, device="cuda", dtype=torch.complex64)
    B = torch.randn((Q, K, N), generator=g, device="cuda", dtype=torch.complex64)
    bad = Q // 2
    A[bad, M // 2, K // 3] = float("inf")
    z = [np.ones((M, K), np.complex64), np.ones((K, N), np.complex64)]
    with lib.Context(2 << 30) as ctx:
        p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, z, [0, 0], 1, [(0, 1)], [0, 2], 0, lib.TN_C64)
        torch.cuda.synchronize()
        got = lib.tn_contract_strided(
            p, Q, [(0, A.data_ptr(), M * K * 8, lib.TN_C64_DEVICE), (1, B.data_ptr(), K * N * 8, lib.TN_C64_DEVICE)],
            (M, N), lib.TN_C64)[0]
    a, b = A.cpu().numpy(), B.cpu().numpy()
    for q in range(Q):
        rows = np.arange(M) != M // 2 if q == bad else np.ones(M, bool)
        if q == bad:
            assert not np.isfinite(got[q][M // 2]).any()
        ref = a[q][rows].astype(np.complex128) @ b[q].astype(np.complex128)
        size = np.abs(a[q][rows]).astype(np.float64) @ np.abs(b[q]).astype(np.float64)
        assert (np.abs(got[q][rows] - ref) <= 8 * np.sqrt(12 * -(-K // 16) + 8) * 2.0 ** -23 * size).all(), q
