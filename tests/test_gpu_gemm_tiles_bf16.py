"""BF16x3 GEMM vertices on k-tiled planes over many and few queries: 64 x 64
tiles where the larger ones would leave compute units idle or run half empty.
Every query is right at the tiles' edges, in its group and by itself.

Bound: FP32 sums of 3 K products, 8 sqrt(12 ceil(K / 16) + 8) 2^-23 of |A| |B|, and
the dropped product of the low terms, 2^-12 with the sums 3M forms."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [0, lib.TN_FORM_3M])
@pytest.mark.parametrize("M,N,K,Q", [
    (256, 256, 144, 160), (129, 127, 144, 70), (129, 127, 144, 3), (65, 130, 144, 2), (64, 300, 528, 4),
    (300, 33, 160, 2), (1, 200, 272, 3), (17, 257, 4112, 1), (500, 400, 208, 9),
])
def test_tiles(M, N, K, Q, form):
    import torch
    g = torch.Generator(device="cuda").manual_seed(M * N + K + Q)
    A = torch.randn((Q, M, K), generator=g, device="cuda", dtype=torch.complex64)
    B = torch.randn((Q, K, N), generator=g, device="cuda", dtype=torch.complex64)
    z = [np.ones((M, K), np.complex64), np.ones((K, N), np.complex64)]
    with lib.Context(2 << 30) as ctx:
        p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, z, [0, 0], 1, [(0, 1)], [0, 2],
                          lib.TN_PREC_BF16X3 | form, lib.TN_C64)
        torch.cuda.synchronize()

        def run(q0, n):
            return lib.tn_contract_strided(p, n, [
                (0, A.data_ptr() + q0 * M * K * 8, M * K * 8, lib.TN_C64_DEVICE),
                (1, B.data_ptr() + q0 * K * N * 8, K * N * 8, lib.TN_C64_DEVICE)], (M, N), lib.TN_C64)[0]

        got, one = run(0, Q), run(Q - 1, 1)
    a, b = A.cpu().numpy(), B.cpu().numpy()
    for q in range(Q):
        size = np.abs(a[q]).astype(np.float64) @ np.abs(b[q]).astype(np.float64)
        tol = 8 * np.sqrt(12 * -(-K // 16) + 8) * 2.0 ** -23 + 2.0 ** -12
        for c in (got[q],) + ((one[0],) if q == Q - 1 else ()):
            assert (np.abs(c - a[q].astype(np.complex128) @ b[q]) <= tol * size).all(), q
