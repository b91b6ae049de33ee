"""FP32 GEMM vertices with a long k that is no multiple of 16: k is summed in
chunks.  Bound, of the 2-norm: an addition to a chunk's sum is off by at most
2^-24 of it, uniformly, and a sum of random signs grows as the root of its
terms, so a chunk of at most 2048 k (4096 additions) and 64 chunks are off by
2^-24 sqrt((4096 + 64) / 6)."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(20, 20001, 24), (64, 32767, 64), (8, 20001, 2000), (200, 30001, 200),
                                   (500, 10001, 500), (1000, 8191, 1000)])
def test_long_k(M, K, N):
    rng = np.random.default_rng([M, K, N])
    A, B = ((rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64) for s in ((M, K), (K, N)))
    with lib.Context(2 << 30) as ctx:
        p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, [A, B], [0, 0], 1, [(0, 1)], [0, 2], 0, lib.TN_C64)
        got, _ = lib.tn_contract(p, None, (M, N), lib.TN_C64)
    ref = A.astype(np.complex128) @ B.astype(np.complex128)
    assert np.linalg.norm(got - ref) <= 2.0 ** -24 * np.sqrt((4096 + 64) / 6) * np.linalg.norm(ref)
