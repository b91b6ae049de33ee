"""FP32 GEMM vertices on planes whose rows have one entry each: every result is
one product, in which the order that its bfloat16 terms are added in shows.  No
less accurate, in the mean square, than one complex64 multiplication (products
rounded, then their sum)."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [(1024, 16, 1152), (1030, 64, 1100), (64, 256, 1030), (1030, 256, 64), (260, 528, 190),
                                   (32, 4096, 512), (512, 4096, 32)])
@pytest.mark.parametrize("form", [0, lib.TN_FORM_3M])
def test_one_product(M, K, N, form):
    rng = np.random.default_rng([M, N, K])
    A = np.zeros((M, K), np.complex64)
    k = rng.integers(0, K, M)
    a = (rng.uniform(0.5, 1.5, M) + 1j * rng.uniform(0.5, 1.5, M)).astype(np.complex64)
    A[np.arange(M), k] = a
    B = (rng.uniform(0.5, 1.5, (K, N)) + 1j * rng.uniform(0.5, 1.5, (K, N))).astype(np.complex64)
    with lib.Context(1 << 30) as ctx:
        p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, [A, B], [0, 0], 1, [(0, 1)], [0, 2], form, lib.TN_C64)
        got, _ = lib.tn_contract(p, None, (M, N), lib.TN_C64)
    b = B[k]
    ref = a.astype(np.complex128)[:, None] * b
    re = a.real[:, None] * b.real - a.imag[:, None] * b.imag
    im = a.real[:, None] * b.imag + a.imag[:, None] * b.real
    assert re.dtype == np.float32
    assert np.linalg.norm(got - ref) <= np.linalg.norm(re + 1j * im.astype(np.float64) - ref)
