"""Bit permutations through the tiled kernel: a GEMM vertex whose operands'
legs (dimension 2) come in shuffled orders, several queries in one call, the
result in another shuffled order: both operand permutations into every kind of
planes (k-tiled), and the complex64 output permutation.  Rows of 2^1 and 2^11
entries, k of 2^4 to 2^10, orders that keep the low legs in place or reverse
all of them.

Bound: a sum of 2 K products, FP32 additions (8 sqrt(2 K + 8) 2^-23 of |A| |B|); BF16x3
drops the product of the low terms (2^-16 of |A| |B|, 3M of sums of parts), and its
sum of K such errors of either sign stays below 2^-12 of |A| |B|."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu
Q = 3


@pytest.fixture(scope="module")
def ctx():
    c = lib.Context(2 << 30)
    yield c
    c.close()


def order(rng, legs, how):
    legs = list(legs)
    if how == "reversed":
        return legs[::-1]
    if how == "low legs kept":
        head = legs[:-6]
        return [head[i] for i in rng.permutation(len(head))] + legs[-6:]
    return [legs[i] for i in rng.permutation(len(legs))]


@pytest.mark.parametrize("how", ["shuffled", "reversed", "low legs kept"])
@pytest.mark.parametrize("m,n,k", [(9, 9, 4), (7, 6, 10), (11, 3, 8), (3, 13, 7), (6, 11, 5)])
@pytest.mark.parametrize("flags", [0, lib.TN_PREC_BF16X3, lib.TN_PREC_BF16X3 | lib.TN_FORM_3M])
def test_shuffled_legs(ctx, m, n, k, how, flags):
    import torch
    rng = np.random.default_rng([m, n, k])
    M, K, N = range(m), range(m, m + k), range(m + k, m + k + n)
    la, lb = order(rng, list(M) + list(K), how), order(rng, list(K) + list(N), how)
    out = order(rng, list(M) + list(N), "shuffled")
    dims = {e: 2 for e in range(m + k + n)}
    a = (rng.standard_normal((Q, 1 << (m + k), 2))).astype(np.float32).view(np.complex64)[..., 0]
    b = (rng.standard_normal((Q, 1 << (k + n), 2))).astype(np.float32).view(np.complex64)[..., 0]
    zero = [np.zeros((2,) * len(x), np.complex64) for x in (la, lb)]
    p = ctx.plan_load([la, lb], dims, zero, [0, 0], 1, [(0, 1)], out, flags, lib.TN_C64)
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    got, _ = lib.tn_contract_strided(p, Q, [(0, da.data_ptr(), a[0].nbytes, lib.TN_C64_DEVICE),
                                            (1, db.data_ptr(), b[0].nbytes, lib.TN_C64_DEVICE)],
                                     (1 << (m + n),), lib.TN_C64, scales=False)
    ctx.free_plan(p)
    tol = 8 * np.sqrt(2.0 * (1 << k) + 8) * 2.0 ** -23 + (2.0 ** -12 if flags else 0)
    for q in range(Q):
        A = a[q].reshape((2,) * len(la)).transpose([la.index(e) for e in list(M) + list(K)]).reshape(1 << m, 1 << k)
        B = b[q].reshape((2,) * len(lb)).transpose([lb.index(e) for e in list(K) + list(N)]).reshape(1 << k, 1 << n)

        def ordered(c):
            rows = list(M) + list(N)
            return c.reshape((2,) * (m + n)).transpose([rows.index(e) for e in out]).reshape(-1)
        ref = ordered(A.astype(np.complex128) @ B.astype(np.complex128))
        size = ordered(np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64))
        over = np.abs(got[q] - ref) / (tol * size)
        assert over.max() <= 1.0, (q, over.max())
