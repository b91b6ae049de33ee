"""One GEMM vertex against complex128, on the kernel its shape selects: the
FP32 GEMM on k-tiled planes (three bfloat16 terms per value, six products) at
tile edges, short and long k, split k, every tile shape, entries of very
different size, and an operand that holds an infinity; and the kernel that
reads its operands in place, at its tile edges and with scattered legs.

Bound: a result entry is a sum of 2 * 6 * ceil(K / 16) matrix products added
to an FP32 accumulator, each addition off by at most 2^-23 of the partial sum
(which |A| |B| bounds), plus the split-k sum; independent errors add in
quadrature, eight standard deviations are allowed.  The dropped products and
the splits are below 2^-24 per term."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = lib.Context(2 << 30)
    yield c
    c.close()


def run_pair(ctx, A, B, flags, cls="gemm"):
    """A (M x K) times B (K x N) as a two-tensor network: one GEMM vertex of
    profile class `cls`."""
    (M, K), N = A.shape, B.shape[1]
    p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, [A, B], [0, 0], 1, [(0, 1)], [0, 2], flags, lib.TN_C64)
    lib.tn_profile_enable(ctx.handle, True)
    lib.tn_profile_read(ctx.handle)
    out, _ = lib.tn_contract(p, None, (M, N), lib.TN_C64)
    stats = lib.tn_profile_read(ctx.handle)
    lib.tn_profile_enable(ctx.handle, False)
    ctx.free_plan(p)
    assert stats[cls]["launches"] == 1, stats
    return out


def bound(A, B):
    K = A.shape[1]
    return 8 * np.sqrt(12 * -(-K // 16) + 8) * 2.0 ** -23 * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64))


def entries(rng, shape, kind):
    x = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    if kind == "positive":
        x = (rng.random(shape) + 1j * rng.random(shape)).astype(np.complex64)
    elif kind == "range":  # sizes over 2^40, rows apart by as much again
        x *= np.exp2(-40 * rng.random(shape)).astype(np.float32)
        x *= np.exp2(-40 * rng.random((shape[0], 1))).astype(np.float32)
    return x


# tiles are 128 x 128, 64 x 256 (M <= 64) and 256 x 64 (N <= 64); k chunks of 16
SHAPES = [(128, 128, 144), (129, 127, 144), (513, 1025, 32), (2048, 515, 16), (65, 64, 528), (64, 257, 160),
          (33, 500, 144), (300, 64, 144), (511, 17, 256), (97, 130, 4096), (40, 40, 16384)]
# in place: 64 x 64 and 32 x 32 tiles, rounds of 16 k
SMALL = [(128, 128, 48), (65, 64, 64), (33, 127, 64), (1024, 1023, 8), (2049, 511, 15), (200, 300, 7), (500, 133, 1),
         (23, 5003, 3), (129, 130, 16), (1000, 40, 17)]


@pytest.mark.parametrize("kind", ["normal", "positive", "range"])
@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("flags", [0, lib.TN_FORM_3M])
def test_gemm_vertex(ctx, M, N, K, kind, flags):
    rng = np.random.default_rng([M, N, K])
    A, B = entries(rng, (M, K), kind), entries(rng, (N, K), kind).T.copy()
    got = run_pair(ctx, A, B, flags)
    ref = A.astype(np.complex128) @ B.astype(np.complex128)
    over = np.abs(got - ref) / bound(A, B)
    assert over.max() <= 1.0, over.max()


@pytest.mark.parametrize("M,N,K", SMALL)
@pytest.mark.parametrize("flags", [0, lib.TN_FORM_3M, lib.TN_PREC_BF16X3, lib.TN_PREC_BF16X3 | lib.TN_FORM_3M])
def test_small_vertex(ctx, M, N, K, flags):
    """FP32: a sum of 4 K products, each addition rounded once.  BF16x3: the
    dropped product of the low terms, at most 2^-16 of |A| |B| (3M: of the sums
    of parts, at most twice as large and twice as many)."""
    rng = np.random.default_rng([M, N, K])
    A, B = entries(rng, (M, K), "range" if K % 2 else "normal"), entries(rng, (N, K), "normal").T.copy()
    got = run_pair(ctx, A, B, flags, "gemm_small")
    ref = A.astype(np.complex128) @ B.astype(np.complex128)
    tol = 8 * np.sqrt(4 * K + 4) * 2.0 ** -23
    if flags & lib.TN_PREC_BF16X3:
        # 3M's sums mix the parts of a row of very different entries
        tol += 2.0 ** -12
    over = np.abs(got - ref) / (tol * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)))
    assert over.max() <= 1.0, over.max()


@pytest.mark.parametrize("M,N,K", [(203, 330, 405), (65, 1000, 33), (67, 64, 1001)])
def test_small_vertex_long_k(ctx, M, N, K):
    """FP32: a long k that is no multiple of 16."""
    rng = np.random.default_rng([M, N, K])
    A, B = entries(rng, (M, K), "normal"), entries(rng, (K, N), "normal")
    got = run_pair(ctx, A, B, 0, "gemm_small")
    size = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    assert (np.abs(got - A.astype(np.complex128) @ B) <= 8 * np.sqrt(4 * K + 4) * 2.0 ** -23 * size).all()


@pytest.mark.parametrize("flags", [0, lib.TN_PREC_BF16X3])
def test_small_vertex_legs(ctx, flags):
    """Contracted and free legs in any order, dimensions not powers of two."""
    rng = np.random.default_rng(11)
    dims = {0: 5, 1: 3, 2: 7, 3: 6, 4: 9, 5: 2, 6: 11, 7: 4}
    la, lb, out = [3, 0, 5, 1, 4], [1, 6, 2, 5, 7], [2, 4, 0, 7, 3, 6]
    A = entries(rng, tuple(dims[x] for x in la), "normal")
    B = entries(rng, tuple(dims[x] for x in lb), "normal")
    p = ctx.plan_load([la, lb], dims, [A, B], [0, 0], 1, [(0, 1)], out, flags, lib.TN_C64)
    got, _ = lib.tn_contract(p, None, tuple(dims[x] for x in out), lib.TN_C64)
    ctx.free_plan(p)
    e = "".join("abcdefgh"[x] for x in la) + "," + "".join("abcdefgh"[x] for x in lb) + "->" + \
        "".join("abcdefgh"[x] for x in out)
    ref = np.einsum(e, A.astype(np.complex128), B.astype(np.complex128))
    size = np.einsum(e, np.abs(A).astype(np.float64), np.abs(B).astype(np.float64))
    assert (np.abs(got - ref) <= (2.0 ** -12 if flags else 8 * 5 * 2.0 ** -23) * size).all()


def test_infinity(ctx):
    """An infinite entry reaches every result of its row, and no other row
    turns infinite or undefined."""
    rng = np.random.default_rng(5)
    A, B = entries(rng, (130, 144), "normal"), entries(rng, (144, 140), "normal")
    A[77, 5] = np.inf
    got = run_pair(ctx, A, B, 0)
    assert not np.isfinite(got[77]).any()
    assert np.isfinite(np.delete(got, 77, axis=0)).all()
