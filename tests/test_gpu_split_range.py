"""FP32 GEMM vertices whose operands hold entries that three bfloat16 terms do
not: smaller than 2^-110, larger than 2^60, infinite, not numbers; as leaves
(whose planes hold them as they are) and as the result of a GEMM that writes
its parent's planes.  The result is as accurate as for any other entries, and
infinities and NaNs reach their row's results as FP32 arithmetic has them.

Bound per GEMM: 8 sqrt(12 ceil(K / 16) + 8) 2^-23 of |A| |B|, as for one vertex
of ordinary entries, and one unit of FP32's smallest subnormal per term."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu
TINY = 2.0 ** -149


@pytest.fixture(scope="module")
def ctx():
    c = lib.Context(2 << 30)
    yield c
    c.close()


def entries(rng, shape):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)


def pair(ctx, A, B):
    (M, K), N = A.shape, B.shape[1]
    p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, [A, B], [0, 0], 1, [(0, 1)], [0, 2], 0, lib.TN_C64)
    out, _ = lib.tn_contract(p, None, (M, N), lib.TN_C64)
    ctx.free_plan(p)
    return out


def rel(K):
    return 8 * np.sqrt(12 * -(-K // 16) + 8) * 2.0 ** -23


# on planes (128 x 128 tiles, 64 x 64, split k) and in place
SHAPES = [(1030, 144, 1100), (130, 144, 140), (65, 528, 33), (40, 16384, 40), (64, 48, 64), (67, 1001, 64)]


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("a,b", [(-124, 0), (0, -124), (-60, -60), (-109, 0), (70, -100), (100, -3)])
def test_sizes(ctx, M, K, N, a, b):
    rng = np.random.default_rng([M, N, K])
    A, B = entries(rng, (M, K)) * np.float32(2.0 ** a), entries(rng, (K, N)) * np.float32(2.0 ** b)
    got = pair(ctx, A, B)
    ref = A.astype(np.complex128) @ B.astype(np.complex128)
    size = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    assert (np.abs(got - ref) <= rel(K) * size + 4 * K * TINY).all()


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_one_small_row(ctx, M, K, N):
    """One row of tiny entries among ordinary ones."""
    rng = np.random.default_rng([M, N, K, 1])
    A, B = entries(rng, (M, K)), entries(rng, (K, N))
    A[M // 3] *= np.float32(2.0 ** -124)
    got = pair(ctx, A, B)
    ref = A.astype(np.complex128) @ B.astype(np.complex128)
    size = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    assert (np.abs(got - ref) <= rel(K) * size + 4 * K * TINY).all()


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("side", "AB")
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_not_finite(ctx, M, K, N, side, value):
    """inf b is an infinity with b's sign, in both parts; the largest finite
    entries do not turn infinite."""
    rng = np.random.default_rng([M, N, K, 2])
    A, B = entries(rng, (M, K)), entries(rng, (K, N))
    m, k, n = M // 2, K // 3, N // 2
    if value == 3.4e38:
        A *= np.float32(2.0 ** -20)
        B *= np.float32(2.0 ** -20)
    (A if side == "A" else B)[(m, k) if side == "A" else (k, n)] = value
    got = pair(ctx, A, B)
    hit = got[m] if side == "A" else got[:, n]
    other = B[k] if side == "A" else A[:, k]
    if np.isnan(value):
        assert np.isnan(hit.real).all() and np.isnan(hit.imag).all()
    elif np.isinf(value):
        s = np.sign(value)
        assert np.array_equal(hit.real, s * np.sign(other.real) * np.inf)
        assert np.array_equal(hit.imag, s * np.sign(other.imag) * np.inf)
    else:
        assert (np.abs(hit - value * other.astype(np.complex128)) <= 2.0 ** -20 * value * np.abs(other)).all()
    rest = np.delete(got, m, axis=0) if side == "A" else np.delete(got, n, axis=1)
    assert np.isfinite(rest).all()


@pytest.mark.parametrize("fuse", ["0", "1"])
@pytest.mark.parametrize("side", "AB")
@pytest.mark.parametrize("form", [0, lib.TN_FORM_3M])
def test_fused_operand(ctx, fuse, side, form, monkeypatch):
    """X(a, s) Y(s, b1, b2) -> P(a, b1, b2), both operands' entries of 2^-62 and
    some rows of X of 1: P's other rows are 2^-124.  P and Z(c, b2) -> root."""
    monkeypatch.setenv("TN_GEMM_FUSE", fuse)
    s, b2 = [10, 11, 12, 13], [20, 21, 22, 23, 24]
    dims = {0: 64, 1: 64, 2: 16, **{x: 2 for x in s + b2}}
    legs, out = [[0] + s, s + [1] + b2, [2] + b2], [0, 1, 2]
    rng = np.random.default_rng(3)
    X, Y, Z = (entries(rng, tuple(dims[x] for x in l)) for l in legs)
    X *= np.float32(2.0 ** -62)
    X[::7] *= np.float32(2.0 ** 62)
    Y *= np.float32(2.0 ** -62)
    tree = [(0, 1), (3, 2)] if side == "A" else [(0, 1), (2, 3)]
    p = lib.tn_plan_load(ctx.handle, legs, dims, [X, Y, Z], [0, 0, 0], 1, tree, out, form, lib.TN_C64)
    assert lib.tn_plan_costs_get(p)["num_permutations"] == 4 - int(fuse)
    got, _ = lib.tn_contract(p, None, (64, 64, 16), lib.TN_C64)
    lib.tn_plan_free(p)
    x, y, z = X.reshape(64, 16), Y.reshape(16, 64, 32), Z.reshape(16, 32)
    e = "as,sbt,ct->abc"
    ref = np.einsum(e, x.astype(np.complex128), y.astype(np.complex128), z.astype(np.complex128), optimize=True)
    size = np.einsum(e, *(np.abs(v).astype(np.float64) for v in (x, y, z)), optimize=True)
    assert (np.abs(got - ref) <= (rel(16) + rel(32)) * size + 64 * TINY).all()


@pytest.mark.parametrize("M,K,N", [(130, 144, 140), (64, 528, 300), (64, 48, 64), (65, 100, 33)])
@pytest.mark.parametrize("form", [0, lib.TN_FORM_3M])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_not_finite_bf16x3(ctx, M, K, N, form, value):
    """BF16x3 (on planes and in place): the row's results are not finite, all
    others are."""
    rng = np.random.default_rng([M, N, K, 3])
    A, B = entries(rng, (M, K)), entries(rng, (K, N))
    A[M // 2, K // 3] = value
    p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, [A, B], [0, 0], 1, [(0, 1)], [0, 2],
                      lib.TN_PREC_BF16X3 | form, lib.TN_C64)
    got, _ = lib.tn_contract(p, None, (M, N), lib.TN_C64)
    ctx.free_plan(p)
    assert not np.isfinite(got[M // 2]).any()
    assert np.isfinite(np.delete(got, M // 2, axis=0)).all()
