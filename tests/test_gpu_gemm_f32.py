"""The FP32 GEMM on k-tiled planes (three bfloat16 terms per value, six
products): one vertex against complex128, at tile edges, short and long k,
split k, every tile shape, entries of very different size, and an operand
that holds an infinity.

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


def run_pair(ctx, A, B, flags):
    """A (M x K) times B (K x N) as a two-tensor network: one GEMM vertex."""
    (M, K), N = A.shape, B.shape[1]
    p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, [A, B], [0, 0], 1, [(0, 1)], [0, 2], flags, lib.TN_C64)
    lib.tn_profile_enable(ctx.handle, True)
    lib.tn_profile_read(ctx.handle)
    out, _ = lib.tn_contract(p, None, (M, N), lib.TN_C64)
    stats = lib.tn_profile_read(ctx.handle)
    lib.tn_profile_enable(ctx.handle, False)
    ctx.free_plan(p)
    assert stats["gemm"]["launches"] == 1, stats
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
SHAPES = [(128, 128, 48), (129, 127, 64), (257, 383, 16), (65, 64, 80), (64, 257, 96), (33, 500, 144), (300, 64, 112),
          (511, 17, 256), (97, 130, 4096), (40, 40, 16384)]


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


def test_infinity(ctx):
    """An infinite entry reaches every result of its row, and no other row
    turns infinite or undefined."""
    rng = np.random.default_rng(5)
    A, B = entries(rng, (130, 64), "normal"), entries(rng, (64, 140), "normal")
    A[77, 5] = np.inf
    got = run_pair(ctx, A, B, 0)
    assert not np.isfinite(got[77]).any()
    assert np.isfinite(np.delete(got, 77, axis=0)).all()
