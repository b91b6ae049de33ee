"""Open results larger than the staging they are converted through (64 MB): every
piece, query, type and form, exact (outer products of small whole numbers)."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


# entries of a result: 5 000 000 (80 MB as complex128, 40 as complex64), and
# 4194304 and one row more (64 MB as complex128)
@pytest.mark.parametrize("rows,cols,Q", [(2000, 2500, 1), (2000, 2500, 3), (2048, 2048, 1), (2049, 2048, 2), (4099, 4001, 1)])
def test_pieces(rows, cols, Q):
    rng = np.random.default_rng(rows)
    a = rng.integers(-30, 31, (Q, rows)) + 1j * rng.integers(-30, 31, (Q, rows))
    b = rng.integers(-30, 31, cols) + 1j * rng.integers(-30, 31, cols)
    want = [np.outer(a[q], b) for q in range(Q)]
    with lib.Context(2 << 30) as ctx:
        for out in ([0, 1], [1, 0]):
            p = ctx.plan_load([[0], [1]], {0: rows, 1: cols}, [a[0], b], [0, 0], 1, [(0, 1)], out)
            shape = (rows, cols) if out == [0, 1] else (cols, rows)
            for flags in (0, lib.TN_FLAG_KEEP_SCALE, lib.TN_FLAG_GRAPH):
                for dt in (lib.TN_C128, lib.TN_C64):
                    got, l2, _ = lib.tn_contract_batch(ctx.handle, [(p, {0: x}) for x in a], [shape] * Q, dt, flags)
                    for q in range(Q):
                        w = want[q] if out == [0, 1] else want[q].T
                        assert np.array_equal(got[q] * got[q].dtype.type(2.0 ** l2[q]), w), (out, flags, dt, q)
            # a shared root: one result for every query
            got, _, _ = lib.tn_contract_batch(ctx.handle, [(p, None)] * 2, [shape] * 2)
            assert np.array_equal(got[0], got[1]) and np.array_equal(got[1], want[0] if out == [0, 1] else want[0].T)
            ctx.free_plan(p)


def test_staging_memory():
    """A complex128 result of 1 GB takes host memory for the caller's array and
    64 MB of staging."""
    n = 1 << 13
    a = np.ones(n, np.complex64)

    def mapped():
        with open("/proc/self/status") as f:
            return next(int(l.split()[1]) for l in f if l.startswith("VmSize")) << 10

    with lib.Context(2 << 30) as ctx:
        small = ctx.plan_load([[0], [1]], {0: 64, 1: n}, [a[:64], a], [0, 0], 1, [(0, 1)], [0, 1], 0, lib.TN_C64)
        lib.tn_contract(small, None, (64, n))
        p = ctx.plan_load([[0], [1]], {0: n, 1: n}, [a, a], [0, 0], 1, [(0, 1)], [0, 1], 0, lib.TN_C64)
        before = mapped()
        out, _ = lib.tn_contract(p, None, (n, n))
        grown = mapped() - before
    assert (out == 1).all()
    assert grown <= out.nbytes + (200 << 20), grown
