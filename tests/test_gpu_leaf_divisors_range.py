"""Small leaves of entries so far apart that dividing by the largest would take
the smallest out of FP32's normal range: a result that depends on the small
entry alone is as accurate as the entry's own rounding (2^-24, and as much
again for the result)."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("big,small", [(1.1e20, 1.3e-25), (3.3, 2.0e-38), (1e25 / 3, 1e-20 / 3), (0.7, 2.0e-38), (1e29, 1.7e-9)])
@pytest.mark.parametrize("part", [1.0, 1j])
def test_small_entry(big, small, part):
    a = np.array([big, small * part, big / 7], dtype=np.complex128)
    b = np.array([0.0, 1.0, 0.0], dtype=np.complex128)
    with lib.Context(64 << 20) as ctx:
        p = ctx.plan_load([[0], [0]], {0: 3}, [a, b], [0, 0], 1, [(0, 1)])
        single = lib.tn_contract(p)[0]
        m, l2 = lib.tn_contract(p, flags=lib.TN_FLAG_KEEP_SCALE)
        (batch,), _, _ = lib.tn_contract_batch(ctx.handle, [(p, {1: b})], [()])
        ctx.free_plan(p)
    for got in (single, m * 2.0 ** l2, batch):
        assert abs(complex(np.asarray(got).reshape(-1)[0]) - small * part) <= 2.0 ** -23 * small
