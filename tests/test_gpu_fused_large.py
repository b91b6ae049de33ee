"""A GEMM that writes its parent's operand planes, 512 MB of them (more than the
last level cache holds: they are stored past it), against the same plan with the
permutation: the same bits."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [lib.TN_PREC_FP32, lib.TN_PREC_BF16X3, lib.TN_PREC_BF16X3 | lib.TN_FORM_3M])
@pytest.mark.parametrize("side", ["A", "B"])
def test_bits(flags, side, monkeypatch):
    # X(a, s) Y(s, b1, b2) -> P(a, b1, b2), 2^26 entries; P and Z(c, b2) -> root
    s, b2 = [10, 11, 12, 13], list(range(20, 28))
    dims = {0: 2 ** 13, 1: 2 ** 5, 2: 2 ** 4, **{x: 2 for x in s + b2}}
    legs, out = [[0] + s, s + [1] + b2, [2] + b2], [0, 1, 2]
    rng = np.random.default_rng(3)
    ts = [(rng.standard_normal(sh) + 1j * rng.standard_normal(sh)).astype(np.complex64)
          for sh in (tuple(dims[x] for x in l) for l in legs)]
    tree = [(0, 1), (3, 2)] if side == "A" else [(0, 1), (2, 3)]
    shape = tuple(dims[x] for x in out)
    got, perms = [], []
    with lib.Context(6 << 30) as ctx:
        for fuse in ("0", "1"):
            monkeypatch.setenv("TN_GEMM_FUSE", fuse)
            p = lib.tn_plan_load(ctx.handle, legs, dims, ts, [0, 0, 0], 1, tree, out, flags)
            got.append(lib.tn_contract(p, None, shape, lib.TN_C64)[0])
            perms.append(lib.tn_plan_costs_get(p)["num_permutations"])
            lib.tn_plan_free(p)
    assert perms[1] == perms[0] - 1
    assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
