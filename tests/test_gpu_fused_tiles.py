"""GEMMs that write their parent's operand planes, over many queries, on every
tile that a launch may choose (32 x 128 and 128 x 32 for results of up to 32 rows
or columns, 64 x 64, 64 x 256, 256 x 64, 128 x 128): the bits of the same plan with
the permutation."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


# bits of the rows of P (a), of its columns (b1 and the four or five of b2 that the
# parent contracts), and queries
@pytest.mark.parametrize("a,b1,b2,Q", [(5, 6, 4, 48), (5, 5, 5, 200), (9, 1, 4, 60), (6, 6, 4, 30), (9, 2, 4, 30),
                                       (7, 3, 4, 3), (7, 3, 5, 70)])
@pytest.mark.parametrize("flags", [0, lib.TN_FORM_3M, lib.TN_PREC_BF16X3, lib.TN_PREC_BF16X3 | lib.TN_FORM_3M])
@pytest.mark.parametrize("side", "AB")
def test_bits(a, b1, b2, Q, flags, side, monkeypatch):
    s, kb = [10, 11, 12, 13], list(range(20, 20 + b2))
    dims = {0: 1 << a, 1: 1 << b1, 2: 16, **{x: 2 for x in s + kb}}
    legs, out = [[0] + s, s + [1] + kb, [2] + kb], [0, 1, 2]
    rng = np.random.default_rng([a, b1, b2, Q])

    def entries(*shape):
        return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)

    ts = [entries(*[dims[x] for x in l]) for l in legs]
    xs = entries(Q, *ts[0].shape)
    tree = [(0, 1), (3, 2)] if side == "A" else [(0, 1), (2, 3)]
    shape = tuple(dims[x] for x in out)
    got, perms = [], []
    with lib.Context(2 << 30) as ctx:
        for fuse in ("0", "1"):
            monkeypatch.setenv("TN_GEMM_FUSE", fuse)
            p = lib.tn_plan_load(ctx.handle, legs, dims, ts, [0, 0, 0], 1, tree, out, flags, lib.TN_C64)
            perms.append(lib.tn_plan_costs_get(p)["num_permutations"])
            got.append(lib.tn_contract_strided(p, Q, [(0, xs, xs[0].nbytes, lib.TN_C64)], shape, lib.TN_C64)[0])
            lib.tn_plan_free(p)
    assert perms[1] == perms[0] - 1
    assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
    ref = np.einsum("qas,sbk,ck->qabc", xs.reshape(Q, -1, 16).astype(np.complex128), ts[1].reshape(16, -1, 1 << b2),
                    ts[2].reshape(16, -1), optimize=True)
    tol = 2e-6 if not flags & lib.TN_PREC_BF16X3 else 1e-4
    assert np.abs(got[1].reshape(ref.shape) - ref).max() <= tol * np.abs(ref).max()
