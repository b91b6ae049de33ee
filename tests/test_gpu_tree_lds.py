"""Per-query subtrees that nearly fill a CU's LDS: a vector taken through a chain
of shared matrices that the call computes first (each an outer product, built
just before its turn), the last d columns wide.  The batch kernel runs them as
long as four queries fit beside the matrices, also where the level kernel, which
keeps step descriptors there too (8 KB), has no room for one.

Bound: five sums of 64 complex products and the matrices' own roundings, at most
8 sqrt(5 * 2 * 64) 2^-24 of the sums of magnitudes."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q", [1, 2, 300])
@pytest.mark.parametrize("d", [40, 46, 50, 52, 64])
def test_chain(d, Q):
    rng = np.random.default_rng([d, Q])

    def entries(*shape):
        return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)

    # leaves: the vector, then per matrix two vectors and k numbers, at last w
    v, dim = entries(Q, 64), [64] * 5 + [d]
    legs, leaves = [[0]], [v[0]]
    groups = []
    for k in range(5):
        a, b, nums = len(legs), len(legs) + 1, list(range(len(legs) + 2, len(legs) + 2 + k))
        legs += [[k], [k + 1]] + [[]] * k
        leaves += [entries(dim[k]) / 8, entries(dim[k + 1])] + [entries() for _ in nums]
        groups.append((a, b, nums))
    w = len(legs)
    legs.append([5])
    leaves.append(entries(d))
    tree, nv = [], len(legs)

    def contract(x, y):
        tree.append((x, y))
        return nv + len(tree) - 1

    mats = []
    for a, b, nums in groups:
        for s in nums:
            a = contract(a, s)
        mats.append(contract(a, b))
    r = 0
    for m in mats:
        r = contract(r, m)
    contract(r, w)
    with lib.Context(64 << 20) as ctx:
        p = ctx.plan_load(legs, {k: n for k, n in enumerate(dim)}, leaves, [0] * nv, 1, tree, None, 0, lib.TN_C64)
        lib.tn_profile_enable(ctx.handle, True)
        lib.tn_profile_read(ctx.handle)
        got = lib.tn_contract_strided(p, Q, [(0, v, 512, lib.TN_C64)])[0].reshape(-1)
        n = {k: x["launches"] for k, x in lib.tn_profile_read(ctx.handle).items() if x["launches"]}
    ref, size = v.astype(np.complex128), np.abs(v).astype(np.float64)
    for a, b, nums in groups:
        m = np.prod([leaves[s].astype(np.complex128) for s in nums]) * np.outer(leaves[a].astype(np.complex128), leaves[b])
        ref, size = ref @ m, size @ np.abs(m)
    ref, size = ref @ leaves[w], size @ np.abs(leaves[w])
    assert (np.abs(got - ref) <= 8 * np.sqrt(5 * 2 * 64) * 2.0 ** -24 * size).all()
    # four queries' LDS: 158 400 bytes at d = 40, 163 520 of 163 840 at 50
    assert ("stream" not in n) == (d <= 50), n
