"""TN_FLAG_CONCURRENT on partitions that each close to a number: their inner
products run on streams of their own, each adding up partial sums of many
blocks, which lie in the partition's own region.  The results have the bits of
the serial order, and complex128's value within FP32 rounding of the entries
(the sums are FP64)."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("parts,log2n", [(2, 12), (2, 20), (5, 16)])
def test_closed_partitions(parts, log2n):
    n = 1 << log2n
    rng = np.random.default_rng([parts, log2n])
    legs, tensors, part = [], [], []
    for k in range(parts):
        for _ in range(2):
            legs.append([k])
            tensors.append((rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64) * 2.0 ** (3 * k))
            part.append(k)
    nv = 2 * parts
    tree = [(2 * k, 2 * k + 1) for k in range(parts)]
    top = nv
    for k in range(1, parts):
        tree.append((top, nv + k))
        top = nv + len(tree) - 1
    ctx = lib.Context(1 << 30)
    p = ctx.plan_load(legs, {k: n for k in range(parts)}, tensors, part, parts, tree, None, 0, lib.TN_C64)
    serial, _ = lib.tn_contract(p)
    ref = np.prod([np.sum(tensors[2 * k].astype(np.complex128) * tensors[2 * k + 1]) for k in range(parts)])
    size = np.prod([np.sum(np.abs(tensors[2 * k].astype(np.complex128) * tensors[2 * k + 1])) for k in range(parts)])
    # each number is rounded to complex64 once, their products once each
    assert abs(complex(serial.reshape(-1)[0]) - ref) <= 2 * parts * 2.0 ** -23 * abs(ref) + 1e-13 * size
    for _ in range(20):
        got, _ = lib.tn_contract(p, flags=lib.TN_FLAG_CONCURRENT)
        assert np.array_equal(got, serial)
    ctx.free_plan(p)
    ctx.close()
