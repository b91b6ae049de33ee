"""Leaves far from one in the subtree kernels: two leaves of 2^-40 make an
intermediate of 2^-80, which fits FP32 as it is, and the product of two such
intermediates fits it only once their scale records are applied, to the operands
before the products.  Every leaf is a power of two away from one of order one,
so the result, read as mantissa and scale, is the unscaled network's.

Bounds: an entry of the chain is a sum of products of eight entries, three
levels of four roundings each (complex: times sqrt(2)) and eight leaf
roundings, below 32 * 2^-24 of the sum of magnitudes; the long chain's as in
the tests of subtrees that fill the LDS."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import output_tensor_ids, random_bitstrings
from paper_2507_20667_amd.planner.workloads import brickwork20

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [-40, 40])
@pytest.mark.parametrize("how", ["complex64 leaves", "bf16x3 leaves", "host overrides", "device overrides",
                                 "concurrent", "batch", "strided"])
def test_chain_of_pairs(shift, how):
    rng = np.random.default_rng(8)
    T = [rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2)) for _ in range(8)]
    S = [t * 2.0 ** shift for t in T]
    dtype = lib.TN_C64 if how in ("complex64 leaves", "concurrent", "batch") else lib.TN_C128
    prec = lib.TN_PREC_BF16X3 if how == "bf16x3 leaves" else 0
    flags = lib.TN_FLAG_KEEP_SCALE | (lib.TN_FLAG_CONCURRENT if how == "concurrent" else 0)
    over = how.endswith("overrides") or how == "strided"
    with lib.Context(64 << 20) as ctx:
        p = ctx.plan_load([[i, i + 1] for i in range(8)], {i: 2 for i in range(9)}, T if over else S, [0] * 4 + [1] * 4, 2,
                          [(0, 1), (2, 3), (8, 9), (4, 5), (6, 7), (11, 12), (10, 13)], [0, 8], prec, dtype)
        if how == "device overrides":
            dev = torch.tensor(np.array(S), dtype=torch.complex64, device="cuda")
            arr = (lib.tn_leaf * 8)(*[lib.tn_leaf(i, dev.data_ptr() + 32 * i, lib.TN_C64_DEVICE) for i in range(8)])
            torch.cuda.synchronize()
            m, l2 = np.zeros((2, 2), np.complex128), ctypes.c_double(0.0)
            rc = lib.load().tn_contract(p, 8, ctypes.cast(arr, ctypes.c_void_p), m.ctypes.data_as(ctypes.c_void_p),
                                        lib.TN_C128, ctypes.byref(l2), flags)
            assert rc == lib.TN_OK, lib.tn_last_error()
            l2 = l2.value
        elif how == "batch":
            out, l2s, _ = lib.tn_contract_batch(ctx.handle, [(p, {0: S[0] * f}) for f in (2, 1, -1)], [(2, 2)] * 3, flags=flags)
            m, l2 = out[1], l2s[1]
        elif how == "strided":
            out, l2s = lib.tn_contract_strided(p, 300, [(i, np.stack([t] * 300).astype(np.complex64), 32, lib.TN_C64)
                                                        for i, t in enumerate(S)], (2, 2), flags=flags)
            m, l2 = out[299], l2s[299]
        else:
            m, l2 = lib.tn_contract(p, dict(enumerate(S)) if over else None, (2, 2), flags=flags)
    got = m * 2.0 ** (float(l2) - 8 * shift)
    ref, size = T[0], np.abs(T[0])
    for t in T[1:]:
        ref, size = ref @ t, size @ np.abs(t)
    assert (np.abs(got - ref) <= 32 * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("Q", [1, 300])
@pytest.mark.parametrize("shift", [-50, 50])
def test_on_the_batch_kernel(shift, Q):
    # a chain of five shared matrices, each an outer product times k numbers,
    # whose queries fit beside them only in the batch kernel
    rng = np.random.default_rng(50)

    def entries(*shape):
        return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)

    dim, legs, leaves, groups = [64] * 5 + [50], [[0]], [entries(64)], []
    for k in range(5):
        groups.append((len(legs), len(legs) + 1, list(range(len(legs) + 2, len(legs) + 2 + k))))
        legs += [[k], [k + 1]] + [[]] * k
        leaves += [entries(dim[k]) / 8, entries(dim[k + 1])] + [entries() for _ in range(k)]
    w, nv, tree = len(legs), len(legs) + 1, []
    legs.append([5])
    leaves.append(entries(50))

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
    S = [np.asarray(t * np.float32(2.0 ** shift), np.complex64) for t in leaves]
    with lib.Context(64 << 20) as ctx:
        p = ctx.plan_load(legs, {k: n for k, n in enumerate(dim)}, S, [0] * nv, 1, tree, None, 0, lib.TN_C64)
        lib.tn_profile_enable(ctx.handle, True)
        lib.tn_profile_read(ctx.handle)
        if Q == 1:
            m, l2 = lib.tn_contract(p, {0: S[0]}, (), flags=lib.TN_FLAG_KEEP_SCALE)
        else:
            out, l2s = lib.tn_contract_strided(p, Q, [(0, np.stack([S[0]] * Q), 512, lib.TN_C64)],
                                               flags=lib.TN_FLAG_KEEP_SCALE)
            m, l2 = out[Q - 1], l2s[Q - 1]
        n = {k: x["launches"] for k, x in lib.tn_profile_read(ctx.handle).items() if x["launches"]}
    assert "stream" not in n, n
    ref, size = leaves[0].astype(np.complex128), np.abs(leaves[0]).astype(np.float64)
    for a, b, nums in groups:
        mat = np.prod([leaves[s].astype(np.complex128) for s in nums]) * np.outer(leaves[a].astype(np.complex128), leaves[b])
        ref, size = ref @ mat, size @ np.abs(mat)
    ref, size = ref @ leaves[w], size @ np.abs(leaves[w])
    got = complex(m.item()) * 2.0 ** (float(l2) - nv * shift)
    assert abs(got - ref) <= 8 * np.sqrt(5 * 2 * 64) * 2.0 ** -24 * size


@pytest.mark.parametrize("shift", [-40, 40])
@pytest.mark.parametrize("queries", [1, 3, 300])
def test_brickwork(queries, shift):
    # the 20-qubit brickwork with every gate tensor scaled: gate chains, the
    # fused pair and packed gate steps (300), the level kernel (1)
    w = brickwork20()
    net, plan = w.net, w.plan
    ids = output_tensor_ids(net)
    xs = random_bitstrings(w.circ.n, queries, 7)
    vecs = np.zeros((len(ids), queries, 2), np.complex64)
    for q, x in enumerate(xs):
        for k in range(len(ids)):
            vecs[k, q, (x >> k) & 1] = 1.0
    gates = [i for i, l in enumerate(net.legs) if len(l) >= 2]
    got = {}
    with lib.Context(1 << 30) as ctx:
        for s in (0, shift):
            tensors = [np.asarray(t, np.complex64) * np.float32(2.0 ** (s if i in gates else 0))
                       for i, t in enumerate(net.tensors)]
            p = ctx.plan_load(net.legs, net.dims, tensors, plan.partition_of, w.num_partitions, plan.tree, None, 0, lib.TN_C64)
            if queries == 1:
                m, l2 = lib.tn_contract(p, {t: vecs[k, 0] for k, t in enumerate(ids)}, flags=lib.TN_FLAG_KEEP_SCALE)
                m, l2 = np.array([m.item()]), np.array([l2])
            else:
                m, l2 = lib.tn_contract_strided(p, queries, [(t, vecs[k], 16, lib.TN_C64) for k, t in enumerate(ids)],
                                                flags=lib.TN_FLAG_KEEP_SCALE)
            got[s] = m * 2.0 ** (l2 - s * len(gates))
    # powers of two: only entries at the end of FP32's range may round elsewhere
    assert (np.abs(got[shift] - got[0]) <= 2.0 ** -30 * 2.0 ** (-w.circ.n / 2)).all()
