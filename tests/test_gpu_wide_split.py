"""Skinny products take more k chunks where the call's memory has room for the
partial sums, and the plan's own chunks where it has not: the same calls work in
the same arenas, with results that differ by FP32 rounding only.

Bound: a sum of K products in FP32, 8 sqrt(12 K / 16 + 8) 2^-23 of |A| |B|."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu
M, N, K = 24, 320, 4096


def test_both_ways_and_every_arena():
    rng = np.random.default_rng(1)
    A = (rng.standard_normal((M, K, 2))).astype(np.float32).view(np.complex64)[..., 0]
    B = (rng.standard_normal((K, N, 2))).astype(np.float32).view(np.complex64)[..., 0]
    ref = A.astype(np.complex128) @ B.astype(np.complex128)
    tol = 8 * np.sqrt(12 * K / 16 + 8) * 2.0 ** -23 * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64))
    seen = []
    # the leaves, the two permuted operands and the result take 22.6 MB; the
    # partial sums of 64 chunks 3.9 MB more
    for kib in range(20000, 32000, 500):
        with lib.Context(kib << 10) as ctx:
            try:
                p = ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: K, 2: N}, [A, B], [0, 0], 1, [(0, 1)], [0, 2], 0,
                                  lib.TN_C64)
                got, _ = lib.tn_contract(p, None, (M, N), lib.TN_C64)
            except lib.TnError as e:
                assert e.status == lib.TN_E_NOMEM and not seen, kib
                continue
            assert (np.abs(got - ref) <= tol).all()
            seen.append(got.tobytes())
    # the plan's chunks first, then the wide split; two results in all
    assert len(set(seen)) == 2 and seen == sorted(seen, key=lambda s: s == seen[-1])


@pytest.mark.parametrize("queries", [1, 3, 40])
def test_queries(queries):
    """The chunk count follows the number of queries; every query is right."""
    import torch
    m, n, k = 8, 130, 528
    g = torch.Generator(device="cuda").manual_seed(queries)
    A = torch.randn((queries, m, k), generator=g, device="cuda", dtype=torch.complex64)
    B = torch.randn((queries, k, n), generator=g, device="cuda", dtype=torch.complex64)
    for flags in (0, lib.TN_PREC_BF16X3, lib.TN_PREC_BF16X3 | lib.TN_FORM_3M):
        with lib.Context(1 << 30) as ctx:
            z = [np.zeros((m, k), np.complex64), np.zeros((k, n), np.complex64)]
            p = ctx.plan_load([[0, 1], [1, 2]], {0: m, 1: k, 2: n}, z, [0, 0], 1, [(0, 1)], [0, 2], flags, lib.TN_C64)
            got, _ = lib.tn_contract_strided(p, queries, [(0, A.data_ptr(), m * k * 8, lib.TN_C64_DEVICE),
                                                          (1, B.data_ptr(), k * n * 8, lib.TN_C64_DEVICE)],
                                             (m, n), lib.TN_C64, scales=False)
        a, b = A.cpu().numpy().astype(np.complex128), B.cpu().numpy().astype(np.complex128)
        for q in range(queries):
            size = np.abs(a[q]) @ np.abs(b[q])
            tol = 8 * np.sqrt(12 * k / 16 + 8) * 2.0 ** -23 + (2.0 ** -12 if flags else 0)
            assert (np.abs(got[q] - a[q] @ b[q]) <= tol * size).all(), (flags, q)
