"""tn_contract on plans with small vertices: subtree kernels when the arena has
room for their programs, one launch per vertex otherwise, and programs that
give way to other calls' memory.  Amplitudes against the state vector
(|a - a_ref| / max(|a_ref|, 2^(-n/2)) <= 1e-5, the FP32 bound)."""
import numpy as np
import pytest

import oracle
from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides, output_tensor_ids, random_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu
N = 12


@pytest.fixture(scope="module")
def case():
    circ = random_circuit(N, 12, 3)
    net = amplitude_network(circ, 0)
    return circ, net, plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 3), 3), \
        oracle.statevector(circ)


def check(got, psi, x):
    err = abs(complex(np.asarray(got).reshape(-1)[0]) - psi[x]) / max(abs(psi[x]), 2.0 ** (-N / 2))
    assert err <= 1e-5, (x, err)


def classes(ctx, p, ovr, flags=0):
    lib.tn_profile_enable(ctx.handle, True)
    lib.tn_profile_read(ctx.handle)
    got, _ = lib.tn_contract(p, ovr, flags=flags)
    lib.tn_profile_enable(ctx.handle, False)
    return got, {k: v["launches"] for k, v in lib.tn_profile_read(ctx.handle).items()}


def test_subtrees_and_concurrent_bits(case):
    circ, net, plan, psi = case
    with lib.Context(64 << 20) as ctx:
        p = ctx.load_network(net, plan.partition_of, 3, plan.tree)
        for x in (0, 5, 2049):
            ovr = amplitude_overrides(net, circ, x)
            got, n = classes(ctx, p, ovr)
            assert n["tree"] >= 1 and n["stream"] <= 8, n
            check(got, psi, x)
            # the partitions side by side give the same bits
            assert lib.tn_contract(p, ovr, flags=lib.TN_FLAG_CONCURRENT)[0] == got
            # nothing of the shared part is kept: the same launches again
            assert classes(ctx, p, ovr)[1] == n


def test_many_override_sets(case):
    """Beyond the layouts a plan keeps for single calls, a new set of
    overridden leaves runs one launch per vertex."""
    circ, net, plan, psi = case
    x = 1234
    ovr = amplitude_overrides(net, circ, x)
    with lib.Context(64 << 20) as ctx:
        p = ctx.load_network(net, plan.partition_of, 3, plan.tree)
        seen = []
        for t in range(24):
            o = dict(ovr)
            o[N + t] = net.tensors[N + t]  # a gate overridden by itself
            got, n = classes(ctx, p, o)
            check(got, psi, x)
            seen.append(n["tree"] > 0)
        assert seen[0] and not seen[-1], seen
        got, n = classes(ctx, p, ovr | {N: net.tensors[N]})  # the first set's layout is still there
        assert n["tree"] > 0
        check(got, psi, x)


def test_programs_give_way(case):
    """A call that needs the whole arena gets it after single calls left their
    programs there, and the single call after it works again."""
    circ, net, plan, psi = case
    x = 77
    ovr = amplitude_overrides(net, circ, x)
    with lib.Context(8 << 20) as ctx:
        lib.tn_contract(ctx.load_network(net, plan.partition_of, 3, plan.tree), ovr)
        # a pair whose operands, result and workspace nearly fill the arena
        m = 384
        a = np.ones((m, m), np.complex64)
        q = None
        while q is None:
            try:
                q = ctx.plan_load([[0, 1], [1, 2]], {0: m, 1: m, 2: m}, [a, a], [0, 0], 1, [(0, 1)], [0, 2], 0,
                                  lib.TN_C64)
                out, _ = lib.tn_contract(q, None, (m, m), lib.TN_C64)
            except lib.TnError as e:
                assert e.status == lib.TN_E_NOMEM
                if q is not None:
                    ctx.free_plan(q)
                    q = None
                m -= 32
                a = np.ones((m, m), np.complex64)
        assert (out == m).all()
        check(lib.tn_contract(ctx.plans[0], ovr)[0], psi, x)
        ctx.free_plan(q)
        check(lib.tn_contract(ctx.plans[0], ovr)[0], psi, x)


def test_tight_arena(case):
    """From the smallest arena that holds the plan and one launch per vertex
    upwards, every size works."""
    circ, net, plan, psi = case
    x = 4001
    ovr = amplitude_overrides(net, circ, x)
    ran = []
    for kib in range(64, 4096, 64):
        with lib.Context(kib << 10) as ctx:
            try:
                p = ctx.load_network(net, plan.partition_of, 3, plan.tree)
                got, n = classes(ctx, p, ovr)
            except lib.TnError as e:
                assert e.status == lib.TN_E_NOMEM and not ran, (kib, ran)
                continue
            check(got, psi, x)
            ran.append(n["tree"] > 0)
    assert ran and not ran[0] and ran[-1], ran
    assert ran == sorted(ran)


def test_noalloc_needs_kept_programs(case):
    """A single call's programs do not count as the strided call's."""
    import torch
    circ, net, plan, psi = case
    ids = output_tensor_ids(net)
    x = 9
    host = np.zeros((N, 2), np.complex64)
    host[np.arange(N), [(x >> k) & 1 for k in range(N)]] = 1
    dev = torch.from_numpy(host).cuda()
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    with lib.Context(64 << 20) as ctx:
        p = ctx.load_network(net, plan.partition_of, 3, plan.tree)
        lib.tn_contract(p, amplitude_overrides(net, circ, x))
        args = [(t, dev.data_ptr() + 16 * k, 16 * N) for k, t in enumerate(ids)]
        with pytest.raises(lib.TnError) as e:
            lib.tn_contract_strided_noalloc(p, 1, args, out.data_ptr())
        assert e.value.status == lib.TN_E_INVALID_ARG
        lib.tn_contract_strided(p, 1, [(t, a, s, lib.TN_C64_DEVICE) for t, a, s in args])
        lib.tn_contract_strided_noalloc(p, 1, args, out.data_ptr())
        check(complex(*out.cpu().tolist()), psi, x)
