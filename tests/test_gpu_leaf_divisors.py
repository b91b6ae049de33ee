"""Gates stored divided by their largest component: every entry point multiplies
its results by the divisors of the leaves it did not override.

A network of many Hadamard gates (1/sqrt 2 is off by 1.7e-8 in FP32, always
with the same sign) shows a missing divisor as a factor of sqrt 2 and an
undivided gate as an error that grows with the gates.  Bound: the FP32
rounding of each of the network's V contractions, at most 2^-24 of the value
twice (product and sum), adding in quadrature, eight standard deviations:
8 sqrt(2 V) 2^-24 of max(|a|, 2^(-n/2))."""
import numpy as np
import pytest

import oracle
from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import (Circuit, amplitude_network, amplitude_overrides, output_tensor_ids)
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu
N = 10


def circuit():
    rng = np.random.default_rng(0)
    c = Circuit(N, name="hadamards")
    for layer in range(24):
        for q in range(N):
            c.add("H", (q,))
            c.add("RZ", (q,), (rng.uniform(0, 6),))
        if layer % 6 == 0:
            for q in range(layer // 6 % 2, N - 1, 2):
                c.add("CX", (q, q + 1))
    return c


@pytest.fixture(scope="module")
def case():
    circ = circuit()
    net = amplitude_network(circ, 0)
    return circ, net, plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 2), 2), \
        oracle.statevector(circ)


@pytest.fixture(scope="module")
def ctx():
    c = lib.Context(256 << 20)
    yield c
    c.close()


def check(net, psi, x, got):
    tol = 8 * np.sqrt(2.0 * net.num_tensors) * 2.0 ** -24
    err = abs(complex(np.asarray(got).reshape(-1)[0]) - psi[x]) / max(abs(psi[x]), 2.0 ** (-N / 2))
    assert err <= tol, (x, err, tol)


XS = [0, 3, 700, 1023]


def test_single_batch_serve_scale(ctx, case):
    circ, net, plan, psi = case
    p = ctx.load_network(net, plan.partition_of, 2, plan.tree)
    for x in XS:
        ovr = amplitude_overrides(net, circ, x)
        check(net, psi, x, lib.tn_contract(p, ovr)[0])
        check(net, psi, x, lib.tn_contract(p, ovr, flags=lib.TN_FLAG_CONCURRENT)[0])
        m, l2 = lib.tn_contract(p, ovr, flags=lib.TN_FLAG_KEEP_SCALE)
        big = max(abs(complex(m.reshape(-1)[0]).real), abs(complex(m.reshape(-1)[0]).imag))
        assert 0.5 <= big < 1.0
        check(net, psi, x, m * 2.0 ** l2)
        t = lib.tn_serve_submit(ctx.handle, p, ovr)
        while (r := lib.tn_serve_poll(ctx.handle, t))[0] == lib.TN_PENDING:
            pass
        check(net, psi, x, r[1])
    check(net, psi, 0, lib.tn_contract(p)[0])
    # queries that override different gates by themselves: the one that
    # leaves a gate alone takes the plan's undivided copy of it
    g = [i for i, tag in enumerate(net.tags) if tag == "gate"]
    qs = [(p, amplitude_overrides(net, circ, x) | {g[k]: net.tensors[g[k]] for k in ks})
          for x, ks in zip(XS, ([], [0, 5], [5, 40], [2]))]
    for flags in (0, lib.TN_FLAG_GRAPH):
        outs, _, _ = lib.tn_contract_batch(ctx.handle, qs, [()] * len(qs), flags=flags)
        for x, o in zip(XS, outs):
            check(net, psi, x, o)
    ctx.free_plan(p)


def test_strided_and_noalloc(ctx, case):
    import torch
    circ, net, plan, psi = case
    p = ctx.load_network(net, plan.partition_of, 2, plan.tree)
    ids = output_tensor_ids(net)
    gate = [i for i, tag in enumerate(net.tags) if tag == "gate"][7]
    host = np.zeros((len(XS), N, 2), np.complex64)
    for i, x in enumerate(XS):
        host[i, np.arange(N), [(x >> k) & 1 for k in range(N)]] = 1
    dev = torch.from_numpy(host).cuda()
    gdev = torch.from_numpy(net.tensors[gate].astype(np.complex64).reshape(-1)).cuda()
    for extra in ([], [(gate, gdev.data_ptr(), 0, lib.TN_C64_DEVICE)]):
        ov = [(t, dev.data_ptr() + 16 * k, 16 * N, lib.TN_C64_DEVICE) for k, t in enumerate(ids)] + extra
        pinned = torch.zeros((len(XS), 2), dtype=torch.float64, pin_memory=True)
        dres = torch.zeros((len(XS), 2), dtype=torch.float64, device="cuda")
        outs = [lib.tn_contract_strided(p, len(XS), ov)[0],
                lib.tn_contract_strided(p, len(XS), ov, out=pinned.numpy().view(np.complex128).reshape(-1))[0],
                lib.tn_contract_strided(p, len(XS), ov, out_dtype=lib.TN_C64)[0]]
        lib.tn_contract_strided_noalloc(p, len(XS), [o[:3] for o in ov], dres.data_ptr())
        outs.append(dres.cpu().numpy().view(np.complex128).reshape(-1))
        for o in outs:
            for x, v in zip(XS, o):
                check(net, psi, x, v)
        assert (outs[0] == outs[1]).all() and (outs[0] == outs[3]).all()
    ctx.free_plan(p)


def test_sliced_and_open(ctx, case):
    circ, net, plan, psi = case
    p = ctx.load_network(net, plan.partition_of, 2, plan.tree)
    legs = [l for l in net.legs[N]][:1] + [net.legs[N + 60][0]]
    s = ctx.slice_plan(p, legs)
    gates = [i for i, l in enumerate(net.legs) if legs[0] in l or legs[1] in l]
    for x in XS:
        ovr = amplitude_overrides(net, circ, x)
        check(net, psi, x, lib.tn_contract(s, ovr)[0])
        for t in gates:
            check(net, psi, x, lib.tn_contract(s, ovr | {t: net.tensors[t]})[0])
    ctx.free_plan(s)
    ctx.free_plan(p)
    onet = amplitude_network(circ, 0, range(4))
    oplan = plan_from_partition(onet.legs, onet.dims, tree_partition(onet.legs, onet.dims, 2), 2)
    p = ctx.load_network(onet, oplan.partition_of, 2, oplan.tree)
    for flags in (0, lib.TN_FLAG_KEEP_SCALE):
        got, l2 = lib.tn_contract(p, None, (16,), flags=flags)
        for x in range(16):
            check(onet, psi, x, got[x] * 2.0 ** l2)
    ctx.free_plan(p)
