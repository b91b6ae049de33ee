"""Open results in both output types, with and without scales, permuted or in
the root's order, batched, captured: the same values (rounded to the type) in
every form, and the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides, random_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu
N, OPEN = 11, 5
XS = [0, 5 << OPEN, 33 << OPEN]


@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("size", [1.0, 1e-150])
def test_forms(reverse, size):
    """size: one leaf times this (a complex64 leaf cannot hold the result)."""
    circ = random_circuit(N, 10, 4)
    net = amplitude_network(circ, 0, range(OPEN))
    out_legs = net.output_legs[::-1] if reverse else net.output_legs
    plan = plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 2), 2)
    tensors = list(net.tensors)
    k = 8  # spread over gates, so that each stays in FP32's range
    for t in range(N, N + k):
        tensors[t] = tensors[t] * size ** (1.0 / k)
    psi = oracle.statevector(circ).reshape([2] * N)
    ref = []
    for x in XS:
        block = psi.reshape(-1)[x:x + (1 << OPEN)].reshape([2] * OPEN)
        ref.append(block.transpose(range(OPEN)[::-1]) if reverse else block)
    with lib.Context(256 << 20) as ctx:
        p = ctx.plan_load(net.legs, net.dims, tensors, plan.partition_of, 2, plan.tree, out_legs)
        qs = [(p, amplitude_overrides(net, circ, x, range(OPEN))) for x in XS]
        shape = (2,) * OPEN
        first = {}
        # twice over, so that captured sequences of one form meet the other
        for flags in (0, lib.TN_FLAG_GRAPH, 0, lib.TN_FLAG_GRAPH, lib.TN_FLAG_GRAPH):
            for keep in (0, lib.TN_FLAG_KEEP_SCALE):
                for dt in (lib.TN_C128, lib.TN_C64):
                    outs, l2, _ = lib.tn_contract_batch(ctx.handle, qs, [shape] * len(qs), dt, flags | keep)
                    for i in range(len(qs)):
                        got = outs[i].astype(np.complex128) * 2.0 ** l2[i]
                        want = ref[i] * size
                        if dt == lib.TN_C64 and not keep and size != 1.0:
                            want = want * 0  # below complex64's range
                        tol = 1e-5 * max(np.abs(ref[i]).max(), 2.0 ** (-N / 2)) * size
                        assert np.abs(got - want).max() <= tol, (flags, keep, dt, i)
                        bits = first.setdefault((keep, dt, i), (outs[i].tobytes(), l2[i]))
                        assert bits == (outs[i].tobytes(), l2[i])
        one, _ = lib.tn_contract(p, qs[1][1], shape, lib.TN_C64)
        assert np.abs(one - (ref[1] if size == 1.0 else 0)).max() <= 1e-5
