"""Per-query subtrees of a few queries in the level kernel, of more in the batch
kernel: the same amplitudes on both sides of the rule's lines, against the
state vector (|a - a_ref| / max(|a_ref|, 2^(-n/2)) <= 1e-5, the FP32 bound)."""
import numpy as np
import pytest

import oracle
from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides, random_circuit
from paper_2507_20667_amd.inputs.circuits import brickwork_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu


# a chain of gates (the batch kernel from two queries on), programs of one
# and of several subtrees (the level kernel up to 256 workgroups)
@pytest.mark.parametrize("make, parts", [
    (lambda: brickwork_circuit(16, 14, 1), 4),
    (lambda: random_circuit(14, 12, 3), 4),
    (lambda: random_circuit(16, 12, 0), 2),
])
def test_few_queries(make, parts):
    circ = make()
    n = circ.n
    net = amplitude_network(circ, 0)
    plan = plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, parts), parts)
    psi = oracle.statevector(circ)
    rng = np.random.default_rng(n)
    with lib.Context(256 << 20) as ctx:
        p = ctx.load_network(net, plan.partition_of, parts, plan.tree)
        for q in (1, 2, 3, 65, 256, 257):
            xs = [int(x) for x in rng.integers(0, 1 << n, q)]
            ovr = [amplitude_overrides(net, circ, x) for x in xs]
            got, _, st = lib.tn_contract_batch(ctx.handle, [(p, o) for o in ovr], [()] * q)
            assert not st.any()
            for x, a in zip(xs, got):
                err = abs(complex(a) - psi[x]) / max(abs(psi[x]), 2.0 ** (-n / 2))
                assert err <= 1e-5, (q, x, err)
