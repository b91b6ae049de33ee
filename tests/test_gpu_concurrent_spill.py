"""TN_FLAG_CONCURRENT on plans whose subtrees keep intermediates in device memory
(from 64 entries on here): the same bits as the serial order and as a batch of
one, though the concurrent layout has no shared parts."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides, random_bitstrings, random_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,depth,seed", [(12, 12, 3), (14, 14, 1), (16, 12, 2), (18, 12, 4), (18, 16, 7)])
@pytest.mark.parametrize("spill", [32, 64, 512])
def test_bits(n, depth, seed, spill, monkeypatch):
    monkeypatch.setenv("TN_TREE_SPILL", str(spill))
    circ = random_circuit(n, depth, seed)
    net = amplitude_network(circ, 0)
    plan = plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 4), 4)
    with lib.Context(1 << 30) as ctx:
        p = ctx.load_network(net, plan.partition_of, 4, plan.tree)
        for x in random_bitstrings(n, 3, seed):
            ovr = amplitude_overrides(net, circ, x)
            a = lib.tn_contract(p, ovr)[0].reshape(-1)
            assert np.array_equal(lib.tn_contract(p, ovr, flags=lib.TN_FLAG_CONCURRENT)[0].reshape(-1), a)
            assert np.array_equal(lib.tn_contract_batch(ctx.handle, [(p, ovr)], [()])[0][0].reshape(-1), a)
