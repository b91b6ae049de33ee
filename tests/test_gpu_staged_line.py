"""Closed results on either side of the number of queries (256) from which the
kernel returns them as values: equal, in both types, to those with their scales
kept (which are always returned as records) within the rounding of the type."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides, brickwork_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("queries", [255, 256, 257, 600])
def test_line(queries):
    circ = brickwork_circuit(12, 9, 2)
    net = amplitude_network(circ, 0)
    plan = plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 3), 3)
    xs = np.random.default_rng(queries).integers(0, 1 << 12, queries)
    with lib.Context(256 << 20) as ctx:
        p = ctx.load_network(net, plan.partition_of, 3, plan.tree)
        qs = [(p, amplitude_overrides(net, circ, int(x))) for x in xs]
        shapes = [()] * queries
        kept, l2, _ = lib.tn_contract_batch(ctx.handle, qs, shapes, lib.TN_C128, lib.TN_FLAG_KEEP_SCALE)
        want = np.array([complex(v) for v in kept]) * np.exp2(l2)
        for dt, eps in ((lib.TN_C128, 2.0 ** -50), (lib.TN_C64, 2.0 ** -23)):
            got, scale, st = lib.tn_contract_batch(ctx.handle, qs, shapes, dt)
            assert not np.any(st) and not np.any(scale)
            assert (np.abs(np.array([complex(v) for v in got]) - want) <= eps * np.abs(want)).all()
