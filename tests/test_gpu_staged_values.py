"""Closed results of many queries converted on the device: the same values as
a query by itself gives (whose record the host converts), in both result types,
from 1024 queries on and below, with scales when asked for.

Both sides round the same FP64 record once, so the bound is the FP64 inner
product's order of summation: 1e-12 of the largest amplitude, 2^-23 in complex64."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides
from paper_2507_20667_amd.inputs.circuits import brickwork_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("queries", [1023, 1024, 1500])
def test_values(queries):
    circ = brickwork_circuit(12, 9, 2)
    net = amplitude_network(circ, 0)
    plan = plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 3), 3)
    xs = np.random.default_rng(queries).integers(0, 1 << 12, queries)
    with lib.Context(256 << 20) as ctx:
        p = ctx.load_network(net, plan.partition_of, 3, plan.tree)
        qs = [(p, amplitude_overrides(net, circ, int(x))) for x in xs]
        c128, l2, st = lib.tn_contract_batch(ctx.handle, qs, [()] * queries, lib.TN_C128)
        c64 = lib.tn_contract_batch(ctx.handle, qs, [()] * queries, lib.TN_C64)[0]
        kept, k2, _ = lib.tn_contract_batch(ctx.handle, qs, [()] * queries, lib.TN_C128, lib.TN_FLAG_KEEP_SCALE)
        one = [complex(np.asarray(lib.tn_contract(p, o)[0]).reshape(-1)[0]) for _, o in qs[:40]]
    c128, c64 = np.array([complex(v) for v in c128]), np.array([complex(v) for v in c64])
    kept = np.array([complex(v) for v in kept]) * np.exp2(np.asarray(k2))
    big = np.abs(c128).max()
    assert not np.asarray(st).any() and not np.asarray(l2).any()
    assert np.abs(c64 - c128).max() <= 2.0 ** -23 * big
    assert np.abs(kept - c128).max() <= 1e-12 * big
    # a single call sums in FP32 along another layout of the same tree
    assert np.abs(np.array(one) - c128[:40]).max() <= 1e-5 * max(big, 2.0 ** -6)
