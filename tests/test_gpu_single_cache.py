"""Programs that single calls left in the arena give way to the cache of shared
parts: a batched call keeps its shared part in every arena in which it keeps it
without them."""
import numpy as np
import pytest

from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides, output_tensor_ids, random_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu
N = 12


def test_cache_fills_beside_single_programs():
    circ = random_circuit(N, 12, 3)
    net = amplitude_network(circ, 0)
    plan = plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 3), 3)
    ovr = amplitude_overrides(net, circ, 5)
    ids = output_tensor_ids(net)
    vec = {t: np.stack([ovr[t]] * 2) for t in ids}

    def kept(kib, singles):
        """Whether a second batched call finds the shared part of the first
        (None: no room for the calls)."""
        with lib.Context(kib << 10) as ctx:
            try:
                p = ctx.load_network(net, plan.partition_of, 3, plan.tree)
                q = ctx.load_network(net, plan.partition_of, 3, plan.tree)
                for t in range(singles):
                    lib.tn_contract(p, ovr | {N + t: net.tensors[N + t]})
                lib.tn_profile_enable(ctx.handle, True)
                n = []
                for _ in range(2):
                    lib.tn_profile_read(ctx.handle)
                    lib.tn_contract_strided(q, 2, [(t, vec[t], 32, lib.TN_C128) for t in ids], scales=False)
                    n.append(lib.tn_profile_read(ctx.handle)["tree"]["launches"])
            except lib.TnError as e:
                assert e.status == lib.TN_E_NOMEM
                return None
            return n[1] < n[0]

    seen = []
    for kib in range(128, 1600, 4):
        alone = kept(kib, 0)
        if alone is not None:
            assert kept(kib, 6) == alone, kib
            seen.append(alone)
    assert True in seen
