"""Serving requests that need all of the arena's room, beside single calls that
upload their subtree programs: the programs count as room that comes back, also
while they are being uploaded, and no request is refused for them."""
import threading
import time

import numpy as np
import pytest

from paper_2507_20667_amd import lib
from paper_2507_20667_amd.inputs import amplitude_network, amplitude_overrides, random_circuit
from paper_2507_20667_amd.planner import plan_from_partition
from paper_2507_20667_amd.planner.plan import tree_partition

pytestmark = pytest.mark.gpu
N, M = 12, 256


def serve_once(ctx, q):
    t = lib.tn_serve_submit(ctx.handle, q)
    t0 = time.time()
    while True:
        st, out, _, _ = lib.tn_serve_poll(ctx.handle, t, (M, M), lib.TN_C64)
        if st != lib.TN_PENDING:
            return out
        assert time.time() - t0 < 30
        time.sleep(0.0003)


def test_requests_of_the_whole_arena():
    circ = random_circuit(N, 12, 3)
    net = amplitude_network(circ, 0)
    plan = plan_from_partition(net.legs, net.dims, tree_partition(net.legs, net.dims, 3), 3)
    ovr = amplitude_overrides(net, circ, 5)
    a = np.ones((M, M), np.complex64)

    def load(ctx):
        return [ctx.load_network(net, plan.partition_of, 3, plan.tree) for _ in range(8)], \
            ctx.plan_load([[0, 1], [1, 2]], {0: M, 1: M, 2: M}, [a, a], [0, 0], 1, [(0, 1)], [0, 2], 0, lib.TN_C64)

    def fits(kib):
        with lib.Context(kib << 10) as ctx:
            try:
                serve_once(ctx, load(ctx)[1])
            except lib.TnError as e:
                assert e.status == lib.TN_E_NOMEM
                return False
            return True

    lo, hi = 1024, 16384  # the smallest arena in which a request fits
    assert fits(hi)
    while hi - lo > 4:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if fits(mid) else (mid, hi)
    with lib.Context(hi << 10) as ctx:
        ps, q = load(ctx)
        stop, failed = threading.Event(), []

        def singles():
            # new sets of overridden leaves: programs to upload in each call
            # (a plan keeps 16 of them)
            for p in ps:
                for t in range(14):
                    if stop.is_set():
                        return
                    try:
                        lib.tn_contract(p, ovr | {N + t: net.tensors[N + t]})
                    except lib.TnError as e:
                        if e.status != lib.TN_E_NOMEM:  # (a request runs)
                            failed.append(e)
                            return

        th = threading.Thread(target=singles)
        th.start()
        n = 0
        try:
            while th.is_alive():
                assert (serve_once(ctx, q) == M).all()
                n += 1
        finally:
            stop.set()
            th.join()
        assert not failed and n >= 1, (failed, n)
