"""TN_FLAG_GRAPH: one capture serves calls of either result type, scales kept or
not, and stays when the arena has less room beside its workspace than it had
before that workspace was kept.  (The library prints its host preparation, with
TN_DEBUG, for launch sequences that are not replayed.)"""
import numpy as np
import pytest

from paper_2507_20667_amd import lib

pytestmark = pytest.mark.gpu


def entries(rng, shape):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)


@pytest.mark.parametrize("closed", [False, True])
def test_one_capture_for_every_form(closed, monkeypatch, capfd):
    rng = np.random.default_rng(1)
    A, B = entries(rng, (40, 48)), entries(rng, (48, 40))
    legs, out, shape = ([[0, 1], [1, 0]], None, ()) if closed else ([[0, 1], [1, 2]], [0, 2], (40, 40))
    other = entries(rng, (40, 48))
    monkeypatch.setenv("TN_DEBUG", "1")
    with lib.Context(64 << 20) as ctx:
        p = ctx.plan_load(legs, {0: 40, 1: 48, 2: 40}, [A, B], [0, 0], 1, [(0, 1)], out, 0, lib.TN_C64)
        qs = [(p, {0: A}), (p, {0: other})]
        forms = [(dt, keep) for keep in (0, lib.TN_FLAG_KEEP_SCALE) for dt in (lib.TN_C128, lib.TN_C64)]
        want = {f: lib.tn_contract_batch(ctx.handle, qs, [shape] * 2, f[0], f[1]) for f in forms}
        capfd.readouterr()
        for dt, keep in forms * 3:
            got, l2, _ = lib.tn_contract_batch(ctx.handle, qs, [shape] * 2, dt, keep | lib.TN_FLAG_GRAPH)
            ref, rl2, _ = want[dt, keep]
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]) and np.array_equal(l2, rl2)
    assert capfd.readouterr().err.count("run_group host: layout") == 1


@pytest.mark.parametrize("kib", range(24500, 41000, 500))
def test_kept_workspace(kib, monkeypatch, capfd):
    """The leaves take 11.3 MB, the workspace 12.3 or, with room for more k
    chunks' partial sums, 2 MB more: whatever the arena holds beside the first
    call's, the next ones replay it; and where two workspaces of the smaller size
    fit, a call without a graph still finds room."""
    m, n, k = 24, 320, 4096
    rng = np.random.default_rng(2)
    A, B = entries(rng, (m, k)), entries(rng, (k, n))
    monkeypatch.setenv("TN_DEBUG", "1")
    with lib.Context(kib << 10) as ctx:
        p = ctx.plan_load([[0, 1], [1, 2]], {0: m, 1: k, 2: n}, [A, B], [0, 0], 1, [(0, 1)], [0, 2], 0, lib.TN_C64)
        capfd.readouterr()
        got = [lib.tn_contract_batch(ctx.handle, [(p, None)], [(m, n)], lib.TN_C64, lib.TN_FLAG_GRAPH)[0][0]
               for _ in range(4)]
        assert capfd.readouterr().err.count("run_group host: layout") == 1
        assert all(np.array_equal(g, got[0]) for g in got)
        if kib >= 35500:
            plain = lib.tn_contract_batch(ctx.handle, [(p, None)], [(m, n)], lib.TN_C64)[0][0]
            assert np.linalg.norm(plain - got[0]) <= 1e-6 * np.linalg.norm(plain)
