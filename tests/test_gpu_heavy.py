"""Lane queue with its heavy nodes on whole wavefronts: sums and full records
of batches whose nodes straddle the cut, against the oracle and against the
same batch with every node on one lane (lanes = 1), where node sizes, events,
an early end (nodes that can no longer change) or an error make a difference."""
import os

import numpy as np
import pytest

from paper_1605_01421_amd import workloads as W

pytestmark = pytest.mark.gpu

NTHREADS = min(16, os.cpu_count() or 1)


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1605_01421_amd import siminf
    siminf.load()
    return siminf


def _sets(case):
    rng = np.random.default_rng(8)
    if case == "uneven":      # heavy-tailed sizes, SIR and SISe, and a spec without nodes
        sets = [s.spec for s in W.ensemble_sets(seed=12, n_sets=6, replicates=1, days=40, nn_range=(1, 700))]
        return sets[:3] + [W.sir_spec(np.zeros((0, 3), int), sets[0].tspan)] + sets[3:]
    tspan = np.arange(0, 41, 5)
    if case == "one node":    # a single node is heavy, nothing is left for the lanes
        return [W.sise_spec(np.array([[900, 100]]), tspan, 0.0175, 0.1, 1.0, (0.1, 0.12, 0.1, 0.11))]
    if case == "dying":       # large nodes that die out or start without infection
        u0 = np.stack([rng.integers(1, 3000, 300), rng.integers(0, 3, 300), np.zeros(300, int)], 1)
        return [W.sir_spec(u0, tspan, 0.05, 0.6)]
    assert case == "events"   # node-local events on heavy and light nodes
    spec = W.sir_with_events(seed=9, Nn=300, days=40)
    ev = {k: np.asarray(v)[np.asarray(spec.events["event"]) != W.EXTTRANS] for k, v in spec.events.items()}
    return [W.sir_spec(np.asarray(spec.u0), np.asarray(spec.tspan), 0.16, 0.077, events=ev)]


@pytest.mark.parametrize("record", [0, 1])
@pytest.mark.parametrize("case", ["uneven", "one node", "dying", "events"])
def test_heavy_nodes(lib, case, record):
    import oracle
    specs, reps = _sets(case), 3
    print("[gpu] heavy", case, record, flush=True)
    batch = [(s, reps) for s in specs]
    m = lib.Model(batch, record=record, lane_queue=1)
    lanes = lib.Model(batch, record=record, lane_queue=1, lanes=1)
    assert m.launch_info()["mode"] == 3 and m.launch_info()["wide"] > 0 and lanes.launch_info()["wide"] == 0
    for x in (m, lanes):
        x.run(33, 4)
        assert x.wait() == 0, x.error_info()
    assert m.counters() == lanes.counters()
    if record:
        assert np.array_equal(m.sums(), lanes.sums())
    for r in range(m.runs):
        ref = oracle.run(specs[r // reps], 33, 4 + r, nthreads=NTHREADS)
        if record:
            nc = ref["U"].shape[2]
            assert np.array_equal(m.sums()[r, :, :nc], ref["U"].astype(np.int64).sum(axis=1)), r
        else:
            U, V = m.trajectory(r)
            assert np.array_equal(U, ref["U"]), r
            if V.size:
                np.testing.assert_allclose(V, ref["V"], rtol=1e-12, atol=0)


def test_heavy_node_error(lib):
    """The first error in serial order, raised by a node on a wavefront."""
    u0 = np.array([[40, 2, 0]] * 30 + [[4000, 400, 0]] + [[50, 1, 0]] * 30)
    spec = W.sir_spec(u0, np.arange(0, 10), 0.4, 0.1)
    spec.S = np.array([[-1, 0], [1, -1], [-1, 1]])  # an infection also removes a recovered
    got = []
    for lanes in (0, 1):
        m = lib.Model(spec, record=lib.RECORD_SUMS, lane_queue=1, lanes=lanes)
        m.run(2, 0)
        assert m.wait() == -5
        got.append(m.error_info())
    assert got[0] == got[1]
