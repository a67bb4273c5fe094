"""Nodes whose steps are made a window at a time (64 steps on a wavefront, 8 on
a group of lanes), at the places where a window can go wrong, bit for bit
against the oracle: days of 0 to a few hundred draws (shorter and longer than
a window, and windows that end exactly at a day's last draw), rates that change
at every step, a rate sum that reaches zero inside a window, the first day
(times below 1, added one by one), start times inside a day, times at a power
of two, large times, and times so small that sums fall halfway between two
values.  Integer states and counters must be equal; the continuous state is
the same sequence of operations (1e-12 relative)."""
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


def _case(kind, t0):
    rng = np.random.default_rng(5)
    tspan = t0 + np.arange(0, 7, dtype=np.float64)
    if kind == "sizes":      # X individuals make about X draws a day: 1 .. 300
        return W.birth_death_spec(np.arange(1, 301), tspan, 0.5, 0.5)
    if kind == "dying":      # every node reaches lambda = 0, most inside a window
        return W.birth_death_spec(rng.integers(1, 200, 120), tspan, 0.1, 1.5)
    if kind == "small":      # a few infected: the rates change a lot at each step
        u0 = np.stack([rng.integers(1, 40, 150), rng.integers(0, 6, 150), rng.integers(0, 5, 150)], 1)
        return W.sir_spec(u0, tspan, 1.5, 0.6)
    if kind == "sis":
        return W.sis_spec(np.stack([rng.integers(0, 60, 90), rng.integers(0, 60, 90)], 1), tspan, 0.02, 0.4)
    # thousands of draws a day
    return W.sise_spec(np.stack([rng.integers(3000, 9000, 12), rng.integers(500, 4000, 12)], 1), tspan, 0.5, 0.8,
                       1.0, (0.1, 0.12, 0.1, 0.11), phi0=0.5)


@pytest.mark.parametrize("opts", [dict(lanes=64, wide=10_000), dict(lanes=1, group=-1),
                                  dict(lanes=64, wide=20, group=40)])
@pytest.mark.parametrize("t0", [0.0, 0.25, 1.0, 2.75, 4095.0, 1048570.5])
@pytest.mark.parametrize("kind", ["sizes", "dying", "small", "sis", "heavy"])
def test_windows(lib, kind, t0, opts):
    import oracle
    spec = _case(kind, t0)
    print("[gpu] window", kind, t0, opts, flush=True)
    ref = oracle.run(spec, 91, 3, nthreads=NTHREADS)
    m = lib.Model(spec, **opts)
    m.run(91, 3)
    assert m.wait() == 0 and ref["status"] == 0
    info = m.launch_info()
    assert info["wide"] + info["group"] > 0, info
    U, V = m.trajectory()
    assert np.array_equal(U, ref["U"])
    if V.size:
        np.testing.assert_allclose(V, ref["V"], rtol=1e-12, atol=0)
    c = m.counters()
    assert (c["transitions"], c["node_days"]) == (ref["transitions"], ref["node_days"])
    lane = lib.Model(spec, lanes=1, lattice=2)
    lane.run(91, 3)
    assert lane.wait() == 0 and lane.counters() == c
