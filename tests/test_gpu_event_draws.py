"""The individuals of an event drawn by many lanes at once, the mailbox words
of models with more than three compartments, a node's arrivals taken by the
lanes that carry it, and the exponentials of the all events method made ahead:
around the sizes at which a window of draws or arrivals, a word or a lane's
share ends, with every way a node is carried, against the oracle.  States are
whole numbers and have to be equal; nothing here has a tolerance."""
import os

import numpy as np
import pytest

from paper_1605_01421_amd import workloads as W

pytestmark = pytest.mark.gpu

NTHREADS = min(16, os.cpu_count() or 1)
SIZES = [1, 3, 4, 5, 7, 8, 9, 16, 17, 63, 64, 65, 128, 129, 700]


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1605_01421_amd import siminf
    siminf.load()
    return siminf


def _check(lib, spec, what, solver="ssm", **opts):
    import oracle
    print("[gpu]", what, spec.name, opts, flush=True)
    ref = oracle.run(spec, 11, 2, nthreads=NTHREADS, solver=solver)
    assert ref["status"] == 0, ref["error"]
    m = lib.Model(spec, solver=solver, **opts)
    for _ in range(2):
        m.run(11, 2)
        assert m.wait() == 0, m.error_info()
        U, V = m.trajectory()
        assert np.array_equal(U, ref["U"])
        if V.size:
            assert np.array_equal(V, ref["V"])
    c = m.counters()
    assert (c["transitions"], c["events"]) == (ref["transitions"], ref["events"])
    m.close()


def _rows(Nn, days, transfers, every, one, shift):
    """Events of each size in SIZES on every node in turn, as exits, internal
    transfers (where there is a shift) and transfers to the next node, and
    proportions from none to all; select `every` takes several compartments,
    `one` a single one."""
    rows = []
    for i in range(Nn):
        for d in range(1, days + 1):
            n = SIZES[(i + d) % len(SIZES)]
            kind = (i + 3 * d) % 4
            if kind == 0:
                rows.append((W.EXIT, d, i, 0, max(n // 8, 1), 0.0, every, -1))
                rows.append((W.ENTER, d, i, 0, max(n // 8, 1), 0.0, one, -1))
            elif kind == 1 and shift is not None:
                rows.append((W.INTTRANS, d, i, 0, 0, (0.0, 0.3, 0.8, 1.0)[d % 4], every, shift))
            elif kind == 2 and transfers:
                rows.append((W.EXTTRANS, d, i, (i + 1) % Nn, n, 0.0, every, -1))
            elif transfers:
                rows.append((W.EXTTRANS, d, i, (i + 5) % Nn, 0, 0.02, every, -1))
                if d % 5 == 0:
                    rows.append((W.EXTTRANS, d, i, (i + 2) % Nn, 0, 1.0, one, -1))
    return W.make_events(rows)


def _sir(Nn, transfers, days=24):
    rng = np.random.default_rng(Nn)
    u0 = np.stack([rng.integers(20000, 40000, Nn), rng.integers(0, 30, Nn), rng.integers(0, 500, Nn)], 1)
    ev = _rows(Nn, days, transfers, 3, 1, None)
    return W.sir_spec(u0, np.arange(0, days + 1), 0.02, 0.05, events=ev, name="SIR draws")


def _five(Nn, days=24, herd=3000, big=0):
    """S, I, Icum, R, V: five compartments take two mailbox words."""
    rng = np.random.default_rng(Nn + 1)
    u0 = np.zeros((Nn, 5), np.int64)
    u0[:, 0] = rng.integers(20000, 40000, Nn)
    u0[:, 1] = rng.integers(0, 30, Nn)
    u0[:, 3] = rng.integers(0, herd, Nn)
    E = np.array([[1, 1, 1], [0, 1, 1], [0, 0, 0], [0, 1, 1], [0, 1, 0]], np.int32)
    N = np.array([[4], [3], [0], [1], [0]], np.int32)
    ev = _rows(Nn, days, True, 1, 0, 0)
    if big:
        # counts beyond 16 bits go through the side array
        u0[:3, 0] += 4 * big
        more = [(W.EXTTRANS, d, i, i + 1, big + d, 0.0, 1, -1) for d in (2, 9) for i in range(2)]
        ev = W.concat_events(ev, W.make_events(more))
    return W.mparse_spec(["S -> b*S*I/(S+I+R+V) -> I + Icum", "I -> g*I -> R"], ["S", "I", "Icum", "R", "V"], u0,
                         np.arange(0, days + 1), gdata=dict(b=0.02, g=0.05), E=E, N=N, events=ev, name="five draws")


@pytest.mark.parametrize("transfers", [False, True])
@pytest.mark.parametrize("opts", [dict(), dict(lanes=64, wide=200), dict(lanes=1, group=-1), dict(lanes=1),
                                  dict(lanes=1, pack=4), dict(lanes=64, wide=9, group=40, pack=8),
                                  dict(lanes=64, wide=70, lattice=2), dict(mode=1)])
def test_sir(lib, transfers, opts):
    _check(lib, _sir(150, transfers), f"transfers {transfers}", **opts)


@pytest.mark.parametrize("Nn,big", [(7, 0), (130, 0), (130, 0xFFF0)])
def test_five_compartments(lib, Nn, big):
    for opts in (dict(), dict(pack=64), dict(mode=1)):
        _check(lib, _five(Nn, big=big), f"{Nn} nodes, big {big}", **opts)


def test_no_transfers_on_lanes_of_a_queue(lib):
    _check(lib, _sir(300, False), "lane queue", lane_queue=1)


def _hub(Nn, days=12):
    """Every node ships to node 0 every day, node 0 to a few and some node to
    itself, in any order: node 0's arrivals fill a window of lanes, or several,
    with transfers it sends in between, before the first and after the last."""
    rng = np.random.default_rng(Nn)
    u0 = np.stack([rng.integers(300, 900, Nn), rng.integers(0, 9, Nn), np.zeros(Nn, int)], 1)
    rows = []
    for d in range(1, days + 1):
        today = [(W.EXTTRANS, d, i, 0, int(rng.integers(1, 9)), 0.0, 3, -1) for i in range(1, Nn)]
        today += [(W.EXTTRANS, d, 0, int(rng.integers(1, Nn)), int(rng.integers(1, 30)), 0.0, 3, -1)
                  for _ in range(d % 6)]
        if d % 3 == 0:
            at = int(rng.integers(0, Nn))
            today.append((W.EXTTRANS, d, at, at, 4, 0.0, 3, -1))
        rows += [today[i] for i in rng.permutation(len(today))]
    return W.sir_spec(u0, np.arange(0, days + 1), 0.1, 0.05, events=W.make_events(rows), name="hub")


@pytest.mark.parametrize("Nn", [2, 9, 10, 64, 65, 66, 200])
def test_hub(lib, Nn):
    for opts in (dict(), dict(lanes=64, wide=Nn), dict(lanes=1, group=-1), dict(lanes=64, wide=1, group=Nn // 2),
                 dict(lanes=1, pack=4), dict(mode=1)):
        _check(lib, _hub(Nn), f"{Nn} nodes", **opts)


@pytest.mark.parametrize("pack", [0, 4, 8, 16, 32, 64])
def test_all_events_method(lib, pack):
    """Two channels (up to 8 exponentials ahead of each) and five (3 ahead at
    4 nodes a wavefront, none at more), with few and with many steps a day,
    nodes past a whole wavefront and a last one that is nearly empty."""
    Nn = 131
    rng = np.random.default_rng(4)
    u0 = np.stack([rng.integers(0, 400, Nn), rng.integers(0, 40, Nn), np.zeros(Nn, int)], 1)
    _check(lib, W.sir_spec(u0, np.arange(0, 31), 0.4, 0.2), "SIR", "aem", pack=pack)
    spec = W.sir_with_events(seed=3, Nn=Nn, days=30)
    _check(lib, spec, "SIR, transfers", "aem", pack=pack)
    tr = ["S -> b*S*I/(S+E+I+R+1) -> E", "E -> 0.7*E -> I", "I -> g*I -> R", "R -> w*R -> S", "S -> 0.01*S -> R"]
    u5 = np.concatenate([u0[:, :1], np.zeros((Nn, 1), int), u0[:, 1:]], 1)
    _check(lib, W.mparse_spec(tr, ["S", "E", "I", "R"], u5, np.arange(0, 31), gdata=dict(b=0.5, g=0.2, w=0.05),
                              name="SEIRS"), "five channels", "aem", pack=pack)
