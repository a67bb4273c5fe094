"""The work that users of this framework have it do, as cases that can be timed.

Every case goes through the public entry points of
``paper_1605_01421_amd.siminf`` (and the seeded input generators of
``workloads``), the way ``surrogate.py`` and ``bench.py`` call them:

* ``listed()`` -- the cases by name;
* ``draw(rng)`` -- one more case from the ranges that the listed ones stand for;
* ``prepare(case, seed)`` -- what a program holds before the call: the model
  handle or the network, and its inputs, made from the seed;
* ``run(state)`` -- one pass, with all of its outputs;
* ``work(case)`` -- the bytes and operations that a pass cannot do without;
* ``exact(case, seed)`` -- the outputs in 64 bits, for the cases whose outputs
  are computed numbers (the simulations return whole numbers, and continuous
  states that follow from them).
"""
import numpy as np
import torch

from paper_1605_01421_amd import siminf
from paper_1605_01421_amd import workloads as W

PROBS = (0.1, 0.5, 0.9)
LR, WEIGHT_DECAY = 1e-5, 1e-4


def listed():
    return [
        # the smallest simulation: the plain SIR example, 100 nodes of 1,000
        # individuals without events, the call of an interactive session
        {"name": "sir-plain", "kind": "plain", "Nn": 100, "days": 99},
        # SIR with births, exits and animal movements over a year: the event
        # workload of the benchmark
        {"name": "sir-events", "kind": "events", "Nn": 10_000, "days": 365, "solver": "ssm"},
        # the same by the all events method, on a region's worth of herds
        {"name": "sir-events-aem", "kind": "events", "Nn": 2_999, "days": 365, "solver": "aem"},
        # a country's herds with an environmental pathogen (SISe), one year of
        # the ten of the full study
        {"name": "sise-events", "kind": "sise", "Nn": 37_000, "days": 365},
        # the spatially coupled model on 1,600 farms, one year
        {"name": "sise-sp", "kind": "sp", "Nn": 1_600, "days": 365},
        # a model given as transition strings, with a vaccination campaign
        {"name": "vaccination", "kind": "vaccination", "Nn": 1_600, "days": 300},
        # the ensemble of parameter sets that the surrogate's targets come
        # from: weekly sums and prevalence quantiles over the replicates
        {"name": "ensemble", "kind": "ensemble", "sets": 64, "replicates": 8},
        # training steps of the surrogate at its minibatch (the last ones of
        # the cosine schedule), then the weights
        {"name": "train-128", "kind": "train", "batch": 128, "steps": 64, "width": 256, "weeks": 52},
        # one large-batch gradient, read back
        {"name": "grad-4096", "kind": "grad", "batch": 4_096, "width": 256, "weeks": 52},
        # inference over a large sweep of parameter sets
        {"name": "infer-65536", "kind": "infer", "batch": 65_536, "width": 256, "weeks": 52},
        # the ensemble's answer with its disagreement for 1,000 held-out sets
        {"name": "predict-1000", "kind": "predict", "batch": 1_000, "members": 4, "width": 256, "weeks": 52,
         "static": False},
        # the same for a handful of sets in a serving loop
        {"name": "predict-8", "kind": "predict", "batch": 8, "members": 4, "width": 256, "weeks": 52, "static": True},
    ]


def _between(rng, lo, hi):
    """A whole number, uniform in its logarithm over [lo, hi]."""
    return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))


def draw(rng):
    kind = rng.choice(["plain", "events", "sise", "sp", "vaccination", "ensemble", "train", "grad", "infer", "predict"])
    if kind == "plain":
        return {"kind": kind, "Nn": _between(rng, 10, 400), "days": rng.randint(30, 200)}
    if kind == "events":
        return {"kind": kind, "Nn": _between(rng, 500, 10_000), "days": rng.randint(60, 365),
                "solver": rng.choice(["ssm", "ssm", "ssm", "aem"])}
    if kind == "sise":
        return {"kind": kind, "Nn": _between(rng, 3_000, 37_000), "days": rng.randint(60, 365)}
    if kind == "sp":
        return {"kind": kind, "Nn": _between(rng, 200, 1_600), "days": rng.randint(60, 365)}
    if kind == "vaccination":
        return {"kind": kind, "Nn": _between(rng, 200, 1_600), "days": rng.randint(60, 300)}
    if kind == "ensemble":
        return {"kind": kind, "sets": rng.randint(8, 64), "replicates": rng.randint(3, 8)}
    net = {"width": rng.choice([64, 96, 128, 130, 192, 200, 256, 256]), "weeks": rng.choice([13, 26, 52, 52])}
    if kind == "train":
        return {"kind": kind, "batch": _between(rng, 16, 512), "steps": rng.randint(16, 64), **net}
    if kind == "grad":
        return {"kind": kind, "batch": _between(rng, 200, 4_096), **net}
    if kind == "infer":
        return {"kind": kind, "batch": _between(rng, 1, 65_536), **net}
    return {"kind": kind, "batch": _between(rng, 1, 4_000), "members": rng.randint(2, 6), "static": rng.random() < 0.3,
            **net}


# ---- inputs ------------------------------------------------------------------

def _dims(case):
    w = case["width"]
    return (8, w, w, w, w, 3 * case["weeks"])


def _weights(dims, seed):
    """Uniform on +-sqrt(6 / fan in), with the small biases of a trained net."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(len(dims) - 1):
        lim = np.sqrt(6.0 / dims[i])
        out.append((rng.uniform(-lim, lim, (dims[i + 1], dims[i])).astype(np.float32),
                    (0.05 * rng.standard_normal(dims[i + 1])).astype(np.float32)))
    return out


def _samples(dims, n, seed):
    """Standardised features, and targets that are a smooth map of them with
    some noise, as float32 tensors on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    X = torch.randn((n, dims[0]), generator=g, device="cuda")
    A = torch.randn((dims[0], dims[-1]), generator=g, device="cuda") / 3
    T = torch.tanh(X @ A) + 0.05 * torch.randn((n, dims[-1]), generator=g, device="cuda")
    return X, T


def _scales(n, seed):
    rng = np.random.default_rng(seed)
    mean = torch.from_numpy((0.2 * rng.random(n)).astype(np.float32)).cuda()
    std = torch.from_numpy(rng.uniform(0.02, 0.2, n).astype(np.float32)).cuda()
    return mean, std


def _spec(case, seed):
    if case["kind"] == "plain":
        rng = np.random.default_rng(seed)
        infected = rng.integers(5, 16, case["Nn"])
        u0 = np.stack([1000 - infected, infected, 0 * infected], axis=1)
        return W.sir_spec(u0, np.arange(1, case["days"] + 2), 0.16, 0.077)
    make = {"events": W.sir_with_events, "sise": W.sise_with_events, "sp": W.sise_sp_with_events,
            "vaccination": W.vaccination_example}[case["kind"]]
    return make(seed=seed, Nn=case["Nn"], days=case["days"])


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind, "seed": 1 + seed % 1_000_003}
    if kind in ("plain", "events", "sise", "sp", "vaccination"):
        state["model"] = siminf.Model(_spec(case, seed), solver=case.get("solver", "ssm"))
        return state
    if kind == "ensemble":
        sets = W.ensemble_sets(seed=seed, n_sets=case["sets"], replicates=case["replicates"])
        state["model"] = siminf.Model([(s.spec, s.replicates) for s in sets], record=siminf.RECORD_SUMS)
        state["replicates"] = case["replicates"]
        return state
    dims, B = _dims(case), case["batch"]
    nets = []
    for k in range(case.get("members", 1)):
        net = siminf.MLP(dims, 4096 if kind == "predict" else B)
        net.set_params(_weights(dims, 64 * seed + k))
        nets.append(net)
    X, T = _samples(dims, B * case.get("steps", 1), seed)
    state.update(nets=nets, net=nets[0], X=X)
    if kind == "train":
        state["batches"] = [(X[i:i + B], T[i:i + B]) for i in range(0, len(X), B)]
    elif kind == "grad":
        state["T"] = T
    elif kind == "predict":
        state["mean"], state["std"] = _scales(dims[-1], seed)
        state["static"] = case["static"]
    return state


# ---- passes --------------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "ensemble":
        m = state["model"]
        m.run(state["seed"])
        q = m.prevalence_quantiles(1, (0, 1, 2), state["replicates"], 1, m.ntspan - 1, PROBS)
        return {"quantiles": q, "sums": m.sums()}
    if kind == "train":
        net, last = state["net"], len(state["batches"]) - 1
        for i, (x, t) in enumerate(state["batches"]):
            loss = net.backward(x, t, PROBS, want_loss=i == last)
            net.adamw(LR, weight_decay=WEIGHT_DECAY)
        return {"loss": loss, "weights": net.get_params()}
    if kind == "grad":
        loss = state["net"].backward(state["X"], state["T"], PROBS)
        return {"loss": loss, "grads": state["net"].get_grads()}
    if kind == "infer":
        return {"Y": state["net"].forward(state["X"])}
    if kind == "predict":
        Y, dis = siminf.ensemble_predict(state["nets"], state["X"], state["mean"], state["std"],
                                         static=state["static"])
        return {"Y": Y, "disagreement": dis}
    m = state["model"]
    m.run(state["seed"])
    U, V = m.trajectory(device=True)
    return {"U": U, "V": V} if V.numel() else {"U": U}


# ---- what a pass cannot do without -------------------------------------------------

# 32- and 64-bit operations of one direct-method step (a Philox block, a
# logarithm, a division, the rates and the choice)
STEP_OPS = 172.0


def work(case):
    kind = case["kind"]
    if kind == "plain":
        # each of the 1,000 individuals goes through at most two transitions
        records = 12.0 * case["Nn"] * (case["days"] + 1)
        return {"bytes": records, "flops": STEP_OPS * case["Nn"] * (1_500.0 + case["days"])}
    if kind in ("events", "sise", "sp", "vaccination"):
        # the record of every node and day, about 0.13 (SIR) or 0.08 (SISe)
        # events of 16 bytes per node and day, and at least one draw
        width, events = {"events": (12, 0.13), "sise": (16, 0.08), "sp": (16, 0.08), "vaccination": (20, 0.13)}[kind]
        days = case["days"] * float(case["Nn"])
        return {"bytes": days * (width + 16 * events), "flops": STEP_OPS * days}
    if kind == "ensemble":
        # about 3,400 nodes a set, each read once, 365 days of about 7 draws
        nodes = 3_400.0 * case["sets"] * case["replicates"]
        return {"bytes": nodes * 28 + 53 * 24.0 * case["sets"] * case["replicates"],
                "flops": STEP_OPS * nodes * 365 * 7}
    dims, B = _dims(case), float(case["batch"])
    params = float(sum(a * b + b for a, b in zip(dims[:-1], dims[1:])))
    macs = float(sum(a * b for a, b in zip(dims[:-1], dims[1:])))
    rows = B * 4 * (dims[0] + dims[-1])
    if kind == "train":
        # three products a layer; weights, gradients and the two moments
        return {"bytes": case["steps"] * (rows + params * 30), "flops": case["steps"] * 6 * macs * B}
    if kind == "grad":
        return {"bytes": rows + params * 6, "flops": 6 * macs * B}
    k = case.get("members", 1)
    return {"bytes": rows + 2 * k * params, "flops": 2 * macs * B * k}


# ---- the outputs in 64 bits ----------------------------------------------------------

def _forward(params, X):
    """The network with erf GELU: h Phi(h) between the layers."""
    h = X
    for i, (Wl, b) in enumerate(params):
        h = h @ Wl.T + b
        if i + 1 < len(params):
            h = 0.5 * h * torch.special.erfc(-h / np.sqrt(2.0))
    return h


def _params64(dims, seed):
    return [(torch.from_numpy(Wl).double().cuda(), torch.from_numpy(b).double().cuda())
            for Wl, b in _weights(dims, seed)]


def _loss_and_grads(params, X, T):
    flat = [p.detach().requires_grad_(True) for pair in params for p in pair]
    Y = _forward(list(zip(flat[0::2], flat[1::2])), X)
    q = torch.tensor(PROBS, dtype=torch.float64, device=X.device).repeat(T.shape[1] // len(PROBS))
    d = T - Y
    loss = torch.where(d > 0, q * d, (q - 1.0) * d).mean()
    return loss.detach(), torch.autograd.grad(loss, flat)


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("train", "grad", "infer", "predict"):
        return None
    dims, B = _dims(case), case["batch"]
    X, T = _samples(dims, B * case.get("steps", 1), seed)
    X, T = X.double(), T.double()
    if kind == "infer":
        return {"Y": _forward(_params64(dims, 64 * seed), X)}
    if kind == "predict":
        mean, std = (t.double() for t in _scales(dims[-1], seed))
        P = torch.stack([_forward(_params64(dims, 64 * seed + k), X) * std + mean for k in range(case["members"])])
        return {"Y": P.mean(0), "disagreement": P.std(0, unbiased=True).mean(1)}
    params = _params64(dims, 64 * seed)
    if kind == "grad":
        loss, g = _loss_and_grads(params, X, T)
        return {"loss": float(loss), "grads": list(zip(g[0::2], g[1::2]))}
    # AdamW with decoupled weight decay, one step a minibatch
    flat = [p for pair in params for p in pair]
    m, v = [torch.zeros_like(p) for p in flat], [torch.zeros_like(p) for p in flat]
    for t in range(1, case["steps"] + 1):
        rows = slice((t - 1) * B, t * B)
        loss, g = _loss_and_grads(list(zip(flat[0::2], flat[1::2])), X[rows], T[rows])
        for i, gi in enumerate(g):
            m[i] = 0.9 * m[i] + 0.1 * gi
            v[i] = 0.999 * v[i] + 0.001 * gi * gi
            step = (m[i] / (1 - 0.9 ** t)) / ((v[i] / (1 - 0.999 ** t)).sqrt() + 1e-8)
            flat[i] = flat[i] - LR * (step + WEIGHT_DECAY * flat[i])
    return {"loss": float(loss), "weights": list(zip(flat[0::2], flat[1::2]))}
