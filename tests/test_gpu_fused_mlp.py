"""Networks whose widths all fit the fused kernels (at most 256), at the edges
of their tiles: widths and batches just below, at and above multiples of 16
and 32, one layer, one row, one output, several workgroups and both row-tile
sizes; and a network one column too wide, which takes the general kernels.
Against the float64 oracle with bfloat16 rounding where the kernels round.
Tolerance: a float32 result that lands on the other side of a bfloat16
rounding boundary moves the next product's operand by one bfloat16 ulp (2^-8
relative), so an entry may be off by a few such ulps of the sum of its
products' magnitudes, per layer passed through."""
import numpy as np
import pytest

from oracle import mlp as ref
from paper_1605_01421_amd import workloads as W

pytestmark = pytest.mark.gpu

PROBS = (0.1, 0.5, 0.9)


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    from paper_1605_01421_amd import siminf
    siminf.load()
    return siminf


def _inputs(dims, B, seed):
    rng = np.random.default_rng(seed)
    params = [(Wl, rng.normal(scale=0.1, size=b.shape)) for Wl, b in W.mlp_init(dims, seed)]
    rparams = [(ref.bf16(Wl), b.astype(np.float32).astype(np.float64)) for Wl, b in params]
    X = rng.normal(size=(B, dims[0])).astype(np.float32)
    T = rng.normal(scale=0.5, size=(B, dims[-1])).astype(np.float32)
    return params, rparams, X, T


@pytest.mark.parametrize("dims,B", [
    ((8, 256, 256, 256, 256, 156), 1), ((8, 256, 256, 256, 256, 156), 129), ((8, 256, 256, 256, 256, 156), 1025),
    ((8, 256, 256, 256, 256, 156), 17000),
    ((1, 1), 1), ((256, 256), 33), ((255, 17, 31), 16), ((3, 16, 33, 32, 5), 15), ((33, 130, 64, 3), 300),
    ((8, 257, 40), 70)])
def test_passes_match_oracle(lib, dims, B):
    import torch
    print("[gpu] fused mlp", dims, B, flush=True)
    params, rparams, X, T = _inputs(dims, B, 21)
    net = lib.MLP(dims, B)
    net.set_params(params)
    Xt, Tt = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    Y = net.forward(Xt).cpu().numpy().astype(np.float64)
    X64, T64 = X.astype(np.float64), T.astype(np.float64)
    want, (A, Z) = ref.forward(rparams, X64, round_bf16=True)
    L = len(rparams)
    scale = np.abs(A[L - 1]) @ np.abs(rparams[L - 1][0]).T + np.abs(rparams[L - 1][1])
    bound = 4 * 2.0 ** -8 * scale + 1e-6 * scale.max()
    assert np.all(np.abs(Y - want) <= bound), float(np.max(np.abs(Y - want) / bound))
    loss = net.backward(Xt, Tt, PROBS)
    # the loss has a kink at Y = T: the reference takes the slope at the
    # network's own outputs (checked above), so that both are on one side
    wl, dY = ref.pinball(Y, T64, PROBS)
    assert abs(loss - wl) <= 1e-6 * wl
    wgrads = ref.backward(rparams, (A, Z), dY, round_bf16=True)
    dz = np.abs(dY)
    scales = [None] * L
    for l in range(L - 1, -1, -1):
        scales[l] = (dz.T @ np.abs(A[l]), dz.sum(axis=0))
        if l > 0:
            dz = (dz @ np.abs(rparams[l][0])) * np.abs(ref.gelu_grad(Z[l - 1]))
    for l, ((gW, gb), (rW, rb)) in enumerate(zip(net.get_grads(), wgrads)):
        for got, exp, sc in ((gW, rW, scales[l][0]), (gb, rb, scales[l][1])):
            tol = 4 * (L - l) * 2.0 ** -8 * sc + 1e-6 * sc.max()
            assert np.all(np.abs(got.astype(np.float64) - exp) <= tol), (l, float(np.max(np.abs(got - exp) / tol)))
    net.close()


@pytest.mark.parametrize("widths", [(256, 256), (300, 256)])
def test_ensemble_of_networks_in_slices(lib, widths):
    """Members of different hidden widths (one may be too wide for the fused
    kernels) and largest batches, in slices, equal their single passes."""
    import torch
    nets, B = [], 150
    for k, w in enumerate(widths):
        dims = (8, w, 20)
        net = lib.MLP(dims, 64 + 40 * k)
        net.set_params(_inputs(dims, 1, 5 + k)[0])
        nets.append(net)
    X = torch.randn((B, 8), generator=torch.Generator().manual_seed(4)).cuda()
    mean, std = torch.zeros(20).cuda(), torch.ones(20).cuda()
    Y, dis = lib.ensemble_predict(nets, X, mean, std)
    P = []
    for net in nets:
        P.append(torch.cat([net.forward(X[i:i + net.max_batch].contiguous()) for i in range(0, B, net.max_batch)]))
    P = torch.stack(P).double()
    assert torch.equal(Y, P.mean(0).float())
    assert torch.allclose(dis.double(), P.std(0, unbiased=True).mean(1), rtol=1e-6, atol=0)
    for net in nets:
        net.close()


@pytest.mark.parametrize("B", [3, 200, 700, 1500, 9000])
@pytest.mark.parametrize("spread", [0.02, 1.0, 12.0])
def test_fused_and_general_kernels_agree_bit_for_bit(lib, B, spread):
    """The fused kernels settle most activations from a cheap GELU, the
    general ones evaluate it.  A network one unit too wide for the fused
    kernels whose extra units have zero weights is the same function, with the
    same products in the same order: outputs must be equal bit for bit, and
    so must the weight gradients of batches that both reduce in one pass,
    for pre-activations from tiny to far beyond the cheap range, and zero."""
    import torch
    rng = np.random.default_rng(31)
    widths = (8, 256, 256, 40)
    params = [(spread * Wl, spread * rng.normal(scale=0.3, size=b.shape)) for Wl, b in W.mlp_init(widths, 9)]
    wide = []
    for l, (Wl, b) in enumerate(params):
        out, inp = Wl.shape
        Wx = np.zeros((out + (l < 2), inp + (l > 0)))
        Wx[:out, :inp] = Wl
        wide.append((Wx, np.append(b, 0.0) if l < 2 else b))
    X = rng.normal(size=(B, 8)).astype(np.float32)
    X[rng.random((B, 8)) < 0.1] = 0.0
    Xt = torch.from_numpy(X).cuda()
    T = torch.from_numpy(rng.normal(size=(B, 40)).astype(np.float32)).cuda()
    a, g = lib.MLP(widths, B), lib.MLP((8, 257, 257, 40), B)
    a.set_params(params)
    g.set_params(wide)
    assert torch.equal(a.forward(Xt), g.forward(Xt))
    la, lg = a.backward(Xt, T, PROBS), g.backward(Xt, T, PROBS)
    assert abs(la - lg) <= 1e-12 * abs(lg)
    if B <= 256:
        for (Wa, _), (Wg, _) in zip(a.get_grads(), g.get_grads()):
            assert np.array_equal(Wa, Wg[:Wa.shape[0], :Wa.shape[1]])
    a.close()
    g.close()
