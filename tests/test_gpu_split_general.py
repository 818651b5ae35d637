"""The split products on operands that their fp16 form does not suit: a few
terms carrying an entry (one or four nonzero columns), zeros (triangular T), and
large entries of one operand meeting small ones of the other (T = D^-1 X with
G' = D A D, D within 2^+-12).  Each precision against FP64.

Tolerances.  One or four columns, QST_F32, entry by entry: each of re and im
is a sum of 2 and 8 products; one rounding each, at most, for the product and
its addition, the scale and the result, 2^-24 of the absolute sum: 4 and 10
units of it, times sqrt 2 for the modulus.  A last column 2^7 above the rest: an
entry is the last term added, so two roundings of 2^-24, 2^-23.  Otherwise the relative Frobenius
error: K terms of random sign rounded (FP32) or truncated (bf16 MFMA, six
products, three real products per complex one) at every step lose at most
about 2^-24 sqrt(K) = 2^-18.5 at K = 2048; 2^-19 is between that bound and
the 2^-20.5 of random rounding.  The fp16 split loses 2^-16 with D within
2^+-12, entries there being 2^-20 of their row's largest on the mean.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def ginibre(g, d):
    return g.standard_normal((d, d)) + 1j * g.standard_normal((d, d))


def operands(n, pattern):
    g, d = np.random.default_rng(1000 + n), 1 << n
    T, A = ginibre(g, d), ginibre(g, d)
    if pattern.startswith("columns"):
        T[:, int(pattern[7:]):] = 0
    elif pattern == "lower":
        T = np.tril(T)
    elif pattern == "opposing":
        D = 2.0 ** g.integers(-12, 13, size=d)
        T, A = T / D[:, None], D[:, None] * A * D[None, :]
    elif pattern == "last":  # one column far above the rest, in last place
        T[:, -1] *= 2.0 ** 7
    elif pattern == "mixed":  # G' dense, T not
        T[d // 2:] *= 2.0 ** -12
    T, G = T.astype(np.complex64), (A + A.conj().T).astype(np.complex64)
    return torch.from_numpy(T).to(DEV), torch.from_numpy(G).to(DEV)


def fro(got, want):
    return float((got.to(torch.complex128) - want).norm() / want.norm())


def abs1(x):
    return x.real.abs() + x.imag.abs()


CASES = [(n, "f32x6") for n in (7, 8, 9, 10, 11)] + [(n, "f32") for n in (8, 10, 11)]


@pytest.mark.parametrize("pattern", ["columns1", "columns4", "lower", "opposing", "mixed", "last"])
@pytest.mark.parametrize("n,prec", CASES)
def test_products_of_operands_that_are_not_dense(n, prec, pattern):
    print(f"products n={n} {prec} {pattern}", flush=True)
    T, G = operands(n, pattern)
    T64, G64 = T.to(torch.complex128), G.to(torch.complex128)
    rho, tau = qst.state_map(T, prec)
    tau64 = T64.abs().square().sum()
    want = (T64 @ T64.mH.contiguous()) / tau64
    assert abs(float(tau) / float(tau64) - 1) < 1e-12
    assert fro(rho, want) <= 2.0 ** -19
    if prec == "f32" and pattern.startswith("columns"):
        units = 4 if pattern == "columns1" else 10
        bound = (abs1(T64) @ abs1(T64).T.contiguous()) / tau64
        assert bool(((rho.to(torch.complex128) - want).abs() <= units * 2.0 ** -23.5 * bound).all())
    if prec == "f32" and pattern == "last":
        assert fro(rho, want) <= 2.0 ** -23
    grad = qst.grad_product(G, T, tau, prec)
    assert fro(grad, (G64 @ T64) * (2 / tau64)) <= 2.0 ** -19


@pytest.mark.parametrize("n,prec", [(7, "f32x6"), (10, "f32x6"), (11, "f32x6"), (10, "f32"), (11, "f32")])
def test_one_call_equals_two_on_both_kinds(n, prec):
    """The combined call equals its two stages bitwise and FP64 within the FP32
    path's 1e-5, whichever products run, and in a captured call the replay's
    inputs decide."""
    print(f"one call n={n} {prec}", flush=True)
    g, d = np.random.default_rng(2000 + n), 1 << n
    f = torch.from_numpy(g.uniform(0.5, 1.5, size=d * d).astype(np.float32)).to(DEV)
    x = ginibre(g, d)
    inputs = {k: torch.from_numpy(v.astype(np.complex64)).to(DEV)
              for k, v in (("dense", x), ("lower", np.tril(x)), ("column", x * (np.arange(d) == 3)[None, :]))}
    want = {}
    for k, T in inputs.items():
        out, tau, grad, _ = qst.likelihood_grad(T, f, prec)
        Tr = T.clone().requires_grad_(True)
        loss = qst.likelihood(Tr, f, prec)
        two, = torch.autograd.grad(loss, Tr)
        assert torch.equal(grad, two) and torch.equal(out[0], loss.detach())
        if k != "column":  # its rho is pure: p runs into rounding
            out64, _, grad64, _ = qst.likelihood_grad(T.to(torch.complex128), f.double(), "f64")
            assert abs(float(out[0]) / float(out64[0]) - 1) < 1e-6
            assert fro(grad, grad64) <= 1e-5
        want[k] = (out.clone(), grad.clone())
    T = inputs["dense"].clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        qst.likelihood_grad(T, f, prec)
    torch.cuda.current_stream().wait_stream(s)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out, _, grad, _ = qst.likelihood_grad(T, f, prec)
    for k in ("lower", "dense", "column", "dense", "lower"):
        T.copy_(inputs[k])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(grad.view(torch.float32), want[k][1].view(torch.float32)), k
        assert torch.equal(out, want[k][0]) or k == "column", k
