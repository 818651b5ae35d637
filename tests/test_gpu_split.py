"""The split products (two fp16 parts per FP32 value, power-of-two scales per
row and column) against FP64 on operands whose rows and columns differ by
many binades, hold zeros, or are not finite.

Tolerance, entry by entry: 2^-17 of sum_k |a_ik| |b_kj| (|z| = |re| + |im|),
the largest that the accumulation alone can lose: a chain of 16 panels adds
64 product blocks, each add rounding toward zero by at most 2^-23 of the
chain's absolute sum; the split, the dropped ll products and the final
roundings are below 2^-20 of it.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def operand(d, seed, pattern, pad):
    g = np.random.default_rng(seed)
    x = g.standard_normal((d, d)) + 1j * g.standard_normal((d, d))
    s = 2.0 ** g.integers(-30, 31, size=d)
    if pattern == "rows":
        x = s[:, None] * x
    elif pattern == "columns":
        x = x * s[None, :]
    elif pattern == "zeros":
        x[d // 3] = 0
        x[:, d // 5] = 0
        x[g.random((d, d)) < 0.3] = 0
    elif pattern == "tiny":
        x = 2.0 ** -55 * x
    elif pattern == "large":
        x = 2.0 ** 50 * x
    big = torch.zeros((d, d + pad), dtype=torch.complex64, device=DEV)
    big[:, :d] = torch.from_numpy(x.astype(np.complex64)).to(DEV)
    return big[:, :d]


def abs1(x):
    return x.real.abs() + x.imag.abs()


@pytest.mark.parametrize("pattern", ["plain", "rows", "columns", "zeros", "tiny", "large"])
@pytest.mark.parametrize("n,pad", [(7, 1), (8, 0), (10, 3), (11, 0), (12, 0)])
def test_split_products_entrywise(n, pad, pattern):
    print(f"split products n={n} pad={pad} {pattern}", flush=True)
    d = 1 << n
    T = operand(d, 100 + n, pattern, pad)
    A = operand(d, 200 + n, pattern if pattern in ("rows", "zeros") else "plain", pad)
    G = (A + A.mH).contiguous()
    T64, G64 = T.to(torch.complex128).contiguous(), G.to(torch.complex128)
    tol = 2.0 ** -17
    rho, tau = qst.state_map(T, "f32x6")
    tau64 = T64.abs().square().sum()
    want = (T64 @ T64.mH.contiguous()) / tau64
    bound = (abs1(T64) @ abs1(T64).T.contiguous()) / tau64
    assert abs(float(tau) / float(tau64) - 1) < 1e-12
    assert bool(((rho.to(torch.complex128) - want).abs() <= tol * bound + 2.0 ** -126).all())
    grad = qst.grad_product(G, T, tau, "f32x6")
    want = (G64 @ T64) * (2 / tau64)
    bound = (abs1(G64) @ abs1(T64)) * (2 / tau64)
    assert bool(((grad.to(torch.complex128) - want).abs() <= tol * bound + 2.0 ** -126).all())


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_split_products_not_finite(bad):
    """A non-finite entry of T reaches every entry of its row of rho and of
    its column of the gradient, and nothing else stays hidden."""
    print(f"split products with {bad}", flush=True)
    d, r, c = 256, 37, 201
    T = operand(d, 300, "plain", 0).contiguous()
    G = operand(d, 301, "plain", 0)
    G = (G + G.mH).contiguous()
    tau = torch.tensor(1.0, dtype=torch.float64, device=DEV)
    T[r, c] = bad
    grad = qst.grad_product(G, T, tau, "f32x6")
    fin = torch.isfinite(grad.real) & torch.isfinite(grad.imag)
    assert not bool(fin[:, c].any())
    assert bool(fin[:, :c].all()) and bool(fin[:, c + 1:].all())
    rho, _ = qst.state_map(T, "f32x6")
    fin = torch.isfinite(rho.real) & torch.isfinite(rho.imag)
    assert not bool(fin[r].any()) and not bool(fin[:, r].any())
