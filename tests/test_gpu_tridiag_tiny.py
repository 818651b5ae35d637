"""The tridiagonal reduction on columns whose squared norms are subnormal: a
matrix of entries near 1e-156, and one whose off-diagonal entries are, through
the eigensolver and the absolute map they feed.

Tolerance: squares near 1e-312 are rounded by 2^-1075, up to 5e-12 of a term, so
a reflector is unitary to a few 1e-12 and d of them to less than 1e-9 (d = 256).
"""
import pytest

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("kind", ["all", "off-diagonal"])
@pytest.mark.parametrize("n", [3, 5, 7, 8])
def test_subnormal_squares(n, kind):
    print(f"tiny columns n={n} {kind}", flush=True)
    d = 1 << n
    X = torch.randn(d, d, dtype=torch.complex128, generator=torch.Generator().manual_seed(700 + n))
    H = (X + X.mH) / 2
    scale = 1e-156 if kind == "all" else 1.0
    T = H * 1e-156
    if kind == "off-diagonal":
        T = T + torch.diag(torch.linspace(1, 2, d, dtype=torch.float64)).to(T.dtype)
    lam, V = torch.linalg.eigh(T / scale)
    want = (V * lam.abs()) @ V.mH
    A, Q, got, sweeps = qst.abs_map(T.to(DEV), 2.0, "f64")
    assert sweeps == 0
    assert float((A.cpu() / scale - want).norm() / want.norm()) <= 1e-9
    got = (got.cpu() / scale).sort().values
    assert float((got - lam).abs().max()) <= 1e-9 * float(lam.abs().max())
    Q = Q.cpu()
    assert float((Q.mH @ Q - torch.eye(d, dtype=Q.dtype)).abs().max()) <= 1e-9
