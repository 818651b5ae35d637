"""The tridiagonal reduction's forms -- the last 96 columns in one workgroup,
one launch per column up to d = 2048, and beyond -- through the eigensolver
they feed: H = Q diag(lam) Q^dagger at the sizes around their borders, for
dense matrices, block-diagonal ones (columns that need no reflector) and ones
of low rank.

Tolerances: d 2^-50 of ||H||_F for the reconstruction (a reduction by d
reflectors, each with a rounding error of a few 2^-53 of ||H||), no less than
1e-13; 1e-13 d for an entry of Q^dagger Q - I, as in test_gpu_absmap.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def hermitian(d, kind):
    g = torch.Generator().manual_seed(900 + d)
    X = torch.randn(d, d, dtype=torch.complex128, generator=g)
    if kind == "blocks":
        size = max(d // 4, 1)
        r = torch.arange(d) // size
        X = torch.where(r[:, None] == r[None, :], X, torch.zeros((), dtype=X.dtype))
    elif kind == "low rank":
        k = max(d // 8, 1)
        Y = X[:, :k].contiguous().to(DEV)
        return Y @ Y.mH.contiguous()
    X = X.to(DEV)
    return 0.5 * (X + X.mH)


@pytest.mark.parametrize("kind", ["dense", "blocks", "low rank"])
@pytest.mark.parametrize("n", [1, 2, 4, 6, 7, 9, 11])
def test_reduction_forms(n, kind):
    check(n, kind)


def test_reduction_beyond_2048():
    check(12, "dense")


def check(n, kind):
    print(f"tridiagonal reduction n={n} {kind}", flush=True)
    d = 1 << n
    H = hermitian(d, kind)
    _, Q, lam, sweeps = qst.abs_map(H, 2.0, "f64")
    assert sweeps == 0
    tol = max(1e-13, d * 2.0 ** -50)
    back = (Q * lam[None, :]) @ Q.mH.contiguous()
    assert float((back - H).norm()) <= tol * float(H.norm())
    eye = torch.eye(d, dtype=Q.dtype, device=DEV)
    assert float((Q.mH.contiguous() @ Q - eye).abs().max()) <= 1e-13 * d
    assert abs(float(lam.sum()) - float(torch.diagonal(H).real.sum())) <= tol * float(H.norm()) * np.sqrt(d)
