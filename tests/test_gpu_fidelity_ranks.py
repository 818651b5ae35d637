"""F_q against rank-r targets at the edges of the eigenvalue kernel's forms (one
wave up to r = 16, four above; odd ranks carry a padding index), against the
nuclear norm of W^dagger T: F_q = ||W^dagger T||_*^2 / (|T|^2 |W|^2).

Tolerance: FP64 sums of d^2 terms and an eigensolver to 1e-15 of the trace,
relative 1e-12 as the path's other FP64 results.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e-90, 1e60])
@pytest.mark.parametrize("r", [1, 2, 3, 7, 8, 15, 16, 17, 31, 32])
def test_fidelity_rank_edges(r, scale):
    print(f"fidelity r={r} scale={scale}", flush=True)
    g = np.random.default_rng(700 + r)
    d = 64
    T = g.standard_normal((d, d)) + 1j * g.standard_normal((d, d))
    W = scale * (g.standard_normal((d, r)) + 1j * g.standard_normal((d, r)))
    F = qst.fidelity_lowrank(torch.from_numpy(T).cuda(), torch.from_numpy(W).cuda(), "f64")
    sv = np.linalg.svd((W / scale).conj().T @ T, compute_uv=False)
    want = sv.sum() ** 2 / (np.linalg.norm(T) ** 2 * np.linalg.norm(W / scale) ** 2)
    assert abs(float(F) - want) <= 1e-12 * want
