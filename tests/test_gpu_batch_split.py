"""The split products of the batched kernel (FP32, 512 threads, d = 128 and
256) on operands with scaled or zero rows and columns, very small or large,
or not finite, mixed with instances below that size, for the tetrahedral and
a general POVM; every instance against the FP64 oracle of the same FP32 data.

Tolerance: 1e-5 relative (L; gradient by Frobenius norm), that of the FP32
path elsewhere.  Frequencies are uniform on [0.5, 1.5), and the rows' and
columns' scales within 2^+-2 of one another, so that no p is so small that
f / p multiplies rho's rounding errors beyond it.
"""
import numpy as np
import pytest

import oracle as O
import synth as S
from workloads import rel_fro

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [7, 3, 8, 7, 6, 8, 1]


def instance(g, n, pattern):
    d = 1 << n
    T = S.ginibre(g, d)
    s = 2.0 ** g.integers(-2, 3, size=d)
    if pattern == "rows":
        T = s[:, None] * T
    elif pattern == "columns":
        T = T * s[None, :]
    elif pattern == "zeros":
        T[d // 3] = 0
        T[:, d // 5] = 0
        T[g.random((d, d)) < 0.3] = 0
    elif pattern == "tiny":
        T = 2.0 ** -40 * T
    elif pattern == "large":
        T = 2.0 ** 40 * T
    return T.astype(np.complex64), g.uniform(0.5, 1.5, size=d * d).astype(np.float32)


def forced_plan(tmp_path, povm, Ts, fs):
    """A plan with 512 threads, whatever the autotuner finds faster."""
    cache = tmp_path / "tune.txt"
    plan = qst.BatchPlan(SHAPES, "f32", povm=povm, tune_cache=str(cache))
    plan.run(*plan.pack(Ts, fs, DEV), use_graph=False)
    torch.cuda.synchronize()
    plan.close()
    key, grid = cache.read_text().split()[:2]
    with open(cache, "a") as fh:
        fh.write(f"{key} {grid} 1 0.0 512 1\n")
    plan = qst.BatchPlan(SHAPES, "f32", povm=povm, tune_cache=str(cache))
    assert plan.info()["threads"] == 512
    return plan


def general_povm():
    U, _ = np.linalg.qr(S.ginibre(S.rng(71), 2))
    return np.array([U @ m @ U.conj().T for m in O.tetrahedral_povm()])


@pytest.mark.parametrize("general", [False, True])
@pytest.mark.parametrize("pattern", ["plain", "rows", "columns", "zeros", "tiny", "large"])
def test_batch_split_products(tmp_path, pattern, general):
    print(f"batched split products: {pattern}, general POVM {general}", flush=True)
    g = S.rng(70)
    Ts, fs = zip(*[instance(g, n, pattern) for n in SHAPES])
    M = general_povm() if general else None
    plan = forced_plan(tmp_path, M, Ts, fs)
    nll, grad, bad = plan.run(*plan.pack(Ts, fs, DEV), use_graph=False)
    torch.cuda.synchronize()
    nll, grad = nll.cpu().numpy(), grad.cpu().numpy()
    assert (bad.cpu().numpy() == 0).all()
    for i, n in enumerate(SHAPES):
        T, f = Ts[i].astype(np.complex128), fs[i].astype(np.float64)
        rho, tau = O.state_map(T)
        Mi = O.tetrahedral_povm() if M is None else M
        p = O.probs_real(rho, Mi)
        L = O.nll_vec(p, f)
        want = (2.0 / tau) * (O.adjoint(O.cotangent(p, f), n, Mi) @ T)
        got = grad[plan.t_off[i]:plan.t_off[i + 1]].reshape(T.shape)
        assert abs(nll[i, 0] - L) <= 1e-5 * abs(L), i
        assert rel_fro(got, want) <= 1e-5, i
    plan.close()


@pytest.mark.parametrize("bad_value", [float("nan"), float("inf")])
def test_batch_split_not_finite(tmp_path, bad_value):
    """A value that is not finite spoils its own instance and no other."""
    print(f"batched split products: {bad_value}", flush=True)
    g = S.rng(72)
    Ts, fs = map(list, zip(*[instance(g, n, "plain") for n in SHAPES]))
    plan = forced_plan(tmp_path, None, Ts, fs)
    nll, grad, _ = plan.run(*plan.pack(Ts, fs, DEV), use_graph=False)
    Ts[2] = Ts[2].copy()
    Ts[2][17, 40] = bad_value
    nll2, grad2, _ = plan.run(*plan.pack(Ts, fs, DEV), use_graph=False)
    torch.cuda.synchronize()
    assert not np.isfinite(nll2[2, 0].item())
    for i in range(len(SHAPES)):
        a, b = plan.t_off[i], plan.t_off[i + 1]
        if i == 2:
            assert not bool(torch.isfinite(torch.view_as_real(grad2[a:b])).all())
        else:
            assert torch.equal(nll[i], nll2[i]) and torch.equal(grad[a:b], grad2[a:b])
    plan.close()
