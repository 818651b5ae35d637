"""The batched kernel (FP32, d = 128 and 256) on instances whose T is not
dense: the 512-thread form has to take the FP32 tiles for them, as the
256-thread form does for every instance, next to dense instances of the same
plan.

Tolerance between the two forms where both take FP32 tiles: 2^-26 of the
gradient's norm.  They run the same products in the same order; tau, an FP64
sum in another order, moves a single-precision result by a rounding at
most, and that in about one of 10^8 values.  (The split products differ from
FP32 tiles by more than 2^-24.)  With the columns of T graded its rows are not
dense but its columns are, so T T^dagger alone takes FP32 tiles and the two
forms differ in G' T.  Against the FP64 oracle: 1e-5, the FP32 path's.
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
SHAPES = [7, 8, 3, 8, 7]
DENSE = (3, 4)  # instances that stay dense


def instance(g, i, n, pattern):
    d = 1 << n
    T = S.ginibre(g, d)
    if i not in DENSE:
        if pattern == "columns":
            T[:, 6:] = 0
        elif pattern == "lower":
            T = np.tril(T)
        elif pattern == "zeros":
            T[g.random((d, d)) < 0.5] = 0
        elif pattern == "graded":
            T = T * 2.0 ** (-12.0 * np.arange(d) / d)[None, :]
    return T.astype(np.complex64), g.uniform(0.5, 1.5, size=d * d).astype(np.float32)


def plan_with(tmp_path, threads, Ts, fs):
    cache = tmp_path / f"tune{threads}.txt"
    plan = qst.BatchPlan(SHAPES, "f32", tune_cache=str(cache))
    plan.run(*plan.pack(Ts, fs, DEV), use_graph=False)
    torch.cuda.synchronize()
    plan.close()
    key, grid = cache.read_text().split()[:2]
    with open(cache, "a") as fh:
        fh.write(f"{key} {grid} 1 0.0 {threads} 1\n")
    plan = qst.BatchPlan(SHAPES, "f32", tune_cache=str(cache))
    assert plan.info()["threads"] == threads
    return plan


@pytest.mark.parametrize("pattern", ["columns", "lower", "zeros", "graded"])
def test_batch_instances_that_are_not_dense(tmp_path, pattern):
    print(f"batched instances not dense: {pattern}", flush=True)
    g = S.rng(73)
    Ts, fs = zip(*[instance(g, i, n, pattern) for i, n in enumerate(SHAPES)])
    got = {}
    for threads in (512, 256):
        plan = plan_with(tmp_path, threads, Ts, fs)
        _, grad, bad = plan.run(*plan.pack(Ts, fs, DEV), use_graph=False)
        torch.cuda.synchronize()
        assert (bad.cpu().numpy() == 0).all()
        off = plan.t_off
        got[threads] = grad.cpu().numpy()
        plan.close()
    for i, n in enumerate(SHAPES):
        T, f = Ts[i].astype(np.complex128), fs[i].astype(np.float64)
        a, b = (got[k][off[i]:off[i + 1]].reshape(T.shape) for k in (512, 256))
        if i not in DENSE and pattern != "graded":
            assert rel_fro(a, b) <= 2.0 ** -26, i
        rho, tau = O.state_map(T)
        want = (2.0 / tau) * (O.adjoint(O.cotangent(O.probs_real(rho), f), n) @ T)
        assert rel_fro(a, want) <= 1e-5, i
