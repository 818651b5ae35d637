"""The one-launch likelihood of small states (N = 1 .. 5) and its neighbour
N = 6 against the oracle: both storage precisions, a rotated POVM, padded T and
G, no gradient, F_c, f = 0 and p <= 0 entries.

Tolerances (relative): FP64 1e-12, FP32 1e-5, as the path's other tests.
"""
import numpy as np
import pytest

import oracle as O
import synth as S
from workloads import rel_fro

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5, "f32x6": 1e-5}


@pytest.mark.parametrize("rotated", [False, True])
@pytest.mark.parametrize("prec", ["f64", "f32", "f32x6"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6])
def test_small_likelihood(n, prec, rotated):
    print(f"small likelihood n={n} {prec} rotated={rotated}", flush=True)
    g = S.rng(8800 + n)
    d = 1 << n
    ct, rt = (np.complex128, np.float64) if prec == "f64" else (np.complex64, np.float32)
    povm = None
    M = O.tetrahedral_povm()
    if rotated:
        U, _ = np.linalg.qr(S.ginibre(g, 2))
        M = povm = np.array([U @ m @ U.conj().T for m in M])
    T = S.ginibre(g, d).astype(ct)
    f = S.multinomial_freqs(g, 2 * 4 ** n, S.porter_thomas_probs(g, 4 ** n, 0.1)).astype(rt)  # zeros among them
    pt = S.porter_thomas_probs(g, 4 ** n, 0.2).astype(rt)
    big = torch.zeros((d, d + 3), dtype=torch.complex128 if prec == "f64" else torch.complex64, device="cuda")
    big[:, :d] = torch.from_numpy(T)
    Tg, fg = big[:, :d], torch.from_numpy(f).cuda()
    out, tau, G, bad = qst.likelihood_forward(Tg, fg, prec, povm)
    out1, tau1, G1, bad1 = qst.likelihood_forward(Tg, fg, prec, povm, with_grad_matrix=False)
    out2, tau2, G2, bad2, fc = qst.likelihood_forward_fc(Tg, fg, torch.from_numpy(pt).cuda(), prec, povm)
    _, _, grad, _ = qst.likelihood_grad(Tg, fg, prec, povm)
    torch.cuda.synchronize()
    Tq, fq = T.astype(np.complex128), f.astype(np.float64)
    rho, wtau = O.state_map(Tq)
    povms = np.array([M] * n)
    p = O.probs_real(rho, povms)
    wL = O.nll_vec(p, fq)
    wG = O.adjoint(O.cotangent(p, fq), n, povms)
    assert abs(float(out[0]) - wL) <= TOL[prec] * abs(wL)
    assert abs(float(out[1]) - fq.sum()) <= 1e-12 and abs(float(tau) - wtau) <= 1e-12 * wtau
    assert rel_fro(G.cpu().numpy(), wG) <= TOL[prec]
    assert rel_fro(grad.cpu().numpy(), 2 / wtau * (wG @ Tq)) <= TOL[prec]
    wfc = np.sqrt(np.clip(p, 0, None) * pt.astype(np.float64)).sum() ** 2
    assert abs(float(fc) - wfc) <= TOL[prec] * wfc
    assert bad.tolist() == [0, 0] and G1 is None
    assert torch.equal(out, out1) and torch.equal(tau, tau1) and torch.equal(bad, bad1)
    assert torch.equal(tau, tau2) and torch.equal(bad, bad2) and rel_fro(G2.cpu().numpy(), wG) <= TOL[prec]


@pytest.mark.parametrize("n", [2, 5])
def test_small_likelihood_bad_entries(n):
    print(f"small likelihood, bad entries n={n}", flush=True)
    d = 1 << n
    M = np.zeros((4, 2, 2), dtype=np.complex128)  # two outcomes of the Z basis, each split in halves
    M[0, 0, 0] = M[1, 0, 0] = M[2, 1, 1] = M[3, 1, 1] = 0.5
    T = torch.zeros((d, d), dtype=torch.complex128, device="cuda")
    T[0, 0] = 1.0
    f = torch.zeros(4 ** n, dtype=torch.float64, device="cuda")
    f[0], f[-1], f[2] = 0.5, 0.25, 0.25  # the last two have p = 0
    out, _, _, bad = qst.likelihood_forward(T, f, "f64", M)
    assert float(out[0]) == np.inf and float(out[1]) == 1.0 and bad.tolist() == [2, 0]
    f[1] = float("nan")
    out, _, _, bad = qst.likelihood_forward(T, f, "f64", M)
    assert np.isnan(float(out[0])) and int(bad[1]) == 1
