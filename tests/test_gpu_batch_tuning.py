"""The batched kernel's tuning: the products of a QST_F32 plan with d >= 128 do
not depend on a timing, and a cache line of earlier kernels is passed over."""
import numpy as np
import pytest

import synth as S

torch = pytest.importorskip("torch")
qst = pytest.importorskip("paper_2207_05341_amd")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def tuned(shapes, cache):
    g = S.rng(74)
    Ts = [S.ginibre(g, 1 << n).astype(np.complex64) for n in shapes]
    fs = [g.uniform(0.5, 1.5, size=4 ** n).astype(np.float32) for n in shapes]
    plan = qst.BatchPlan(shapes, "f32", tune_cache=str(cache))
    plan.run(*plan.pack(Ts, fs, DEV), use_graph=False)
    torch.cuda.synchronize()
    info = plan.info()
    plan.close()
    return info


@pytest.mark.parametrize("shapes", [[7] * 4, [8, 3, 7]])
def test_earlier_kernels_lines_are_passed_over(tmp_path, shapes):
    print(f"tuning cache {shapes}", flush=True)
    first = tmp_path / "a.txt"
    assert tuned(shapes, first)["threads"] == 512
    key, grid = first.read_text().split()[:2]
    second = tmp_path / "b.txt"
    second.write_text(f"{key[key.index('prec'):]} {grid} 1 0.0 256 1\n")
    assert tuned(shapes, second)["threads"] == 512
    assert len(second.read_text().splitlines()) == 2  # tuned anew, and noted
    assert tuned(shapes, second)["threads"] == 512
    assert len(second.read_text().splitlines()) == 2  # the new line is taken
