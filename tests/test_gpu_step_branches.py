"""Time steps of the first-order scheme and of one-level solvers: the load vector at the
Gauss points and the operator evaluated per cell, against the stored blocks."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, rel, say, torch
from paper_2602_16312_amd import api, problem
from workloads import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("bdf", [1, 2])
@pytest.mark.parametrize("name,kw,form", [
    ("c2", dict(n=17, p=3, jitter=0.1, group=[17]), "mapped"), ("c2", dict(n=17, p=1, jitter=0.1, group=[17]), "hybrid"),
    ("c3", dict(n=7, jitter=0.1, seed=3, penalty=("paper", 2.0), group=[7]), "mapped"),
    ("e1", dict(n=9, p=4, group=[3]), "box"), ("e1", dict(n=9, p=2, group=[]), "box"), ("e1", dict(n=5, p=4, group=[]), "box"),
    ("c3", dict(n=3, group=[]), "box"), ("c3", dict(n=3, p=3, group=[]), "box")])
def test_steps_match_blocks(name, kw, form, bdf):
    pr = make_problem(name, **kw)
    rng = np.random.default_rng(6)
    U = [rng.uniform(0.0, 1.0, pr["N"]) for _ in range(2)]
    W = [rng.uniform(0.2, 0.8, pr["S"] * pr["N"]) for _ in range(2)]
    for prec, tol in (("fp64", 1e-10), ("mixed", 1e-9)):   # the time series' bound; solves to 1e-12 either way
        out = []
        for layout in ("axis_ell", "auto"):
            h, s = problem.build(pr, precision=prec, fine_layout=layout, bdf=bdf)
            assert s.forms()["level_form"][0] == (form if layout == "auto" else "axis_ell_sparse")
            st = api.State(dev(U[0]), dev(U[1]), dev(W[0]), dev(W[1]), torch.empty(pr["N"], dtype=torch.float64, device="cuda"))
            say("step branches", name, kw, bdf, prec, layout)
            for k in range(2):
                assert api.time_step(s, st, pr["dt"], iapp=dev(np.full(pr["N"], 0.1)), tol=1e-12)["converged"]
            out.append((host(st.U), host(st.W)))
        assert rel(out[1][0], out[0][0]) <= tol, prec
        assert rel(out[1][1], out[0][1]) <= tol, prec
