"""Small levels of Q4 boxes, a lane per row: operator rows against the oracle (random
full conductivities), and V-cycles through every epilogue against the row kernels."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, rel, say, torch
from oracle.assemble import assemble
from paper_2602_16312_amd import api, problem
from workloads import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def boxes(n, group):
    pr = make_problem("e1", n=n, p=4, group=group)
    xx, yy = np.random.default_rng(8).uniform(0.05, 0.2, (2, pr["n_cells"]))
    xy = np.random.default_rng(9).uniform(-0.9, 0.9, pr["n_cells"]) * np.sqrt(xx * yy)
    return {**pr, "D_cell": np.stack([xx, xy, yy], axis=1)}


# 9, 16, 25, 2,025 cells (a lane per row, groups of 8, ragged), 4,096 and 4,225 (the last by cells)
@pytest.mark.parametrize("n", [3, 4, 5, 45, 64, 65])
def test_rows_match_oracle(n):
    pr = boxes(n, [n])
    nc, b = pr["n_cells"], pr["b"]
    scale = np.random.default_rng(3).uniform(0.5, 2.0, nc)
    h, s = problem.build(pr, precision="mixed", cell_scale=scale)
    assert s.forms()["level_form"][0] == "box"
    cells = np.unique(np.concatenate([[0, 7, 8, nc - 1, nc - 2], np.random.default_rng(4).integers(0, nc, 24)]) % nc)
    M, A = assemble(pr, scale, row_cells=cells)
    rows = (cells[:, None] * b + np.arange(b)).ravel()
    x = np.random.default_rng(5).standard_normal(pr["N"])
    ref = ((1.5 * pr["chi"] * pr["Cm"] / pr["dt"]) * M + A)[rows] @ x
    y = torch.empty(pr["N"], dtype=torch.float64, device="cuda")
    for prec, tol in (("fp64", 1e-13), ("mixed", 3e-6)):   # as for the other forms
        say("row boxes", n, prec)
        api.apply(s, 0, dev(x), y, prec)
        assert rel(host(y)[rows], ref) <= tol, prec


@pytest.mark.parametrize("mg", [dict(), dict(cheb_degree=1), dict(jacobi="cell_block"),
                                dict(cheb_degree=1, jacobi="cell_block")])
@pytest.mark.parametrize("n,group", [(3, [3]), (4, [2]), (45, [9]), (65, [13]), (114, [19])])
def test_cycles(n, group, mg):
    pr = boxes(n, group)
    r = dev(np.random.default_rng(2).standard_normal(pr["N"]))
    for prec, tol in (("fp64", 1e-11), ("mixed", 2e-5)):     # as against the oracle's V-cycle
        z, lam = [], None
        for layout in ("axis_ell", "auto"):
            say("row boxes, cycle", n, mg, prec, layout)
            h, s = problem.build(pr, precision=prec, fine_layout=layout, lam_override=lam, **mg)
            i = s.info()
            lam = np.stack([i["lam_lo"][:-1], i["lam_hi"][:-1]], axis=1)
            z.append(torch.empty_like(r))
            api.vcycle(s, r, z[-1])
        assert rel(host(z[1]), host(z[0])) <= tol, prec
        x, y = torch.zeros_like(r), torch.empty_like(r)
        assert api.pcg_solve(s, r, x, tol=1e-10)["converged"]   # residuals and partials of the FP64 level
        api.apply(s, 0, x, y)
        assert rel(host(y), host(r)) <= 1e-8
