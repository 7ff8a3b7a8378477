"""3D Q3 boxes with the cell-block smoother: V-cycles at the edges of the groups of 4
and 16 cells (27, 64 and 1,331 boxes by 4, 2,197 by 16) against the row kernels."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, rel, say, torch
from paper_2602_16312_amd import api, problem
from workloads import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("degree", [1, 3])
@pytest.mark.parametrize("n", [3, 4, 11, 13])
def test_cycles(n, degree):
    pr = make_problem("c3", n=n, p=3, group=[n])
    r = dev(np.random.default_rng(2).standard_normal(pr["N"]))
    for prec, tol in (("fp64", 1e-11), ("mixed", 2e-5)):     # as against the oracle's V-cycle
        z, lam = [], None
        for layout in ("axis_ell", "auto"):
            say("cell-block groups", n, degree, prec, layout)
            h, s = problem.build(pr, precision=prec, fine_layout=layout, lam_override=lam, jacobi="cell_block",
                                 cheb_degree=degree)
            i = s.info()
            lam = np.stack([i["lam_lo"][:-1], i["lam_hi"][:-1]], axis=1)
            z.append(torch.empty_like(r))
            api.vcycle(s, r, z[-1])
        assert s.forms()["level_form"][0] == "box"
        assert rel(host(z[1]), host(z[0])) <= tol, prec
        x = torch.zeros_like(r)
        assert api.pcg_solve(s, r, x, tol=1e-10)["converged"]   # residuals and partials of the FP64 level
        y = torch.empty_like(r)
        api.apply(s, 0, x, y)
        assert rel(host(y), host(r)) <= 1e-8
