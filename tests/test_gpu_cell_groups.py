"""Cell-per-lane fine-level kernels at the edges of their workgroups (16, 32 and
64 cells, ragged last groups, 3D Q3 quads) against oracle-assembled rows."""
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


# cells: 25, 4,225 and 8,281 (Q2, Q3, Q4 squares), 4,913 and 9,261 (Q2 cubes), 27 and 1,331 (Q3 cubes)
@pytest.mark.parametrize("name,kw", [
    ("e1", dict(n=5, p=2, group=[5])), ("e1", dict(n=65, p=2, group=[13])), ("e1", dict(n=91, p=3, group=[13])),
    ("e1", dict(n=91, p=4, group=[13])), ("c3", dict(n=17, group=[17])), ("c3", dict(n=21, group=[7])),
    ("c3", dict(n=3, p=3, group=[3])), ("c3", dict(n=11, p=3, group=[11]))])
def test_cell_groups_match_oracle_rows(name, kw):
    pr = make_problem(name, **kw)
    n, b = pr["n_cells"], pr["b"]
    scale = np.random.default_rng(3).uniform(0.5, 2.0, n)
    h, s = problem.build(pr, precision="mixed", cell_scale=scale, fine_layout="matrix_free")
    rng = np.random.default_rng(4)
    cells = np.unique(np.concatenate([[0, 15, 16, 31, 32, 63, 64, n - 1, n - 2], rng.integers(0, n, 24)]) % n)
    M, A = assemble(pr, scale, row_cells=cells)
    rows = (cells[:, None] * b + np.arange(b)).ravel()
    x = rng.standard_normal(pr["N"])
    ref = ((1.5 * pr["chi"] * pr["Cm"] / pr["dt"]) * M + A)[rows] @ x
    y = torch.empty(pr["N"], dtype=torch.float64, device="cuda")
    for prec, tol in (("fp64", 1e-13), ("mixed", 3e-6)):   # the bounds of the small parity cases
        say("cell groups", name, kw, prec)
        api.apply(s, 0, dev(x), y, prec)
        assert rel(host(y)[rows], ref) <= tol, prec
