"""The stored-block forms of agglomerated levels at the sizes where they are chosen,
against the row kernels: products, and V-cycles through every epilogue (point and
cell-block smoother, degrees 1 and 3)."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, rel, say, torch
from paper_2602_16312_amd import api, problem
from workloads import make_problem

pytestmark = pytest.mark.gpu
CUBE = dict(jitter=0.1, seed=3, penalty=("paper", 2.0))
MG = [dict(), dict(cheb_degree=1), dict(jacobi="cell_block"), dict(cheb_degree=1, jacobi="cell_block")]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def pair(pr, form, prec, other, **mg):
    """Solvers of a problem by rows and in the automatic form, with the same intervals."""
    out, lam = [], None
    for layout in (other, "auto"):
        h, s = problem.build(pr, precision=prec, fine_layout=layout, lam_override=lam, **mg)
        i = s.info()
        lam = np.stack([i["lam_lo"][:-1], i["lam_hi"][:-1]], axis=1)
        out.append(s)
    assert out[1].forms()["level_form"][1] == form and out[0].forms()["level_form"][1] == other
    return out


# level 1: 4,225 boxes of 4, 9 and 16, 4,096 of 8, 2,704 of 25, 2,744 of 27 (the last two ragged last
# groups of 16); 5,832 of 8, 8,100 of 25 and 4,913 of 27 (groups of 64); 4,225 overlapping boxes of 4 and 9, 5,832 of 8
@pytest.mark.parametrize("name,kw,form", [
    ("e1", dict(n=130, p=1, group=[2, 13]), "nodal_blocks"), ("e1", dict(n=130, p=2, group=[2, 13]), "nodal_blocks"),
    ("e1", dict(n=130, p=3, group=[2, 13]), "nodal_blocks"), ("c3", dict(n=32, p=1, group=[2, 16]), "nodal_blocks"),
    ("c3", dict(n=36, p=1, group=[2, 18]), "nodal_blocks"), ("e1", dict(n=104, p=4, group=[2, 13]), "nodal_blocks"),
    ("e1", dict(n=180, p=4, group=[2, 15]), "nodal_blocks"), ("c3", dict(n=28, group=[2, 14]), "nodal_blocks"),
    ("c3", dict(n=34, group=[2, 17]), "nodal_blocks"),
    ("c2", dict(n=130, p=1, group=[2, 13]), "whole_blocks"), ("c2", dict(n=130, group=[2, 13]), "whole_blocks"),
    ("c3", dict(n=36, p=1, group=[2, 18], **CUBE), "whole_blocks")])
def test_products(name, kw, form):
    pr = make_problem(name, **kw)
    s = pair(pr, form, "mixed", "axis_ell")
    x = dev(np.random.default_rng(5).standard_normal(s[0].info()["n_cells"][1] * pr["b"]))
    y = {}
    for prec in ("fp64", "mixed"):
        for k in range(2):
            y[k, prec] = torch.empty_like(x)
            say("level blocks", name, kw, prec, k)
            api.apply(s[k], 1, x, y[k, prec], prec)
    assert rel(host(y[1, "fp64"]), host(y[0, "fp64"])) <= 1e-13      # as for the other block forms
    assert rel(host(y[1, "mixed"]), host(y[0, "fp64"])) <= 3e-6


# level 1: 64 and 27 agglomerates of 64; 324 boxes of 4, 8 (343), 9 and 16, 2,116 of 25, 2,744 of 27; 289
# overlapping boxes of 4 and 9, 343 of 8; groups of 64: 4,225 of 9 (both kinds)
@pytest.mark.parametrize("mg", MG)
@pytest.mark.parametrize("name,kw,form", [
    ("c3", dict(n=8, p=3, group=[2, 2]), "row_blocks"), ("c3", dict(n=6, p=3, group=[2, 3]), "row_blocks"),
    ("e1", dict(n=36, p=1, group=[2, 9]), "nodal_blocks"), ("e1", dict(n=36, p=2, group=[2, 9]), "nodal_blocks"),
    ("e1", dict(n=36, p=3, group=[2, 9]), "nodal_blocks"), ("c3", dict(n=14, p=1, group=[2, 7]), "nodal_blocks"),
    ("e1", dict(n=92, p=4, group=[2, 23]), "nodal_blocks"), ("c3", dict(n=28, group=[2, 14]), "nodal_blocks"),
    ("c2", dict(n=34, p=1, group=[2, 17]), "whole_blocks"), ("c2", dict(n=34, group=[2, 17]), "whole_blocks"),
    ("c3", dict(n=14, p=1, group=[2, 7], **CUBE), "whole_blocks"),
    ("e1", dict(n=130, p=2, group=[2, 13]), "nodal_blocks"), ("c2", dict(n=130, group=[2, 13]), "whole_blocks")])
def test_cycles(name, kw, form, mg):
    pr = make_problem(name, **kw)
    r = dev(np.random.default_rng(2).standard_normal(pr["N"]))
    for prec, tol in (("fp64", 1e-11), ("mixed", 2e-5)):     # as against the oracle's V-cycle
        z = []
        for s in pair(pr, form, prec, "axis_ell", **mg):
            z.append(torch.empty_like(r))
            say("level blocks, cycle", name, kw, mg, prec)
            api.vcycle(s, r, z[-1])
        assert rel(host(z[1]), host(z[0])) <= tol, prec


@pytest.mark.parametrize("mg", MG)
def test_faces_once(mg):
    """10,212 irregular agglomerates, faces held once in FP32, against the slots."""
    pr = make_problem("c4", h=0.034, agglo=("rtree_str", 8, 4))
    s = pair(pr, "faces_once", "mixed", "tile_ell", **mg)
    r = dev(np.random.default_rng(2).standard_normal(pr["N"]))
    x = dev(np.random.default_rng(5).standard_normal(s[0].info()["n_cells"][1] * 8))
    y, z = {}, []
    for k in range(2):
        for prec in ("fp64", "mixed"):
            y[k, prec] = torch.empty_like(x)
            say("faces once", mg, k, prec)
            api.apply(s[k], 1, x, y[k, prec], prec)
        z.append(torch.empty_like(r))
        api.vcycle(s[k], r, z[k])
    assert np.array_equal(host(y[1, "fp64"]), host(y[0, "fp64"]))
    assert rel(host(y[1, "mixed"]), host(y[0, "fp64"])) <= 3e-6
    assert rel(host(z[1]), host(z[0])) <= 2e-5
