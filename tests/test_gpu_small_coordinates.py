"""Meshes in units in which an absolute tolerance on coordinates says nothing: the
operator of slightly distorted cells against the oracle's rows."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, rel, say, torch
from oracle.assemble import assemble
from paper_2602_16312_amd import api, problem
from paper_2602_16312_amd._ffi import DGMGError
from workloads import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


# unit square of 17x17 cells scaled to 1e-13, and to 1 mm with vertices off by up to 2e-13 m
@pytest.mark.parametrize("scale,jitter,form", [(1e-13, 0.1, "hybrid"), (1e-3, 4e-9, "hybrid"), (1e-3, 0.0, "box")])
def test_q1_rows_match_oracle(scale, jitter, form):
    pr = make_problem("c2", n=17, p=1, jitter=jitter, group=[17])
    pr["xyz"] = pr["xyz"] * scale
    h, s = problem.build(pr, precision="mixed")
    assert s.forms()["level_form"][0] == form
    M, A = assemble(pr, None)
    ref = ((1.5 * pr["chi"] * pr["Cm"] / pr["dt"]) * M + A) @ (x := np.random.default_rng(4).standard_normal(pr["N"]))
    y = torch.empty(pr["N"], dtype=torch.float64, device="cuda")
    for prec, tol in (("fp64", 1e-13), ("mixed", 3e-6)):   # as for the other operators
        say("small coordinates", scale, jitter, prec)
        api.apply(s, 0, dev(x), y, prec)
        assert rel(host(y), ref) <= tol, prec


@pytest.mark.parametrize("p", [2, 3])
def test_distorted_cells_of_any_unit_are_no_boxes(p):
    def tiny(name, **kw):   # the time step shrinks with the area, so that the mass term stays
        pr = make_problem(name, n=17, p=p, group=[17], **kw)
        return {**pr, "xyz": pr["xyz"] * 1e-13, "dt": pr["dt"] * 1e-26}

    pr = tiny("c2", jitter=0.1)
    with pytest.raises(DGMGError) as e:
        problem.build(pr, precision="mixed", fine_layout="matrix_free")
    assert e.value.code == -6
    h, s = problem.build(pr, precision="mixed")
    M, A = assemble(pr, None)
    ref = ((1.5 * pr["chi"] * pr["Cm"] / pr["dt"]) * M + A) @ (x := np.random.default_rng(4).standard_normal(pr["N"]))
    y = torch.empty(pr["N"], dtype=torch.float64, device="cuda")
    for prec, tol in (("fp64", 1e-13), ("mixed", 3e-6)):
        say("small coordinates", p, prec)
        api.apply(s, 0, dev(x), y, prec)
        assert rel(host(y), ref) <= tol, prec
    h, s = problem.build(tiny("e1"), precision="mixed", fine_layout="matrix_free")   # real boxes still are
    assert s.info()["fine_layout"] == "matrix_free"
