"""Q1 meshes in units in which an absolute tolerance on coordinates says nothing: the
operator of slightly distorted cells against the oracle's rows."""
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
