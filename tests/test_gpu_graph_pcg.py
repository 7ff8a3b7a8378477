"""PCG with its search directions replayed as graphs: bitwise equal, solve after
solve, to the launch-by-launch solves of the non-allocating entry point, with
other calls on the solver in between."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, say, torch
from paper_2602_16312_amd import api, problem
from workloads import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("name,kw,mg", [
    ("c1", dict(n=16), dict()), ("c2", dict(n=16, group=[4]), dict()), ("c2", dict(n=16, group=[4]), dict(cheb_degree=1)),
    ("c2", dict(n=16, group=[4]), dict(cheb_degree=2)), ("c3", dict(n=6, group=[3]), dict()), ("c4", dict(h=0.15), dict()),
    ("c4", dict(h=0.15), dict(jacobi="cell_block"))])
def test_replays_equal_single_launches(name, kw, mg, prec):
    pr = make_problem(name, **kw)
    h, s = problem.build(pr, precision=prec, **mg)
    rng = np.random.default_rng(7)
    z = torch.empty(pr["N"], dtype=torch.float64, device="cuda")
    for k in range(5):
        b = dev(rng.standard_normal(pr["N"]))
        x = [torch.zeros_like(b) for _ in range(3)]
        say("graph pcg", name, kw, mg, prec, k)
        its = [api.pcg_solve(s, b, x[0], tol=1e-9), api.pcg_solve_noalloc(s, b, x[1], tol=1e-9)]
        assert its[0] == its[1]
        assert np.array_equal(host(x[0]), host(x[1])), k
        # renames the flexible buffers, overwrites the V-cycle's
        api.pcg_solve(s, b, x[2], tol=1e-5, flexible=True)
        api.vcycle(s, x[2], z)
        api.apply(s, 0, x[2], z)


def test_stopping_with_work_queued_ahead():
    """A solve that ends earlier than its reduction factor promised, and one cut off by max_it."""
    pr = make_problem("c2", n=16, group=[4])
    h, s = problem.build(pr, precision="fp64")
    A = [torch.empty(pr["N"], dtype=torch.float64, device="cuda") for _ in range(2)]
    x = dev(np.random.default_rng(1).standard_normal(pr["N"]))
    api.apply(s, 0, x, A[0])
    for opts in (dict(tol=1e-3), dict(tol=1e-14), dict(tol=1e-9, max_it=2), dict(tol=1e-9, max_it=0),
                 dict(tol=0.5, tol_mode="rel_b"), dict(tol=1e30, tol_mode="abs")):
        y = [torch.zeros_like(x) for _ in range(2)]
        say("queued ahead", opts)
        r = [api.pcg_solve(s, A[0], y[0], **opts), api.pcg_solve_noalloc(s, A[0], y[1], **opts)]
        assert r[0] == r[1]
        assert np.array_equal(host(y[0]), host(y[1]))
