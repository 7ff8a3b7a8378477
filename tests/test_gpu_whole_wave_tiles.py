"""Tiles of whole-wave cells (blocks of 25) and of straddling ones (27) at their edges:
the level products on the axis and the slot layouts against the oracle, and the
multi-column kernels, which take their cells across tiles, against them."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, rel, say, torch
from oracle.assemble import system_matrix
from paper_2602_16312_amd import api, problem
from workloads import make_problem

pytestmark = pytest.mark.gpu
R = 8
CUBE = dict(jitter=0.1, seed=3, penalty=("paper", 2.0))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


# 9, 16, 49, 81 squares (Q4) and 8, 27, 64 hexahedra (Q2): one cell past a tile, whole
# tiles, ragged ones; agglomerated levels of regular and of ragged bins
@pytest.mark.parametrize("layout", ["axis_ell", "tile_ell"])
@pytest.mark.parametrize("name,kw", [("c2", dict(n=3, p=4, jitter=0.1, group=[3])),
                                     ("c2", dict(n=4, p=4, jitter=0.1, group=[2])),
                                     ("c2", dict(n=7, p=4, jitter=0.1, group=[4])),
                                     ("c2", dict(n=9, p=4, jitter=0.1, group=[3])),
                                     ("c3", dict(n=2, group=[2], **CUBE)), ("c3", dict(n=3, group=[2], **CUBE)),
                                     ("c3", dict(n=4, group=[2], **CUBE))])
def test_products_and_columns(name, kw, layout):
    pr = make_problem(name, **kw)
    assert pr["b"] in (25, 27)
    X = np.random.default_rng(5).standard_normal((pr["N"], R))
    ref = system_matrix(pr)[0] @ X
    # operator: as for the other layouts; columns: sums of 189 terms in another order
    for prec, tol, ctol in (("fp64", 1e-13, 1e-13), ("mixed", 3e-6, 3e-6)):
        h, s = problem.build(pr, precision=prec, max_rhs=R, fine_layout=layout)
        assert s.info()["fine_layout"] == layout
        nl = s.info()["n_levels"]
        for level in range(max(1, nl - 1)):
            n = s.info()["n_cells"][level] * pr["b"]
            say("whole-wave tiles", name, kw, layout, prec, level)
            Y = torch.empty(n * R, dtype=torch.float64, device="cuda")
            y = torch.empty(n, dtype=torch.float64, device="cuda")
            api.apply_multi(s, level, dev(X[:n].ravel()), Y, precision=prec)
            for c in range(R):
                api.apply(s, level, dev(np.ascontiguousarray(X[:n, c])), y, precision=prec)
                assert rel(host(Y).reshape(n, R)[:, c], host(y)) <= ctol, (prec, level, c)
                if level == 0:
                    assert rel(host(y), ref[:, c]) <= tol, (prec, c)
        say("whole-wave tiles, cycle", name, kw, layout, prec)
        Z = torch.empty(pr["N"] * R, dtype=torch.float64, device="cuda")
        z = torch.empty(pr["N"], dtype=torch.float64, device="cuda")
        api.vcycle_multi(s, dev(X.ravel()), Z)
        for c in range(R):
            api.vcycle(s, dev(np.ascontiguousarray(X[:, c])), z)
            # as against the oracle's V-cycle
            assert rel(host(Z).reshape(-1, R)[:, c], host(z)) <= (1e-11 if prec == "fp64" else 2e-5), (prec, c)
