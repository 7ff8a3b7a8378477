"""Cell kernels on distorted cells (metric data at the Gauss points) and on the
stored blocks of agglomerated boxes: operator rows against the oracle, and
V-cycles and level products against the row kernels of the axis layout."""
import numpy as np
import pytest

from gpu_util import dev, host, need_gpu, rel, say, torch
from oracle.assemble import assemble
from paper_2602_16312_amd import api, problem
from workloads import make_problem

pytestmark = pytest.mark.gpu
CUBE = dict(jitter=0.1, seed=3, penalty=("paper", 2.0))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


# 256, 289, 4,225 squares (Q1 to Q4) and 343, 4,913 hexahedra (Q1, Q2): both group sizes, ragged groups
@pytest.mark.parametrize("name,kw", [
    ("c2", dict(n=16, group=[4])), ("c2", dict(n=17, p=3, jitter=0.1, group=[17])),
    ("c2", dict(n=17, p=4, jitter=0.1, penalty=("fixed", 900.0), group=[17])),
    ("c2", dict(n=65, group=[13])), ("c2", dict(n=65, p=3, jitter=0.1, group=[13])),
    ("c2", dict(n=65, p=4, jitter=0.1, group=[13])), ("c3", dict(n=7, group=[7], **CUBE)),
    ("c3", dict(n=17, group=[17], **CUBE)), ("c2", dict(n=17, p=1, group=[17])), ("c2", dict(n=65, p=1, group=[13])),
    ("c3", dict(n=7, p=1, group=[7], **CUBE)), ("c3", dict(n=17, p=1, group=[17], **CUBE))])
def test_mapped_rows_match_oracle(name, kw):
    pr = make_problem(name, **kw)
    n, b = pr["n_cells"], pr["b"]
    scale = np.random.default_rng(3).uniform(0.5, 2.0, n)
    h, s = problem.build(pr, precision="mixed", cell_scale=scale)
    assert s.info()["fine_layout"] == ("axis_ell" if pr["p"] == 1 else "matrix_free")
    assert not s.info()["sparse_faces"]
    rng = np.random.default_rng(4)
    cells = np.unique(np.concatenate([[0, 15, 16, 63, 64, n - 1, n - 2], rng.integers(0, n, 24)]) % n)
    M, A = assemble(pr, scale, row_cells=cells)
    rows = (cells[:, None] * b + np.arange(b)).ravel()
    x = rng.standard_normal(pr["N"])
    ref = ((1.5 * pr["chi"] * pr["Cm"] / pr["dt"]) * M + A)[rows] @ x
    y = torch.empty(pr["N"], dtype=torch.float64, device="cuda")
    for prec, tol in (("fp64", 1e-13), ("mixed", 3e-6)):   # as for the operator on boxes
        say("mapped rows", name, kw, prec)
        api.apply(s, 0, dev(x), y, prec)
        assert rel(host(y)[rows], ref) <= tol, prec


@pytest.mark.parametrize("mg", [dict(), dict(cheb_degree=1), dict(jacobi="cell_block"),
                                dict(cheb_degree=1, jacobi="cell_block")])
@pytest.mark.parametrize("name,kw", [("c2", dict(n=20, group=[4])), ("c3", dict(n=8, group=[2], **CUBE)),
                                     ("c3", dict(n=8, p=1, group=[2], **CUBE)), ("c1", dict(n=16))])
def test_mapped_vcycle_matches_blocks(name, kw, mg):
    pr = make_problem(name, **kw)
    r = dev(np.random.default_rng(2).standard_normal(pr["N"]))
    z = [torch.empty_like(r) for _ in range(2)]
    for prec, tol in (("fp64", 1e-11), ("mixed", 2e-5)):   # as against the oracle's V-cycle
        lam = None
        for k, layout in enumerate(("axis_ell", "auto")):
            h, s = problem.build(pr, precision=prec, fine_layout=layout, lam_override=lam, **mg)
            i = s.info()
            lam = np.stack([i["lam_lo"][:-1], i["lam_hi"][:-1]], axis=1)
            say("mapped vcycle", name, mg, prec, layout)
            api.vcycle(s, r, z[k])
        assert rel(host(z[1]), host(z[0])) <= tol, prec


# level 1: 1,024 boxes of 9 and 16 DoFs, 2,704 of 25, 2,197 of 27, 64 and 27 of 64 (by rows),
# 289 overlapping boxes of 9 and of 4 DoFs
@pytest.mark.parametrize("name,kw", [
    ("e1", dict(n=64, p=2, group=[2, 8])), ("e1", dict(n=64, p=3, group=[2, 8])),
    ("e1", dict(n=104, p=4, group=[2, 13])), ("c3", dict(n=26, group=[2, 13])),
    ("c3", dict(n=8, p=3, group=[2, 2])), ("c3", dict(n=6, p=3, group=[2, 3])),
    ("c2", dict(n=68, group=[4, 17])), ("c2", dict(n=68, p=1, group=[4, 17]))])
def test_stored_boxes_match_rows(name, kw):
    pr = make_problem(name, **kw)
    out = {}
    for layout in ("axis_ell", "auto"):
        h, s = problem.build(pr, precision="mixed", fine_layout=layout)
        n = s.info()["n_cells"][1] * pr["b"]
        x = dev(np.random.default_rng(5).standard_normal(n))
        for prec in ("fp64", "mixed"):
            y = torch.empty_like(x)
            say("stored boxes", name, layout, prec)
            api.apply(s, 1, x, y, prec)
            out[layout, prec] = host(y)
    assert rel(out["auto", "fp64"], out["axis_ell", "fp64"]) <= 1e-13
    assert rel(out["auto", "mixed"], out["axis_ell", "fp64"]) <= 3e-6


@pytest.mark.parametrize("mg", [dict(), dict(cheb_degree=1), dict(jacobi="cell_block"),
                                dict(cheb_degree=1, jacobi="cell_block")])
def test_faces_held_once_match_tile_slots(mg):
    pr = make_problem("c4", h=0.042, agglo=("rtree_str", 8, 4))
    r = dev(np.random.default_rng(2).standard_normal(pr["N"]))
    z = [torch.empty_like(r) for _ in range(2)]
    y, lam = {}, None
    for k, layout in enumerate(("tile_ell", "auto")):
        h, s = problem.build(pr, precision="mixed", fine_layout=layout, lam_override=lam, **mg)
        i = s.info()
        assert i["n_cells"][1] >= 4000 and i["level_layout"][1] == "tile_ell"
        lam = np.stack([i["lam_lo"][:-1], i["lam_hi"][:-1]], axis=1)
        x = dev(np.random.default_rng(5).standard_normal(i["n_cells"][1] * 8))
        for prec in ("fp64", "mixed"):
            y[layout, prec] = torch.empty_like(x)
            say("faces once", mg, layout, prec)
            api.apply(s, 1, x, y[layout, prec], prec)
        api.vcycle(s, r, z[k])
    assert np.array_equal(host(y["auto", "fp64"]), host(y["tile_ell", "fp64"]))
    assert rel(host(y["auto", "mixed"]), host(y["tile_ell", "fp64"])) <= 3e-6
    assert rel(host(z[1]), host(z[0])) <= 2e-5


@pytest.mark.parametrize("name,kw", [("c2", dict(n=17, p=3, jitter=0.1, group=[17])), ("c2", dict(n=17, p=4, jitter=0.1, group=[17])),
                                     ("c3", dict(n=7, group=[7], **CUBE)), ("c3", dict(n=9, group=[3]))])
def test_step_on_gauss_point_mass(name, kw):
    """The load vector formed at the Gauss points, in a time step, against the stored mass blocks'."""
    pr = make_problem(name, **kw)
    rng = np.random.default_rng(6)
    U = [rng.uniform(0.0, 1.0, pr["N"]) for _ in range(2)]
    W = [rng.uniform(0.2, 0.8, pr["S"] * pr["N"]) for _ in range(2)]
    out = []
    for layout in ("axis_ell", "auto"):
        h, s = problem.build(pr, precision="fp64", fine_layout=layout)
        st = api.State(dev(U[0]), dev(U[1]), dev(W[0]), dev(W[1]), torch.empty(pr["N"], dtype=torch.float64, device="cuda"))
        say("mass step", name, kw, layout)
        assert api.time_step(s, st, pr["dt"], iapp=dev(np.full(pr["N"], 0.1)), tol=1e-13)["converged"]
        out.append((host(st.U), host(st.W)))
    assert rel(out[1][0], out[0][0]) <= 1e-10              # the time series' bound
    assert np.array_equal(out[1][1], out[0][1])
