"""How a PCG call ends: an error of the work that was still queued is reported."""
import pytest

from gpu_util import need_gpu, say
from stream_shim import run_child

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def test_an_error_of_the_last_wait_is_reported(tmp_path):
    say("error of the last wait (child process)")
    out = run_child(tmp_path, r"""
pr = make_problem("c2", n=16, group=[4])
h, s = problem.build(pr, precision="mixed")
b = torch.from_numpy(np.random.default_rng(1).standard_normal(pr["N"])).cuda()
zero = torch.zeros_like(b)
x = torch.zeros_like(b)
for solve in (api.pcg_solve, api.pcg_solve_noalloc):
    # converged, cut off, nothing to do
    for rhs, opts in ((b, dict(tol=1e-8)), (b, dict(tol=1e-8, max_it=2)), (zero, dict())):
        x.zero_()
        rc = solve(s, rhs, x, **opts)["rc"]
        shim.shim_fail(1)
        try:
            x.zero_()
            solve(s, rhs, x, **opts)
            print("missed", solve.__name__, opts, flush=True)
        except F.DGMGError as e:
            print("reported", e.code, flush=True)
        shim.shim_fail(0)
        x.zero_()
        assert solve(s, rhs, x, **opts)["rc"] == rc
""")
    assert out.count("reported -4") == 6, out
    assert "missed" not in out


def coarse_solves(s, b, **opts):
    """(V-cycles that a solve from zero ran, its iterations)"""
    from gpu_util import torch
    from paper_2602_16312_amd import api
    x = torch.zeros_like(b)
    api.profile_begin(s, "coarse", s.info()["n_levels"] - 1)
    its = api.pcg_solve(s, b, x, **opts)["its"]
    n, _ = api.profile_end(s)
    return n, its


def small_solver(name, mg, **kw):
    import numpy as np
    from gpu_util import dev
    from paper_2602_16312_amd import problem
    from workloads import make_problem
    pr = make_problem(name, **kw)
    h, s = problem.build(pr, precision="fp64", **mg)
    return s, dev(np.random.default_rng(1).standard_normal(pr["N"]))


def test_no_direction_for_no_iterations():
    s, b = small_solver("c2", {}, n=16, group=[4])
    say("max_it 0")
    assert coarse_solves(s, b, max_it=0) == (0, 0)
    say("max_it 1 and 2")
    assert coarse_solves(s, b, max_it=1) == (1, 1)
    assert coarse_solves(s, b, max_it=2) == (2, 2)


# one level (an exact inverse); a spectrum so small that the second reduction is the square of the first
@pytest.mark.parametrize("name,kw,mg", [("c1", dict(n=8, group=[]), dict()), ("c2", dict(n=6, group=[], jitter=0.1), dict()),
                                        ("e1", dict(n=4, group=[2]), dict(jacobi="cell_block")),
                                        ("c1", dict(n=16), dict()), ("c2", dict(n=16, group=[4]), dict())])
@pytest.mark.parametrize("tol", [1e-4, 1e-8, 1e-10])
def test_no_direction_is_thrown_away(name, kw, mg, tol):
    s, b = small_solver(name, mg, **kw)
    say("directions", name, kw, tol)
    n, its = coarse_solves(s, b, tol=tol)
    assert its > 0 and n == its


def test_the_wait_follows_the_devices_scheduling_mode(tmp_path):
    """A process that chose blocking waits gets a synchronisation per stopping test,
    one that did not a poll (one synchronisation, at the end); the same solution."""
    body = r"""
mode = MODE
if mode:
    assert hip.hipSetDeviceFlags(ctypes.c_uint(mode)) == 0
pr = make_problem("c2", n=16, group=[4])
h, s = problem.build(pr, precision="mixed")
b = torch.from_numpy(np.random.default_rng(1).standard_normal(pr["N"])).cuda()
for k, solve in enumerate((api.pcg_solve, api.pcg_solve_noalloc)):
    x = torch.zeros_like(b)
    torch.cuda.synchronize()
    before = shim.shim_calls()
    its = solve(s, b, x, tol=1e-9)["its"]
    print("calls", shim.shim_calls() - before, its, repr(float(x.norm())), flush=True)
"""
    got = {}
    for mode in (0, 2, 4):   # automatic, yield, blocking
        say("scheduling mode (child process)", mode)
        out = run_child(tmp_path, body.replace("MODE", str(mode)))
        got[mode] = [l.split()[1:] for l in out.splitlines() if l.startswith("calls")]
        assert len(got[mode]) == 2, out
    for k in range(2):
        calls, its = {m: int(v[k][0]) for m, v in got.items()}, int(got[0][k][1])
        assert calls[0] == 1 and calls[2] == 1 and calls[4] == its + 2   # the first residual's and the end's
        assert got[0][k][1:] == got[2][k][1:] == got[4][k][1:]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("mg", [dict(cheb_sweeps=0), dict(cheb_sweeps=1, cheb_degree=2), dict(cheb_sweeps=0, jacobi="cell_block")])
def test_recorded_directions_without_or_with_one_sweep(prec, mg):
    """Graphs against single launches where the V-cycle has other kernels than usual."""
    import numpy as np
    from gpu_util import dev, host, torch
    from paper_2602_16312_amd import api, problem
    from workloads import make_problem
    pr = make_problem("c2", n=16, group=[2, 4])
    h, s = problem.build(pr, precision=prec, **mg)
    assert s.forms()["pcg_graphs"] == "held"
    b = dev(np.random.default_rng(3).standard_normal(pr["N"]))
    for _ in range(3):
        x = [torch.zeros_like(b) for _ in range(2)]
        say("recorded directions", prec, mg)
        its = [f(s, b, y, tol=1e-9, max_it=3) for f, y in ((api.pcg_solve, x[0]), (api.pcg_solve_noalloc, x[1]))]
        assert its[0] == its[1] and np.array_equal(host(x[0]), host(x[1]))
