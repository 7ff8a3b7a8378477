"""The form that the set-up chooses for each level, and whether the PCG's directions
are held as graphs, as the solver reports them."""
import pytest

from gpu_util import need_gpu, say
from paper_2602_16312_amd import problem
from stream_shim import run_child
from workloads import make_problem

pytestmark = pytest.mark.gpu
CUBE = dict(jitter=0.1, seed=3, penalty=("paper", 2.0))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


@pytest.mark.parametrize("name,kw,mg,forms", [
    ("c1", dict(n=16), {}, ["box", "none"]), ("c1", dict(n=12), {}, ["axis_ell_sparse", "none"]),
    ("e1", dict(n=64, p=2, group=[2, 8]), {}, ["box", "nodal_blocks", "none"]),
    ("e1", dict(n=64, p=3, group=[2, 8]), {}, ["box", "nodal_blocks", "none"]),
    ("e1", dict(n=128, p=4, group=[2, 16]), {}, ["box", "nodal_blocks", "none"]),
    ("e1", dict(n=64, p=4, group=[2, 8]), {}, ["box", "axis_ell", "none"]),
    # nested boxes whose face blocks hold roundoff where others of the degree hold zeros
    ("e1", dict(n=60, p=3, group=[2, 10]), {}, ["box", "nodal_blocks", "none"]),
    ("e1", dict(n=104, p=3, group=[2, 13]), {}, ["box", "nodal_blocks", "none"]),
    ("e1", dict(n=104, p=4, group=[2, 13]), {}, ["box", "nodal_blocks", "none"]),
    ("c3", dict(n=32, group=[2, 8]), {}, ["box", "nodal_blocks", "none"]),
    # on either side of the sizes where rows and slots are as fast
    ("e1", dict(n=90, p=4, group=[2, 9]), {}, ["box", "axis_ell", "none"]),
    ("e1", dict(n=92, p=4, group=[2, 23]), {}, ["box", "nodal_blocks", "none"]),
    ("c3", dict(n=26, group=[2, 13]), {}, ["box", "axis_ell", "none"]),
    ("c3", dict(n=28, group=[2, 14]), {}, ["box", "nodal_blocks", "none"]),
    ("c4", dict(h=0.036, agglo=("rtree_str", 8, 4)), {}, ["hybrid", "tile_ell", "tile_ell", "none"]),
    ("c4", dict(h=0.034, agglo=("rtree_str", 8, 4)), {}, ["hybrid", "faces_once", "tile_ell", "none"]),
    ("c3", dict(n=8, p=3, group=[2, 2]), {}, ["box", "row_blocks", "none"]),
    ("c2", dict(n=68, group=[2, 17]), {}, ["mapped", "whole_blocks", "none"]),
    ("c2", dict(n=68, p=1, group=[2, 17]), {}, ["hybrid", "whole_blocks", "none"]),
    ("c2", dict(n=68, p=3, jitter=0.1, group=[2, 17]), {}, ["mapped", "axis_ell", "none"]),
    ("c3", dict(n=7, group=[7], **CUBE), {}, ["mapped", "none"]),
    ("c3", dict(n=4, p=3, group=[2], **CUBE), {}, ["axis_ell_sparse", "none"]),
    ("c2", dict(n=16, group=[4]), dict(fine_layout="axis_ell"), ["axis_ell_sparse", "none"]),
    ("c2", dict(n=16, group=[4]), dict(fine_layout="tile_ell"), ["tile_ell", "none"]),
    ("c2", dict(n=16, group=[4]), dict(max_rhs=8), ["axis_ell", "none"]),
    ("c4", dict(h=0.03, agglo=("rtree_str", 8, 4)), {}, ["hybrid", "faces_once", "tile_ell", "none"])])
def test_forms(name, kw, mg, forms):
    pr = make_problem(name, **kw)
    say("forms", name, kw, mg)
    h, s = problem.build(pr, precision="mixed", **mg)
    assert s.forms()["level_form"] == forms


@pytest.mark.parametrize("degree", [1, 2, 3])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_graphs_are_held(prec, degree):
    for name, kw in (("c1", dict(n=16)), ("c2", dict(n=16, group=[4])), ("c3", dict(n=6, group=[3])), ("c4", dict(h=0.15))):
        for jacobi in ("point", "cell_block"):
            say("graphs", name, kw, prec, degree, jacobi)
            h, s = problem.build(make_problem(name, **kw), precision=prec, cheb_degree=degree, jacobi=jacobi)
            assert s.forms()["pcg_graphs"] == ("held" if degree > 1 else "unused")


def test_a_failure_to_record_is_reported(tmp_path):
    """The solver then launches kernel by kernel, to the same result, and says why."""
    say("graphs refused (child process)")
    out = run_child(tmp_path, r"""
pr = make_problem("c2", n=16, group=[4])
b = torch.from_numpy(np.random.default_rng(1).standard_normal(pr["N"])).cuda()
x = []
for refuse in (0, 1):
    shim.shim_refuse(refuse)
    h, s = problem.build(pr, precision="mixed")
    shim.shim_refuse(0)
    print("graphs", s.forms()["pcg_graphs"], flush=True)
    x.append(torch.zeros_like(b))
    api.pcg_solve(s, b, x[-1], tol=1e-9)
assert torch.equal(*x)
""")
    lines = [l.split(None, 1)[1] for l in out.splitlines() if l.startswith("graphs")]
    assert lines[0] == "held" and lines[1].startswith("failed: ") and len(lines[1]) > 12, out


def test_set_up_captures_no_stream(tmp_path):
    """While one thread captures a stream, other threads' calls on the legacy stream fail."""
    say("captures (child process)")
    out = run_child(tmp_path, r"""
pr = make_problem("c2", n=16, group=[4])
b = torch.from_numpy(np.random.default_rng(1).standard_normal(pr["N"])).cuda()
h, s = problem.build(pr, precision="mixed")
x = torch.zeros_like(b)
api.pcg_solve(s, b, x, tol=1e-9)
print("graphs", s.forms()["pcg_graphs"], "captures", shim.shim_captures(), flush=True)
""")
    assert "graphs held captures 0" in out, out


def test_solvers_of_several_threads():
    """Set-ups and solves of four threads at once, each on a stream of its own: no call
    fails and every result equals the serial one."""
    import threading
    import numpy as np
    from gpu_util import torch
    from paper_2602_16312_amd import api
    cases = [("c1", dict(n=16), "fp64"), ("c2", dict(n=16, group=[4]), "mixed"), ("e1", dict(n=12, p=4, group=[3]), "fp64"),
             ("c3", dict(n=6, group=[3]), "mixed")]
    prs = [make_problem(name, **kw) for name, kw, _ in cases]

    def work(k, out, stream):
        with torch.cuda.stream(stream):
            b = torch.from_numpy(np.random.default_rng(k).standard_normal(prs[k]["N"])).cuda()
            res = []
            for _ in range(8):
                h, s = problem.build(prs[k], precision=cases[k][2])
                for _ in range(3):
                    x = torch.zeros_like(b)
                    its = api.pcg_solve(s, b, x, tol=1e-9, stream=stream)["its"]
                    res.append((its, x.cpu().numpy()))
                assert s.forms()["pcg_graphs"] == "held"
            out[k] = res

    say("threads, serial")
    ref = {}
    for k in range(len(cases)):
        work(k, ref, torch.cuda.current_stream())
    for r in range(3):
        say("threads, round", r)
        out, failed = {}, []

        def guarded(k):
            try:
                work(k, out, torch.cuda.Stream())
            except Exception as e:   # reported by the test's own thread
                failed.append((k, e))

        threads = [threading.Thread(target=guarded, args=(k,)) for k in range(len(cases))]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not failed, failed
        for k in range(len(cases)):
            for (i0, x0), (i1, x1) in zip(ref[k], out[k]):
                assert i0 == i1 and np.array_equal(x0, x1), k
