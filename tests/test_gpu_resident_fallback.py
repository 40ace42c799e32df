"""Launches of the resident kernel that do not run, forced from the host (every
kernel leaves by its ordinary exits): the solve goes on in the streaming kernels
with the result of one that ran.  Bars as elsewhere: the oracle's decisions,
steps within one, x within 1e-10 at equal step counts."""
import numpy as np
import pytest

from paper_2103_07210_amd import inputs as I
from paper_2103_07210_amd.inputs import FaultEvent, OctProblem, Problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2103_07210_amd import ftgcr
    ftgcr.load()
    return ftgcr


def _decisions(log):
    return [(d["step"], d["nu"], d["action"]) for d in log]


def _err(a, b):
    a, b = np.asarray(a).ravel(), np.asarray(b).ravel()
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def _same_as_oracle(ft, orc, rhs, x, st, k, plan):
    _, so, logo, _ = orc.solve(rhs, tol=1e-10, k=k, plan=plan)
    assert st["status"] == so["status"] == ft.CONVERGED
    assert _decisions(st["log"]) == _decisions(logo), (st["log"], logo)
    assert st["events_applied"] == so["events_applied"]
    assert abs(st["steps_executed"] - so["steps_executed"]) <= 1
    xe, _, _, _ = orc.solve(rhs, tol=1e-14, k=k, plan=plan, max_steps=st["steps_executed"])
    assert _err(x.cpu().numpy(), xe) <= 1e-10


def _oracle(oracle_mod, pb):
    return (oracle_mod.OctOracle if isinstance(pb, OctProblem) else oracle_mod.Oracle)(pb)


def _plans(pb):
    """Flips that double or halve every entry of r (twice as large a norm: seen
    against the norm before them, not against the one after), alone and among
    others, at a first and at a later pass of a cycle."""
    n = pb.n
    r = dict(start=0, count=n)
    return {"r": [FaultEvent(6, "r", 52, **r)],
            "r at a cycle's start": [FaultEvent(7, "r", 52, **r)],
            "r and others": [FaultEvent(6, "r", 51, start=0, count=n // 3), FaultEvent(6, "ap", 51, start=n // 2, count=3),
                             FaultEvent(6, "r", 52, start=n // 4, count=n // 2), FaultEvent(6, "x", 40, start=0, count=n)]}


@pytest.mark.parametrize("outcome", ["LATE", "REFUSED"])
@pytest.mark.parametrize("which", ["r", "r at a cycle's start", "r and others"])
@pytest.mark.parametrize("pb", [Problem(64, 16, 16), OctProblem(7, 21)], ids=lambda v: str(v.shape))
def test_flip_in_r_before_a_launch_that_does_not_run(ft, oracle_mod, pb, which, outcome):
    """The second launch starts at the step with the flips."""
    print("[gpu-case] fallback", pb, which, outcome, flush=True)
    rhs, plan = I.rhs(pb, 31), _plans(pb)[which]
    s = ft.Solver(pb, kmax=3)
    s.debug_resident(2, getattr(ft, "RESIDENT_" + outcome))
    x, st = s.solve(rhs, tol=1e-10, k=3, plan=plan)
    assert st["detections"] == 1
    _same_as_oracle(ft, _oracle(oracle_mod, pb), rhs, x, st, 3, plan)
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("pb", [Problem(64, 32, 8), OctProblem(12, 21)], ids=lambda v: str(v.shape))
def test_solve_after_a_failed_one(ft, pb, precision):
    """A launch that came apart after 40 steps fails its solve; the rounds it
    exchanged leave no trace in the handle's next solves (a handle without a
    past gives the same bits)."""
    print("[gpu-case] after a failed solve", pb, precision, flush=True)
    s, fresh = ft.Solver(pb, precision, kmax=3), ft.Solver(pb, precision, kmax=3)
    s.debug_resident(1, ft.RESIDENT_BROKEN)
    s.set_options(max_steps=40)
    with pytest.raises(ft.FtgcrError) as e:
        s.solve(I.rhs(pb, 32), tol=1e-10, k=3)
    assert e.value.code == ft.E_HIP
    s.debug_resident(0)
    s.set_options(max_steps=100000)
    for seed in (33, 34):
        x, st = s.solve(I.rhs(pb, seed), tol=1e-8, k=3)
        y, su = fresh.solve(I.rhs(pb, seed), tol=1e-8, k=3)
        assert st["status"] == ft.CONVERGED and st["steps_executed"] == su["steps_executed"]
        assert bool((x == y).all())
    s.close()
    fresh.close()


def test_batch_after_a_failed_one(ft):
    print("[gpu-case] after a failed batch", flush=True)
    pbs = [Problem(64, 32, 8), Problem(40, 20, 15), Problem(64, 32, 7)]
    groups = [[ft.Solver(pb, kmax=3) for pb in pbs] for _ in range(2)]
    rhs = [I.rhs(pb, 35 + m) for m, pb in enumerate(pbs)]
    groups[0][2].debug_resident(1, ft.RESIDENT_BROKEN)
    with pytest.raises(ft.FtgcrError) as e:
        ft.solve_batch(groups[0], rhs, tols=[1e-8] * 3, k=3)
    assert e.value.code == ft.E_HIP
    groups[0][2].debug_resident(0)
    out = [ft.solve_batch(g, rhs, tols=[1e-8] * 3, k=3) for g in groups]
    for x, y, a, b in zip(out[0][0], out[1][0], out[0][1], out[1][1]):
        assert a["status"] == ft.CONVERGED and a["steps_executed"] == b["steps_executed"]
        assert bool((x == y).all())
    for g in groups:
        for s in g:
            s.close()


@pytest.mark.parametrize("outcome", ["LATE", "REFUSED"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("pb", [Problem(250, 33, 9), OctProblem(12, 21)], ids=lambda v: str(v.shape))
def test_no_launch_runs(ft, pb, precision, outcome):
    """From the first launch on: the streaming kernels' result to the last bit;
    blocks that start late in the next solve's launches are counted afresh."""
    print("[gpu-case] no launch runs", pb, precision, outcome, flush=True)
    rhs = I.rhs(pb, 36)
    order = ft.ORDER_XCD if isinstance(pb, OctProblem) else ft.ORDER_X   # the mesh's default
    s, streaming = ft.Solver(pb, precision, kmax=3), ft.Solver(pb, precision, kmax=3, order_stencil=order)
    fresh = ft.Solver(pb, precision, kmax=3)
    s.debug_resident(1, getattr(ft, "RESIDENT_" + outcome))
    x, st = s.solve(rhs, tol=1e-8, k=3)
    y, su = streaming.solve(rhs, tol=1e-8, k=3)
    assert st["status"] == ft.CONVERGED and st["steps_executed"] == su["steps_executed"]
    assert bool((x == y).all())
    if outcome == "LATE":
        s.debug_resident(0)
        x, st = s.solve(rhs, tol=1e-8, k=3)
        y, su = fresh.solve(rhs, tol=1e-8, k=3)
        assert st["steps_executed"] == su["steps_executed"]
        assert bool((x == y).all())
    for h in (s, streaming, fresh):
        h.close()


@pytest.mark.parametrize("outcome", ["LATE", "REFUSED"])
@pytest.mark.parametrize("launch", [1, 2, 4])
@pytest.mark.parametrize("mesh", ["lat-lon", "octahedral"])
def test_batch_goes_on_streaming(ft, oracle_mod, mesh, launch, outcome):
    """One member's launches do not run from the given one on (the second starts
    at the flips of its step 6): every member ends as alone, with the flips
    before and after that."""
    print("[gpu-case] batch goes on streaming", mesh, launch, outcome, flush=True)
    pbs = ([Problem(64, 32, 8), Problem(40, 20, 17), Problem(33, 18, 8), Problem(64, 16, 16)] if mesh == "lat-lon"
           else [OctProblem(7, 21), OctProblem(9, 17), OctProblem(5, 30)])
    rhs = [I.rhs(pb, 40 + m) for m, pb in enumerate(pbs)]
    n = [pb.n for pb in pbs]
    plans = [[] for _ in pbs]
    plans[0] = [FaultEvent(6, "r", 52, start=0, count=n[0]), FaultEvent(6, "x", 40, start=0, count=n[0]),
                FaultEvent(31, "r", 62, idx=np.array([n[0] // 2])), FaultEvent(33, "e", 62, idx=np.array([3])),
                FaultEvent(60, "ap", 62, idx=np.array([n[0] - 1]))]
    plans[2] = [FaultEvent(9, "r", 52, start=0, count=n[2]), FaultEvent(47, "r", 62, idx=np.array([5]))]
    solvers = [ft.Solver(pb, kmax=3) for pb in pbs]
    solvers[0].debug_resident(launch, getattr(ft, "RESIDENT_" + outcome))
    xs, sts = ft.solve_batch(solvers, rhs, tols=[1e-10] * len(pbs), k=3, plans=plans)
    for m, pb in enumerate(pbs):
        _same_as_oracle(ft, _oracle(oracle_mod, pb), rhs[m], xs[m], sts[m], 3, plans[m])
    for s in solvers:
        s.close()
