"""Which solves and batches run in the resident kernel: a launch of it forced to
end as broken fails the solve, so a solve that succeeds did not make one."""
import numpy as np
import pytest

from paper_2103_07210_amd import inputs as I
from paper_2103_07210_amd.inputs import OctProblem, Problem

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


def _resident(ft, solvers, call):
    for s in solvers:
        s.debug_resident(1, ft.RESIDENT_BROKEN)
    try:
        call()
        return False
    except ft.FtgcrError as e:
        assert e.code == ft.E_HIP
        return True
    finally:
        for s in solvers:
            s.debug_resident(0)


def test_tilings_asked_for_stream(ft):
    print("[gpu-case] tilings asked for", flush=True)
    pbs = [Problem(64, 32, 8), Problem(33, 18, 8)]
    rhs = [I.rhs(pb, 50 + m) for m, pb in enumerate(pbs)]
    solvers = [ft.Solver(pb, kmax=3, max_steps=9) for pb in pbs]

    def single():
        return _resident(ft, solvers[:1], lambda: solvers[0].solve(rhs[0], tol=1e-10, k=3))

    def batch():
        return _resident(ft, solvers, lambda: ft.solve_batch(solvers, rhs, tols=[1e-10] * 2, k=3))

    assert single() and batch()
    solvers[0].set_options(levels_per_block=4)
    assert not single() and not batch()
    solvers[0].set_options(levels_per_block=0, batch_levels_per_block=4)
    assert single() and not batch()
    # the autotuner's choice is of the streaming kernels' tiling alone
    kc = ft.autotune_batch(solvers, rhs, k=3, steps=6)
    assert solvers[0].options()["batch_levels_per_block"] == kc
    assert batch()
    solvers[0].set_options(batch_levels_per_block=2 * kc)
    assert not batch()
    solvers[0].set_options(batch_levels_per_block=kc)   # asked for now
    assert not batch()
    solvers[0].set_options(batch_levels_per_block=0)
    assert batch()
    for s in solvers:
        s.close()


def test_handles_of_other_sizes_and_kmax(ft):
    """Handles that share a kernel and need more or less LDS of it keep their
    launches whatever handle came last."""
    print("[gpu-case] handles of other kmax", flush=True)
    pbs = [(Problem(64, 32, 8), 16), (Problem(512, 16, 8), 4), (Problem(40, 8, 8), 1)]
    solvers = [ft.Solver(pb, kmax=k, max_steps=20) for pb, k in pbs]
    rhs = [I.rhs(pb, 52) for pb, _ in pbs]
    for order in ((0, 1, 2), (2, 1, 0)):
        for m in order:
            for k in {1, pbs[m][1]}:
                assert _resident(ft, [solvers[m]], lambda: solvers[m].solve(rhs[m], tol=1e-30, k=k))
                x, st = solvers[m].solve(rhs[m], tol=1e-30, k=k)
                one = ft.Solver(pbs[m][0], kmax=pbs[m][1], max_steps=20)
                y, _ = one.solve(rhs[m], tol=1e-30, k=k)
                assert st["steps_executed"] == 20 and bool((x == y).all())
                one.close()
    for s in solvers:
        s.close()


# either side of where a form of the kernel stops paying
FORMS = [("fp64", OctProblem(87, 17), False), ("fp64", OctProblem(119, 20), True), ("fp64", Problem(250, 129, 17), True),
         ("mixed", OctProblem(87, 33), False), ("mixed", OctProblem(119, 33), True), ("mixed", OctProblem(87, 57), False),
         ("mixed", Problem(250, 129, 41), True), ("mixed", Problem(250, 129, 57), False),
         ("mixed", OctProblem(12, 81), False), ("mixed", OctProblem(12, 80), True), ("mixed", Problem(64, 32, 96), True)]


@pytest.mark.parametrize("precision,pb,resident", FORMS, ids=lambda v: str(getattr(v, "shape", v)))
def test_forms_that_pay(ft, oracle_mod, precision, pb, resident):
    """Whichever runs, the first steps are the oracle's (mixed: one round of 8
    steps, vectors rounded to 2^-24, ten roundings a step and a growth of 100)."""
    print("[gpu-case] forms", precision, pb, flush=True)
    rhs = I.rhs(pb, 53)
    opts = {} if precision == "fp64" else {"max_refinements": 1, "inner_max_steps": 8, "inner_tol": 1e-12}
    s = ft.Solver(pb, precision, kmax=3, max_steps=8, **opts)
    assert _resident(ft, [s], lambda: s.solve(rhs, tol=1e-14, k=3)) == resident
    x, st = s.solve(rhs, tol=1e-14, k=3)
    o = (oracle_mod.OctOracle if isinstance(pb, OctProblem) else oracle_mod.Oracle)(pb)
    xo, _, _, _ = o.solve(rhs, tol=1e-14, k=3, max_steps=8)
    assert st["steps_executed"] == 8
    x, xo = x.cpu().numpy().ravel(), np.asarray(xo).ravel()
    assert np.linalg.norm(x - xo) <= (1e-10 if precision == "fp64" else 1e-3) * np.linalg.norm(xo)
    s.close()


@pytest.mark.parametrize("vec,every,resident", [("x", 1, False), ("x", 2, True), ("e", 2, False), ("e", 4, True)])
def test_events_in_close_succession(ft, oracle_mod, vec, every, resident):
    """Launches between events where they pay; the same solve either way."""
    print("[gpu-case] events", vec, every, flush=True)
    pb = Problem(256, 128, 32)
    rhs = I.rhs(pb, 54)
    plan = [I.FaultEvent(t, vec, 20, start=t, count=1) for t in range(2, 40, every)]
    s = ft.Solver(pb, kmax=3, max_steps=39)
    assert _resident(ft, [s], lambda: s.solve(rhs, tol=1e-14, k=3, plan=plan[:-1]))
    s.set_options(max_steps=38)
    assert _resident(ft, [s], lambda: s.solve(rhs, tol=1e-14, k=3, plan=plan)) == resident
    x, st = s.solve(rhs, tol=1e-14, k=3, plan=plan)
    xo, so, _, _ = oracle_mod.Oracle(pb).solve(rhs, tol=1e-14, k=3, plan=plan, max_steps=38)
    assert st["steps_executed"] == so["steps_executed"] == 38
    assert st["detections"] == so["detections"] == 0
    assert st["events_applied"] == so["events_applied"]
    x, xo = x.cpu().numpy().ravel(), np.asarray(xo).ravel()
    assert np.linalg.norm(x - xo) <= 1e-10 * np.linalg.norm(xo)
    s.close()


BATCHES = [([Problem(480, 100, 5)] * 6, False), ([Problem(480, 100, 5)] * 2, True), ([OctProblem(60, 17)] * 4, False),
           ([OctProblem(16, 51)] * 4, True), ([Problem(128, 64, 16)] * 6, True),
           ([Problem(384, 128, 24), Problem(64, 32, 8)], True)]


@pytest.mark.parametrize("pbs,resident", BATCHES, ids=lambda v: str(len(v)) + "x" + str(v[0].shape) if isinstance(v, list) else str(v))
def test_batches_that_pay(ft, oracle_mod, pbs, resident):
    """Whichever runs, every member's first steps are the oracle's."""
    print("[gpu-case] batches", len(pbs), pbs[0], flush=True)
    solvers = [ft.Solver(pb, kmax=3, max_steps=8) for pb in pbs]
    rhs = [I.rhs(pb, 55 + m) for m, pb in enumerate(pbs)]
    assert _resident(ft, solvers, lambda: ft.solve_batch(solvers, rhs, tols=[1e-14] * len(pbs), k=3)) == resident
    xs, sts = ft.solve_batch(solvers, rhs, tols=[1e-14] * len(pbs), k=3)
    for m in {0, len(pbs) - 1}:
        o = (oracle_mod.OctOracle if isinstance(pbs[m], OctProblem) else oracle_mod.Oracle)(pbs[m])
        xo, _, _, _ = o.solve(rhs[m], tol=1e-14, k=3, max_steps=8)
        assert sts[m]["steps_executed"] == 8
        x, xo = xs[m].cpu().numpy().ravel(), np.asarray(xo).ravel()
        assert np.linalg.norm(x - xo) <= 1e-10 * np.linalg.norm(xo)
    for s in solvers:
        s.close()


@pytest.mark.parametrize("vec", ["x", "r", "ap", "e"])
@pytest.mark.parametrize("every", [1, 3, 30])
@pytest.mark.parametrize("who", ["one", "all"])
def test_batch_with_events(ft, oracle_mod, who, every, vec):
    """Events in close succession in streaming launches of all members, the steps
    after them and sparse events resident: every member as alone."""
    print("[gpu-case] batch events", who, every, vec, flush=True)
    pbs = [Problem(64, 32, 8), Problem(40, 20, 15), Problem(64, 32, 8, hill_lon=0.4)]
    rhs = [I.rhs(pb, 58 + m) for m, pb in enumerate(pbs)]
    plans = [[I.FaultEvent(t, vec, 51, start=t, count=5) for t in range(2 + m, 62, every)] if m == 1 or who == "all" else []
             for m in range(len(pbs))]
    plans[1].append(I.FaultEvent(70, "r", 62, start=3, count=1))
    solvers = [ft.Solver(pb, kmax=3) for pb in pbs]
    xs, sts = ft.solve_batch(solvers, rhs, tols=[1e-10] * len(pbs), k=3, plans=plans)
    for m, pb in enumerate(pbs):
        o = oracle_mod.Oracle(pb)
        _, so, logo, _ = o.solve(rhs[m], tol=1e-10, k=3, plan=plans[m])
        assert sts[m]["status"] == so["status"] == ft.CONVERGED
        assert sts[m]["events_applied"] == so["events_applied"]
        assert [(d["step"], d["nu"], d["action"]) for d in sts[m]["log"]] == [(d["step"], d["nu"], d["action"]) for d in logo]
        assert abs(sts[m]["steps_executed"] - so["steps_executed"]) <= 1
        xe, _, _, _ = o.solve(rhs[m], tol=1e-14, k=3, plan=plans[m], max_steps=sts[m]["steps_executed"])
        x = xs[m].cpu().numpy().ravel()
        assert np.linalg.norm(x - xe.ravel()) <= 1e-10 * np.linalg.norm(xe)
    for s in solvers:
        s.close()
