"""The column pass, the batched column pass of members of different depths and
FT-GMRES beyond the cache against the oracle, at the sizes where they can go
wrong: level counts on either side of every template depth and of a group of
eight rows, one to three columns, a last wavefront nearly empty.  Bars as
elsewhere: P^{-1} to 1e-12 (1e-13 of the largest entry), solves with identical
decisions, steps within one and x within 1e-10 at equal step counts."""
import numpy as np
import pytest

from paper_2103_07210_amd import inputs as I
from paper_2103_07210_amd.inputs import FaultEvent, OctProblem, Problem

pytestmark = pytest.mark.gpu

LEVELS = [1, 2, 7, 8, 9, 15, 16, 17, 24, 25, 31, 32, 33, 40, 41, 48, 49, 56, 57, 63, 64, 65, 79, 80, 81, 95, 96]


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


def _rel(a, b):
    a, b = np.asarray(a).ravel(), np.asarray(b).ravel()
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("nz", LEVELS)
def test_column_solve_at_every_depth(ft, oracle_mod, nz):
    print("[gpu-case] column depth", nz, flush=True)
    for nx, ny in ((3, 1), (43, 3), (64, 2)):   # 3, 129 and 128 columns
        pb = Problem(nx, ny, nz, hill_amp=0.9, hill_lon=0.3)
        s = ft.Solver(pb, kmax=2)
        r = np.random.default_rng(nz).uniform(-1, 1, pb.shape)
        e = s.apply_pinv(r).cpu().numpy()
        ref = oracle_mod.Oracle(pb).apply_pinv(r)
        np.testing.assert_allclose(e, ref, rtol=1e-12, atol=1e-13 * np.abs(ref).max())
        s.close()


@pytest.mark.parametrize("streaming", [False, True])
@pytest.mark.parametrize("mesh", ["lat-lon", "octahedral"])
def test_batch_of_different_depths(ft, oracle_mod, mesh, streaming):
    """Every member's columns are solved at its own level count whatever the
    deepest member's; flips in r and L(p) cover the member's whole grid."""
    print("[gpu-case] batch depths", mesh, streaming, flush=True)
    if mesh == "lat-lon":
        pbs = [Problem(33, 9, nz, hill_lon=0.4 * m, hill_amp=0.2 + 0.1 * m)
               for m, nz in enumerate((5, 9, 16, 17, 33, 64))]
    else:
        pbs = [OctProblem(n, nz) for n, nz in ((4, 5), (7, 17), (5, 33), (9, 51))]
    rhs = [I.rhs(pb, 40 + m) for m, pb in enumerate(pbs)]
    plans = [[] for _ in pbs]
    plans[1] = [FaultEvent(5, "r", 62, idx=np.array([pbs[1].n - 1]))]
    plans[2] = [FaultEvent(6, "ap", 62, idx=np.array([pbs[2].n - 2]))]
    solvers = [ft.Solver(pb, kmax=3) for pb in pbs]
    if streaming:
        solvers[0].set_options(order_stencil=1)
    xs, sts = ft.solve_batch(solvers, rhs, tols=[1e-10] * len(pbs), k=3, plans=plans)
    for m, pb in enumerate(pbs):
        o = (oracle_mod.Oracle if mesh == "lat-lon" else oracle_mod.OctOracle)(pb)
        _, so, logo, _ = o.solve(rhs[m], tol=1e-10, k=3, plan=plans[m])
        assert sts[m]["status"] == ft.CONVERGED, m
        assert abs(sts[m]["steps_executed"] - so["steps_executed"]) <= 1, m
        assert _decisions(sts[m]["log"]) == _decisions(logo), m
        xe, _, _, _ = o.solve(rhs[m], tol=1e-13, k=3, plan=plans[m], max_steps=sts[m]["steps_executed"])
        assert _rel(xs[m].cpu().numpy(), xe) <= 1e-10, m
    for s in solvers:
        s.close()


def test_gmres_beyond_the_cache(ft, oracle_mod):
    """17 basis vectors of 16.8 MB exceed the cache, so they are read with the
    non-temporal hint: 20 steps (a full cycle and the next one's start)."""
    print("[gpu-case] gmres non-temporal", flush=True)
    pb = Problem(256, 128, 64)
    rhs = I.rhs(pb, 3)
    s = ft.Solver(pb, kmax=16, method=ft.METHOD_GMRES, max_steps=20)
    x, st = s.solve(rhs, tol=1e-10, k=16)
    xo, so, logo, _ = oracle_mod.Oracle(pb).solve(rhs, tol=1e-10, k=16, max_steps=20, method="gmres")
    assert st["steps_executed"] == so["steps_executed"] == 20
    assert _decisions(st["log"]) == _decisions(logo)
    assert _rel(x.cpu().numpy(), xo) <= 1e-10
    s.close()


@pytest.mark.parametrize("levels", [0, 8])
def test_octahedral_levels_per_block(ft, oracle_mod, levels):
    """O_110 x 40 is the smallest mesh with enough blocks for 8 levels: 4 by
    default, 8 where asked for; 12 steps (two cycles and a half) of either."""
    print("[gpu-case] octahedral levels per block", levels, flush=True)
    pb = OctProblem(110, 40)
    rhs = I.rhs(pb, 5)
    s = ft.Solver(pb, kmax=5, max_steps=12, levels_per_block=levels)
    assert s.tiling()["levels_per_block"] == (levels or 4)
    x, st = s.solve(rhs, tol=1e-10, k=5)
    xo, so, logo, _ = oracle_mod.OctOracle(pb).solve(rhs, tol=1e-10, k=5, max_steps=12)
    assert st["steps_executed"] == so["steps_executed"] == 12
    assert _decisions(st["log"]) == _decisions(logo)
    assert _rel(x.cpu().numpy(), xo) <= 1e-10
    s.close()


@pytest.mark.parametrize("ny,nz", [(2048, 64), (2052, 64), (2056, 63)])
@pytest.mark.parametrize("k", [4, 16])
def test_folded_partials(ft, oracle_mod, ny, nz, k):
    """16384 stencil blocks (reduced by one block each) and 16416 and 16448
    (folded first): 20 steps, one of them with a flip in e."""
    print("[gpu-case] folded partials", ny, nz, k, flush=True)
    pb = Problem(3, ny, nz, hill_amp=0.6)
    rhs = I.rhs(pb, 9)
    plan = [FaultEvent(6, "e", 62, idx=np.array([pb.n // 2]))]
    s = ft.Solver(pb, kmax=k, max_steps=20, levels_per_block=2)
    x, st = s.solve(rhs, tol=1e-13, k=k, plan=plan)
    xo, so, logo, _ = oracle_mod.Oracle(pb).solve(rhs, tol=1e-13, k=k, plan=plan, max_steps=20)
    assert st["steps_executed"] == so["steps_executed"] == 20
    assert _decisions(st["log"]) == _decisions(logo)
    assert _rel(x.cpu().numpy(), xo) <= 1e-10
    s.close()
