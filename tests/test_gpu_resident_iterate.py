"""The iterate that the resident kernel updates in place: with the fault layer
off its buffer is the same from the second cycle on, and after a flip in x
inside a cycle from that cycle on.  The level counts put all the rows that a
half column lacks of its template into groups of their own (and one count on
either side), at up to four and at eight wavefronts a block, in both precisions.
13 steps (four cycles of three and a step) against the oracle's 13: FP64 to
1e-10.  In the mixed form the steps are one refinement round whose vectors are
rounded to binary32 (2^-24 = 6e-8): about ten roundings a step, 13 steps and a
growth of at most 100 between a vector's rounding and the iterate's give 1e-3;
one level of a column counted twice would be an error of a tenth or more."""
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


CASES = [("fp64", Problem(40, 20, nz)) for nz in (16, 17, 32, 33, 34, 49)] + \
    [("fp64", Problem(288, 117, nz)) for nz in (9, 17, 18)] + \
    [("mixed", Problem(40, 20, nz)) for nz in (33, 64, 65, 66, 80, 81, 82)] + \
    [("mixed", Problem(288, 117, nz)) for nz in (17, 18, 33)] + \
    [("fp64", OctProblem(9, 33)), ("mixed", OctProblem(9, 33)), ("mixed", OctProblem(9, 65)),
     ("mixed", OctProblem(88, 17))]


@pytest.mark.parametrize("how", ["fault layer off", "flip in x"])
@pytest.mark.parametrize("precision,pb", CASES, ids=lambda v: str(getattr(v, "shape", v)))
def test_iterate_updated_in_place(ft, oracle_mod, precision, pb, how):
    print("[gpu-case] iterate in place", precision, pb, how, flush=True)
    rhs = I.rhs(pb, 21)
    off = how == "fault layer off"
    # the sign of a third of the entries of x (the sum up to there, whatever its
    # rounding), which the detector does not see
    plan = None if off else [FaultEvent(5, "x", 63, start=0, count=pb.n // 3)]
    steps = 13
    o = (oracle_mod.OctOracle if isinstance(pb, OctProblem) else oracle_mod.Oracle)(pb)
    xo, so, _, _ = o.solve(rhs, tol=1e-14, k=3, plan=plan, ft=not off, max_steps=steps)
    opts = {} if precision == "fp64" else {"max_refinements": 1, "inner_max_steps": steps, "inner_tol": 1e-12}
    s = ft.Solver(pb, precision, kmax=3, ft=0 if off else 1, max_steps=steps, **opts)
    x, st = s.solve(rhs, tol=1e-14, k=3, plan=plan)
    s.close()
    assert st["steps_executed"] == so["steps_executed"] == steps
    assert st["detections"] == so["detections"] == 0
    assert st["events_applied"] == so["events_applied"] == (0 if off else 1)
    x = x.cpu().numpy().reshape(pb.nz, -1)
    xo = np.asarray(xo).reshape(pb.nz, -1)
    bar = 1e-10 if precision == "fp64" else 1e-3
    for k in range(pb.nz):   # level by level: one of them wrong is not averaged away
        assert np.linalg.norm(x[k] - xo[k]) <= bar * np.linalg.norm(xo[k]), (k, pb)
