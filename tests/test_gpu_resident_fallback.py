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
