"""FT-GMRES on either side of the vector length from which the Krylov vectors are
read with the non-temporal hint (32 MiB, 4194304 cells): a cycle of six steps and
half the next against the oracle, x within 1e-10."""
import numpy as np
import pytest

from paper_2103_07210_amd import inputs as I
from paper_2103_07210_amd.inputs import OctProblem, Problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pb", [Problem(256, 172, 95), Problem(256, 176, 94), OctProblem(104, 89), OctProblem(104, 90)],
                         ids=lambda v: str(v.shape))
def test_gmres_around_the_hint(oracle_mod, pb):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_2103_07210_amd import ftgcr as ft
    print("[gpu-case] gmres hint", pb, flush=True)
    rhs = I.rhs(pb, 3)
    s = ft.Solver(pb, kmax=6, method=ft.METHOD_GMRES, max_steps=9)
    x, st = s.solve(rhs, tol=1e-10, k=6)
    o = (oracle_mod.OctOracle if isinstance(pb, OctProblem) else oracle_mod.Oracle)(pb)
    xo, so, logo, _ = o.solve(rhs, tol=1e-10, k=6, max_steps=9, method="gmres")
    assert st["steps_executed"] == so["steps_executed"] == 9 and not st["log"] and not logo
    x, xo = x.cpu().numpy().ravel(), np.asarray(xo).ravel()
    assert np.linalg.norm(x - xo) <= 1e-10 * np.linalg.norm(xo)
    s.close()
