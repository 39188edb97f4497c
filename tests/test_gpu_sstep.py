"""The s-step least squares at the ends of its restart lengths and where the basis ends early,
against sparse LU solutions."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle.model import ExactSolver

from .helpers import gpu_context, medium, oracle_problem, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


# interior, layer, levels, restart; 3 x 3 grid with 12 steps: the Krylov space (9 unknowns) is
# exhausted inside the cycle, so a Cholesky pivot vanishes
@pytest.mark.parametrize("n, w, levels, m", [(24, 8, 3, 1), (24, 8, 3, 2), (24, 8, 3, 11), (24, 8, 3, 12), (1, 1, 2, 12)])
def test_restart_lengths_solve(n, w, levels, m):
    nmap = medium(n, seed=4) if n > 1 else np.array([[1.4]])
    prob = oracle_problem(nmap, w=w, levels=levels)
    b = synth.complex_field((3, *prob.shape), 80)
    b[1] *= 1e-3
    with gpu_context(nmap, w=w, levels=levels, max_batch=3, restart=m, rtol=1e-7, max_iters=20000) as ctx:
        x, st = ctx.solve(to_dev(b))
        x = to_np(x)
    assert st.converged, st
    ex = ExactSolver(prob)
    for q in range(3):
        # residual 1e-7 times the inverse's amplification on these small grids (under 30)
        assert rel(x[q], ex.solve(b[q].astype(np.complex64).astype(np.complex128))) < 1e-5
