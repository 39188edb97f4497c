"""One restart of GMRES beside the FP64 oracle: after m steps both hold the minimiser over the same
space, so that a wrong basis vector, product or coefficient shows in the solution at once (a whole
solve only takes more cycles).  Sizes where the basis product (3D marches: low tiles, tall ones at
24 right-hand sides) and the Arnoldi step (up to 64 blocks, and beyond) change."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle import krylov as okrylov
from oracle.discretization import helmholtz_matrix
from oracle.multigrid import Hierarchy

from .helpers import gpu_context, medium, oracle_problem, rel, to_dev, to_np

pytestmark = pytest.mark.gpu

M = 4


def one_restart(nmap, w, levels, B, check, **opts):
    """Solutions and residuals of one restart against the oracle's for the right-hand sides `check`."""
    from paper_2107_03679_amd import helm

    prob = oracle_problem(nmap, w=w, levels=levels)
    hier = Hierarchy(prob)
    a = helmholtz_matrix(prob)
    b = synth.complex_field((B, *prob.shape), 33)
    with gpu_context(nmap, w=w, levels=levels, max_batch=B, restart=M, max_iters=M, **opts) as ctx:
        x, st = ctx.solve(to_dev(b))
        x = to_np(x)
    sstep = opts["krylov"] == helm.KRYLOV_SSTEP
    solve = okrylov.sstep_gmres if sstep else okrylov.fgmres
    precond = lambda r: hier.cycle(r, None, 0, 1)  # noqa: E731
    for q in check:
        rhs = prob.h ** 2 * b[q].ravel()
        ref, info = solve(lambda v: a @ v, precond, rhs, rtol=1e-6, restart=M, max_iters=M)
        basis = [rhs]
        for _ in range(M):
            basis.append(a @ precond(basis[-1]))
        s = np.linalg.svd(np.array([v / np.linalg.norm(v) for v in basis]), compute_uv=False)
        # a basis vector in single precision goes through some 100 roundings a point (the cycle's
        # levels and the product); the least squares amplify that by the condition of the basis
        tol = 100 * 2.0 ** -24 * s[0] / s[-1]
        assert tol < 0.01
        assert st.iters[q] == M and info.iters == M
        assert abs(st.rel_res_true[q] / info.rel_res_true - 1) < tol, (q, tol, st.rel_res_true[q], info.rel_res_true)
        assert rel(x[q].ravel(), ref) < tol, (q, tol, rel(x[q].ravel(), ref))


@pytest.mark.parametrize("krylov", ["SSTEP", "FGMRES"])
@pytest.mark.parametrize("n, B", [(56, 1), (32, 3), (56, 24)])
def test_3d(n, B, krylov):
    from paper_2107_03679_amd import helm

    one_restart(medium(n, d=3, seed=12), 4, 4, B, {0, B - 1}, krylov=getattr(helm, "KRYLOV_" + krylov))


# grids 25 (one block), 361 (64 blocks, the last one ragged) and 369 (67)
@pytest.mark.parametrize("n, levels", [(8, 3), (344, 4), (352, 4)])
@pytest.mark.parametrize("krylov, reorth", [("SSTEP", 0), ("FGMRES", 0), ("FGMRES", 1)])
def test_2d(n, levels, krylov, reorth):
    from paper_2107_03679_amd import helm

    one_restart(medium(n, seed=14), 8, levels, 2, {0, 1}, krylov=getattr(helm, "KRYLOV_" + krylov), reorth=reorth)
