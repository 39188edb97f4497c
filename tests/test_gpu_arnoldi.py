"""The Arnoldi step at the sizes where it changes: up to 64 blocks of a right-hand side (131072
points) the update forms the coefficients itself, beyond a launch of its own does."""
from __future__ import annotations

import numpy as np
import pytest

import synth

from .helpers import gpu_context, medium, rel, to_np

pytestmark = pytest.mark.gpu


# grids 25 (one block), 361 (64 blocks, the last one ragged) and 369 (67)
@pytest.mark.parametrize("n, levels", [(8, 3), (344, 4), (352, 4)])
@pytest.mark.parametrize("reorth", [0, 1])
@pytest.mark.parametrize("restart", [3, 30])
def test_arnoldi_step(n, levels, reorth, restart):
    """Both Krylov methods meet the target of 1e-6 by the float-float residual; their solutions
    agree to 200 times that (the residual's amplification in the error)."""
    from paper_2107_03679_amd import helm

    nmap = medium(n, seed=14)
    with gpu_context(nmap, levels=levels, max_batch=2, krylov=helm.KRYLOV_SSTEP) as ctx:
        b = ctx.plane_wave_rhs(synth.directions_2d(2))
        ref, st = ctx.solve(b)
        assert st.converged
    with gpu_context(nmap, levels=levels, max_batch=2, krylov=helm.KRYLOV_FGMRES, reorth=reorth, restart=restart) as ctx:
        x, st = ctx.solve(b)
        assert st.converged and np.all(st.rel_res_true <= 1e-6)
    assert rel(to_np(x), to_np(ref)) < 2e-4
