"""Memory of a context: the coarsest inverse and the TV prox work in the Krylov basis, or, where it is
too small for the inverse, in memory of the call."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import synth
from oracle import inverse as oinv
from oracle.multigrid import Hierarchy

from .helpers import gpu_context, medium, oracle_problem, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


def test_coarsest_inverse_keeps_no_workspace():
    """33^2 coarsest points (a 65^2 grid): 19 MB of operator, 9 MB of inverse, a basis of 135 kB."""
    nmap = medium(49, seed=8)
    prob = oracle_problem(nmap, levels=2)
    hier = Hierarchy(prob)
    r = synth.complex_field((2, 33, 33), 72)
    with gpu_context(medium(49, seed=9), levels=2, max_batch=2, restart=1) as ctx:
        assert ctx.info.coarsest_n == 33
        before = ctx.info.workspace_bytes
        assert before < 8 * 1089 ** 2 + (4 << 20)  # the inverse, and fields of 65^2
        ctx.update_n(torch.tensor(nmap, dtype=torch.float32, device="cuda"))
        z = to_np(ctx.coarse_solve(to_dev(r)))
    ref = np.stack([hier.coarse_lu.solve(ri.ravel()).reshape(33, 33) for ri in r])
    # the bound of the other inverse tests: a 64-bit inverse rounded to 32 bits
    assert rel(z, ref) < 1e-6


def _bytes(ctx):
    from paper_2107_03679_amd import helm

    info = helm.HelmInfo()
    ctx.lib.helm_get_info(ctx._h, ctypes.byref(info))
    return info.workspace_bytes


# 12^3 interior on 17^3: 97 kB of prox fields, a basis of 432 kB with restart 10, of 79 kB with 1
@pytest.mark.parametrize("restart, own", [(10, 0), (1, (4 * 3 + 2) * 12 ** 3 * 4)])
def test_prox_between_solves(restart, own):
    nmap = medium(12, d=3, seed=4)
    v = np.random.default_rng(3).standard_normal((12, 12, 12)).astype(np.float32)
    with gpu_context(nmap, w=1, levels=3, max_batch=1, restart=restart, max_iters=100) as ctx:
        assert ctx.n_e == 17
        b = ctx.plane_wave_rhs(synth.directions_cone(1))
        x0, st0 = ctx.solve(b)
        before = _bytes(ctx)
        w = ctx.tv_prox(torch.tensor(v, device="cuda"), 0.3, lo=0.05, iters=20).cpu().numpy()
        assert _bytes(ctx) - before == own
        x, st = ctx.solve(b)
        ctx.update_n(torch.tensor(nmap, dtype=torch.float32, device="cuda"))
        x2, _ = ctx.solve(b)
    assert bool((x == x0).all()) and bool((x2 == x0).all()) and (st.iters == st0.iters).all()
    assert rel(w, oinv.tv_prox(v.astype(np.float64), 0.3, lo=0.05, iters=20)) < 2e-5
