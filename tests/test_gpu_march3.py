"""The 3D marches (multigrid legs, level residual, basis product) at the edges of their tiles:
62 x 6 or 62 x 14 own points, 30 x 6 coarse points, chunks of 2 to 16 planes."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle.multigrid import Hierarchy

from .helpers import gpu_context, medium, oracle_problem, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


# grids 65, 33, 17, 9 (a second tile of three points in x) and 41, 21, 11, 6
@pytest.mark.parametrize("n", [56, 32])
@pytest.mark.parametrize("cycle", [1, 3])
def test_marches_match_oracle_and_flat_kernels(n, cycle):
    nmap = medium(n, d=3, seed=11)
    prob = oracle_problem(nmap, w=4, levels=4)
    hier = Hierarchy(prob)
    r = synth.complex_field((2, *prob.shape), 90)
    gamma = [2, 1, 1, 1] if cycle == 3 else 1
    ref = np.stack([hier.cycle(ri.ravel(), None, 0, gamma).reshape(prob.shape) for ri in r])
    for fused in (1, 0):
        with gpu_context(nmap, w=4, levels=4, max_batch=2, cycle=cycle, fused=fused, coarse_single_launch=0) as ctx:
            assert ctx.n_e == n + 9
            z = to_np(ctx.precondition(to_dev(r)))
        assert rel(z, ref) < 1e-5  # the bound the other 3D cycle tests use


def test_tall_and_low_tiles_agree():
    """48 right-hand sides on 65^3 take 14 rows a workgroup on the finest level, one takes 6;
    every point is the same arithmetic, so the fields are equal."""
    nmap = medium(56, d=3, seed=11)
    with gpu_context(nmap, w=4, levels=4, max_batch=48, restart=2, cycle=3) as ctx:
        r = to_dev(synth.complex_field((1, *ctx.grid_shape()), 91))
        one = ctx.precondition(r)
        many = ctx.precondition(r.expand(48, *ctx.grid_shape()).contiguous())
        assert bool((many == one).all())


@pytest.mark.parametrize("n, B", [(56, 1), (32, 3), (56, 24)])
def test_basis_product(n, B):
    """The s-step solver's basis product (low tiles, and tall ones at 24 right-hand sides) against
    the other Krylov method, which forms A z by another kernel: both end at the same solution to the
    tolerance they solve to (1e-6, each its own error)."""
    from paper_2107_03679_amd import helm

    nmap = medium(n, d=3, seed=12)
    sols = []
    for krylov in (helm.KRYLOV_SSTEP, helm.KRYLOV_FGMRES):
        with gpu_context(nmap, w=4, levels=4, max_batch=B, krylov=krylov) as ctx:
            b = ctx.plane_wave_rhs(synth.directions_cone(B))
            x, st = ctx.solve(b)
            assert st.converged and np.all(st.rel_res_true <= 1e-6)
            sols.append(to_np(x))
    assert rel(sols[0], sols[1]) < 1e-4
