"""The levels of a cycle at the sizes where their kernels or launches change: the two-launch
form of the coarse levels (coarsest grids of more than 128 points) and the coarsest inverse
against the FP64 oracle, the march lengths of the 3D legs against each other."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle.multigrid import Hierarchy

from .helpers import gpu_context, medium, oracle_problem, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


# interior, levels, dim, right-hand sides -> coarse sizes (layer of 8 cells)
@pytest.mark.parametrize("n, levels, d, B", [
    (25, 3, 2, 3),   # 41, 21, 11^2: 121 points, one launch
    (29, 3, 2, 3),   # 45, 23, 12^2: 144 points, the first split
    (73, 4, 2, 2),   # 89, 45, 23, 12^2: two levels above the coarsest in the launch
    (77, 3, 2, 1),   # 93, 47, 24^2: 576 points, the last row block half full
    (5, 3, 3, 2),    # 21, 11, 6^3
    (13, 3, 3, 5),   # 29, 15, 8^3: 15^3 points in four passes of the workgroup
    (29, 3, 2, 60),  # over 256 workgroups of 32 rows: 64 rows each
    (77, 3, 2, 20),
    (13, 3, 3, 20),
])
def test_split_coarse_cycle_matches_oracle(n, levels, d, B):
    nmap = medium(n, seed=5, d=d)
    prob = oracle_problem(nmap, levels=levels)
    hier = Hierarchy(prob)
    r = synth.complex_field((B, *prob.shape), 70)
    with gpu_context(nmap, levels=levels, max_batch=B) as ctx:
        assert ctx.info.coarsest_n == hier.sizes[-1]
        z = to_np(ctx.precondition(to_dev(r)))
    ref = np.stack([hier.vcycle(ri.ravel()).reshape(prob.shape) for ri in r])
    # single precision through ~10 stages and a 64-bit inverse rounded to 32 bits: the bound the
    # other cycle tests use
    assert rel(z, ref) < 1e-5


@pytest.mark.parametrize("n, B", [(31, 48), (18, 200)])
def test_march_lengths_agree(n, B):
    """A batch marches through more planes per workgroup than one right-hand side (49^3: 16 and 2
    planes in the finest up-leg); every point is the same arithmetic, so the fields are equal
    (four levels: with three the coarsest grid is solved alone, by another kernel at B < 4)."""
    nmap = medium(n, seed=6, d=3)
    with gpu_context(nmap, levels=4, max_batch=B, restart=4, cycle=3) as ctx:
        r = to_dev(synth.complex_field((1, *ctx.grid_shape()), 71))
        one = ctx.precondition(r)
        many = ctx.precondition(r.expand(B, *ctx.grid_shape()).contiguous())
        assert bool((many == one).all())


# coarsest grids of 25 (one 32-point block), 36, 256 (whole blocks), 529, 64 and 343 points
@pytest.mark.parametrize("n, levels, d", [(49, 5, 2), (65, 5, 2), (105, 4, 2), (161, 4, 2), (9, 4, 3), (33, 4, 3)])
def test_coarsest_inverse_matches_oracle(n, levels, d):
    nmap = medium(n, seed=8, d=d)
    prob = oracle_problem(nmap, levels=levels)
    hier = Hierarchy(prob)
    diag = hier.K[-1].diagonal()
    assert np.all(np.abs(diag) > np.asarray(abs(hier.K[-1]).sum(axis=1)).ravel() - np.abs(diag))  # inverted on the GPU
    shape = (hier.sizes[-1],) * d
    r = synth.complex_field((5, *shape), 72)
    other = medium(n, seed=9, d=d)
    with gpu_context(other, levels=levels, max_batch=5) as ctx:
        import torch

        ctx.update_n(torch.tensor(nmap, dtype=torch.float32, device="cuda"))
        z = to_np(ctx.coarse_solve(to_dev(r)))
    ref = np.stack([hier.coarse_lu.solve(ri.ravel()).reshape(shape) for ri in r])
    # the 64-bit inverse rounded to 32 bits and a single-precision product of a well-conditioned matrix
    assert rel(z, ref) < 1e-6


@pytest.mark.parametrize("n, levels, B", [(161, 4, 1), (161, 4, 3), (161, 4, 8), (161, 4, 17), (49, 5, 9)])
def test_coarse_products_agree(n, levels, B):
    """The product's tiles of 1, 4, 8 and 16 right-hand sides (529 points: two passes over the
    columns, the last rows' workgroup with one row; 25: one pass) against the oracle and, sums in
    the same order, each other."""
    nmap = medium(n, seed=8)
    prob = oracle_problem(nmap, levels=levels)
    hier = Hierarchy(prob)
    shape = (hier.sizes[-1],) * 2
    r = synth.complex_field((B, *shape), 73)
    with gpu_context(nmap, levels=levels, max_batch=B, restart=1) as ctx:
        z = ctx.coarse_solve(to_dev(r))
        assert bool((ctx.coarse_solve(to_dev(r[:1])) == z[:1]).all())
    ref = np.stack([hier.coarse_lu.solve(ri.ravel()).reshape(shape) for ri in r])
    assert rel(to_np(z), ref) < 1e-6
