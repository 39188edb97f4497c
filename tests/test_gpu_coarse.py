"""The levels of a cycle at the sizes where their kernels or launches change: the two-launch
form of the coarse levels (coarsest grids of more than 128 points) against the FP64 oracle,
the march lengths of the 3D legs against each other."""
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
