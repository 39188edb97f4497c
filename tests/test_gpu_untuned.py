"""Untuned 2D launches choose their shape by size: on both sides of the line (1024 workgroups)
the solve is the same, iterate for iterate, as with every shape forced."""
from __future__ import annotations

import json

import pytest

import synth

from .helpers import gpu_context, medium

pytestmark = pytest.mark.gpu


# grid 257: 85 workgroups of the finest up-leg per right-hand side (1020 and 1105), 255 for the
# matvec shape (groups of four); grid 33: a launch of one tile
@pytest.mark.parametrize("n, levels, B", [(16, 3, 1), (240, 4, 12), (240, 4, 13)])
def test_untuned_shapes(tmp_path, n, levels, B):
    nmap = medium(n, seed=15)
    with gpu_context(nmap, levels=levels, max_batch=B) as ctx:
        b = ctx.plane_wave_rhs(synth.directions_2d(B))
        x0, st0 = ctx.solve(b)
        assert st0.converged
        first, forced = tmp_path / "first.jsonl", tmp_path / "forced.jsonl"
        ctx.autotune(B, cache=str(first))
        line = json.loads(first.read_text().splitlines()[0])
        assert min(line["up"]) >= 0 and line["mv"] >= 0  # what is stored is always a shape
        for up, mv in ((0, 0), (1, 1)):
            line["up"], line["down"], line["mv"], line["coarse_max"] = [up] * levels, [0] * levels, mv, 48 * 48
            forced.write_text(json.dumps(line) + "\n")
            assert ctx.autotune(B, cache=str(forced))["from_cache"]
            x, st = ctx.solve(b)
            assert bool((x == x0).all()) and (st.iters == st0.iters).all()
