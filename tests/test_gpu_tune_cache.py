"""Lines of the autotuner's cache without a shape for the fused finest up-leg + basis matvec, or with
one outside the table: the first shape, in a context of its own."""
from __future__ import annotations

import json

import pytest

import synth

from .helpers import gpu_context, medium

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mv", [None, 99, -1])
def test_line_without_a_valid_matvec_shape(tmp_path, mv):
    nmap = medium(40, seed=3)
    first, edited = tmp_path / "first.jsonl", tmp_path / "edited.jsonl"
    with gpu_context(nmap, max_batch=2) as ctx:
        ctx.autotune(2, cache=str(first))
        b = ctx.plane_wave_rhs(synth.directions_2d(2))
        x0, st0 = ctx.solve(b)
    line = json.loads(first.read_text())
    del line["mv"]
    if mv is not None:
        line["mv"] = mv
    edited.write_text(json.dumps(line) + "\n")
    with gpu_context(nmap, max_batch=2) as ctx:
        t = ctx.autotune(2, cache=str(edited))
        assert t["from_cache"] and (t["up_mv_rows"], t["up_mv_rhs_per_block"]) == (16, 4)
        x, st = ctx.solve(b)
        assert bool((x == x0).all()) and (st.iters == st0.iters).all()
