"""Calls that take another way through the library because of where their buffers lie or how many
right-hand sides they have: the same bits as the ordinary way."""
from __future__ import annotations

import ctypes
import json

import numpy as np
import pytest
import torch

import synth

from .helpers import gpu_context, medium

pytestmark = pytest.mark.gpu


# one region and several; w where v is, ahead of it and behind it
@pytest.mark.parametrize("shape, iters", [((40, 40), 9), ((130, 130), 19), ((30,) * 3, 7)])
@pytest.mark.parametrize("shift", [0, 3, -57])
def test_prox_into_its_own_input(shape, iters, shift):
    count = int(np.prod(shape))
    v = torch.randn(count, device="cuda", generator=torch.Generator(device="cuda").manual_seed(5))
    with gpu_context(medium(shape[0], d=len(shape)), w=4, levels=3, max_batch=1, restart=1) as ctx:
        want = ctx.tv_prox(v.view(shape), 0.3, lo=0.05, iters=iters)
        buf = torch.zeros(count + 200, device="cuda")
        buf[100:100 + count] = v
        out = buf[100 + shift:100 + shift + count]
        rc = ctx.lib.helm_tv_prox(ctx._h, ctypes.c_void_p(buf[100:].data_ptr()), 0.3, 0.05, iters,
                                  ctypes.c_void_p(out.data_ptr()))
        assert rc == 0 and bool((out.view(shape) == want).all())


@pytest.mark.parametrize("shape", [(2, 17, 45), (1, 6, 9, 33)])
def test_network_buffers_at_any_alignment(shape):
    """An input at 4, 8 and 12 bytes is converted first, at 16 the first layer reads it as it is; the
    output is written where it is."""
    from paper_2107_03679_amd import helm

    net = helm.Net(seed=3, dim=len(shape) - 1)
    x = torch.randn((*shape, 4), device="cuda", generator=torch.Generator(device="cuda").manual_seed(6))
    want = net.forward(x)
    call = net.lib.helm_net_forward3 if len(shape) == 4 else net.lib.helm_net_forward
    for off in (0, 1, 2, 3):
        xb = torch.zeros(x.numel() + 8, device="cuda")
        yb = torch.full((want.numel() + 8,), -7.0, device="cuda")
        xb[off:off + x.numel()] = x.reshape(-1)
        torch.cuda.synchronize()
        rc = call(net._h, *shape, ctypes.c_void_p(xb[off:].data_ptr()), ctypes.c_void_p(yb[off:].data_ptr()))
        assert rc == 0 and bool((yb[off:off + want.numel()] == want.reshape(-1)).all()), off
        assert bool((yb[:off] == -7.0).all()) and bool((yb[off + want.numel():] == -7.0).all())
    net.close()


# grid 257: 85 workgroups for each four right-hand sides, 1020 and 1105: both sides of the line at
# 1024 for the finest up-leg with the basis product
@pytest.mark.parametrize("B", [48, 49])
def test_untuned_matvec_shapes(tmp_path, B):
    nmap = medium(240, seed=15)
    with gpu_context(nmap, levels=4, max_batch=B, restart=3) as ctx:
        assert ctx.n_e == 257
        b = ctx.plane_wave_rhs(synth.directions_2d(B))
        x0, st0 = ctx.solve(b)
        assert st0.converged
        first, forced = tmp_path / "first.jsonl", tmp_path / "forced.jsonl"
        ctx.autotune(B, cache=str(first))
        line = json.loads(first.read_text().splitlines()[0])
        for mv in (0, 1):
            line["up"], line["down"], line["mv"], line["coarse_max"] = [0] * 4, [0] * 4, mv, 48 * 48
            forced.write_text(json.dumps(line) + "\n")
            assert ctx.autotune(B, cache=str(forced))["from_cache"]
            x, st = ctx.solve(b)
            assert bool((x == x0).all()) and (st.iters == st0.iters).all()
