"""The sensor operator's products at the edges of their tiles, against the FP64 oracle."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle.farfield import sensor_matrix
from oracle.model import scattering_potential

from .helpers import gpu_context, medium, oracle_problem, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


# odd pixel counts, the last sensor tile and pass (128 sensors) and each right-hand-side group partly filled
@pytest.mark.parametrize("dim, n, M, B", [(2, 11, 1, 1), (2, 11, 130, 17), (2, 33, 67, 33), (2, 16, 128, 64), (3, 5, 40, 16),
                                          (3, 7, 131, 40)])
def test_products_at_tile_edges(dim, n, M, B):
    w, levels = 4, 2
    nmap = medium(n, d=dim, seed=6)
    prob = oracle_problem(nmap, w=w, levels=levels)
    rng = np.random.default_rng(M)
    v = rng.standard_normal((M, dim))
    sens = v / np.linalg.norm(v, axis=1, keepdims=True) * (n * np.sqrt(dim) / 2 + 3)
    G = sensor_matrix(prob, sens)
    u = synth.complex_field((B, *prob.shape), 90).astype(np.complex64)
    r = synth.complex_field((B, M), 91).astype(np.complex64)
    with gpu_context(nmap, w=w, levels=levels, max_batch=B, restart=1) as ctx:
        ctx.farfield_set(sens)
        y = to_np(ctx.farfield(to_dev(u)))
        s, rhs = (to_np(a) for a in ctx.farfield_adjoint(to_dev(r)))
    f = scattering_potential(prob)
    inner = (slice(None),) + prob.interior_slices()
    ref = (f * u)[inner].reshape(B, -1) @ G.T
    sref = np.zeros((B, *prob.shape), dtype=complex)
    sref[inner] = (r.astype(complex) @ G.conj()).reshape(B, *(n,) * dim)
    # single-precision G and sums of at most 1089 terms
    assert rel(y, ref) < 2e-6
    assert rel(s, sref) < 2e-6 and rel(rhs, f * sref) < 2e-6
    assert not np.any(s[np.broadcast_to(~prob.interior_mask(), s.shape)])
