"""A sensor's value has the same bits whatever batch it is formed in, and stays accurate where a launch
has many sensors and sources."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from oracle.farfield import sensor_matrix
from oracle.model import scattering_potential

from .helpers import gpu_context, medium, oracle_problem, rel, to_dev, to_np

pytestmark = pytest.mark.gpu


def _sensors(n, dim, M):
    v = np.random.default_rng(M).standard_normal((M, dim))
    return v / np.linalg.norm(v, axis=1, keepdims=True) * (n * np.sqrt(dim) / 2 + 3)


# 125^2: 26 chunks of 608 pixels, the last one partly filled; 256^2: 158 of 416
@pytest.mark.parametrize("dim, n, M", [(2, 125, 1200), (2, 256, 180), (3, 19, 70)])
def test_values_do_not_depend_on_the_batch(dim, n, M):
    nmap = medium(n, d=dim, seed=6)
    prob = oracle_problem(nmap, w=4, levels=4 if n > 60 else 2)
    sens = _sensors(n, dim, M)
    u = synth.complex_field((65, *prob.shape), 90).astype(np.complex64)
    r = synth.complex_field((65, M), 91).astype(np.complex64)
    with gpu_context(nmap, w=4, levels=prob.levels, max_batch=65, restart=1) as ctx:
        ctx.farfield_set(sens)
        y, (s, rhs) = ctx.farfield(to_dev(u)), ctx.farfield_adjoint(to_dev(r))
        for B in (1, 16, 17, 33):
            assert bool((ctx.farfield(to_dev(u[:B])) == y[:B]).all()), B
            sb, rb = ctx.farfield_adjoint(to_dev(r[:B]))
            assert bool((sb == s[:B]).all()) and bool((rb == rhs[:B]).all()), B
        last = ctx.farfield(to_dev(u[64:]))
        assert bool((last == y[64:]).all())
    few = slice(0, 40)
    G = sensor_matrix(prob, sens[few])
    inner = (slice(None),) + prob.interior_slices()
    ref = (scattering_potential(prob) * u)[inner].reshape(65, -1) @ G.T
    # single-precision G and sums: some 1200 roundings of a chunk's partial sums, which are a few
    # tenths of the value, in quadrature
    assert rel(to_np(y)[:, few], ref) < 2e-6


def test_many_sensors_keep_their_sums_short():
    """4096 sensors at 256^2: wavefronts enough with 8 chunks, but 64 of 1024 pixels are taken."""
    nmap = medium(256, seed=6)
    prob = oracle_problem(nmap, w=4, levels=4)
    sens = _sensors(256, 2, 4096)
    u = synth.complex_field((2, *prob.shape), 92).astype(np.complex64)
    with gpu_context(nmap, w=4, levels=4, max_batch=2, restart=1) as ctx:
        ctx.farfield_set(sens)
        y = to_np(ctx.farfield(to_dev(u)))
    few = slice(0, 4096, 200)
    inner = (slice(None),) + prob.interior_slices()
    ref = (scattering_potential(prob) * u)[inner].reshape(2, -1) @ sensor_matrix(prob, sens[few]).T
    assert rel(y[:, few], ref) < 2e-6  # some 2000 roundings of a chunk's partial sums, as above
