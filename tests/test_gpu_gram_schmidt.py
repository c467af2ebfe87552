"""The Gram-Schmidt kernels of the Lanczos driver at the edges of their tiles (needs an MI355X).

A run of `steps` Lanczos steps orthogonalises against 1 ... steps vectors, so steps one past 64, 128
and 256 cross every change of tile (64, 32 and 16 elements, then update and dots in two launches),
on a lattice whose vectors have fewer tiles than the launch has blocks and on one with a ragged
site block.  With full reorthogonalisation the computed T is that of an operator within a few
hundred roundings (steps * 2^-53 ~ 3e-14) of A, so its extreme eigenvalues agree with the oracle's to
1e-11 lmax; the leading coefficients, before any Ritz value has converged, to 1e-10 of their size.
"""
import numpy as np
import pytest

import synth
from oracle import solvers

pytestmark = pytest.mark.gpu

lq = pytest.importorskip("paper_1312_3265_amd")


@pytest.mark.parametrize("dims,formulation,steps", [
    ((4, 4, 4, 4), synth.WILSON, 1), ((4, 4, 4, 4), synth.STAGGERED_WILSON, 9),
    ((4, 4, 4, 4), synth.WILSON, 65), ((4, 4, 4, 4), synth.WILSON, 129),
    ((4, 4, 4, 4), synth.WILSON, 258), ((6, 4, 6, 8), synth.STAGGERED_WILSON, 66),
])
def test_lanczos_across_the_tile_changes(dims, formulation, steps):
    U = synth.gauge_field(dims, "haar", 1000)
    g = lq.Gauge(lq.Lattice(dims), U)
    v0 = synth.gaussian_field(dims, formulation, 7)
    res = lq.condition_number(g, formulation, 0.5, v0, steps=steps)
    lo, hi, _, (a, b) = solvers.condition_number(formulation, U, 0.5, v0, steps)
    assert res["steps"] == len(a)
    np.testing.assert_allclose(res["alpha"][:30], a[:30], rtol=1e-10)
    np.testing.assert_allclose(res["beta"][:29], b[:29], rtol=1e-10)
    assert abs(res["lmin"] - lo) <= 1e-11 * hi
    assert abs(res["lmax"] - hi) <= 1e-11 * hi


@pytest.mark.parametrize("dims,formulation,steps", [
    ((6, 6, 6, 6), synth.WILSON, 12),      # 1296 sites: a ragged block of 64
    ((6, 6, 8, 10), synth.WILSON, 40),     # 552 tiles of 64 elements on 512 blocks
    ((6, 6, 8, 10), synth.WILSON, 70),     # 1104 tiles of 32
])
def test_lanczos_with_more_than_one_tile_per_block(dims, formulation, steps):
    """Blocks that take a second tile use the other half of the double-buffered LDS; same bounds as
    above."""
    test_lanczos_across_the_tile_changes(dims, formulation, steps)
