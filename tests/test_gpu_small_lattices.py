"""Lattices at the edges of the 64-site and 256-site blocks (needs an MI355X).

Fields of up to 16384 sites are cut into blocks of one wavefront, and the staggered Wilson stencil
splits a site's terms over eight of them: 4^4 has fewer blocks than partials, 6^4 a ragged last
block, 16 x 16 x 8 x 8 is the largest such lattice and 8 x 8 x 8 x 34 the first beyond it.
Bounds: the matvecs' as in test_gpu_parity.py (FP64 1e-13, FP32 4e-6, 16-bit 1e-4 of the field's
largest component); batches bitwise.
"""
import numpy as np
import pytest

import synth
from oracle import staggered_wilson, wilson

pytestmark = pytest.mark.gpu

lq = pytest.importorskip("paper_1312_3265_amd")
torch = pytest.importorskip("torch")

MODS = {synth.WILSON: wilson, synth.STAGGERED_WILSON: staggered_wilson}
DIMS = [(4, 4, 4, 4), (6, 6, 6, 6), (16, 16, 8, 8), (8, 8, 8, 34)]


def _gauge(dims, bc=(1, 1, 1, 1), eo=0):
    U = synth.gauge_field(dims, "near_identity", 31, 0.436)
    return U, lq.Gauge(lq.Lattice(dims, bc), U,
                       lq.FEAT_CORNERS | lq.FEAT_F32 | lq.FEAT_Q16 | (lq.FEAT_EO if eo else 0))


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("formulation", [synth.WILSON, synth.STAGGERED_WILSON])
def test_matvecs_of_every_precision(formulation, dims):
    bc = (-1, 1, 1, -1)
    U, g = _gauge(dims, bc)
    psi = synth.gaussian_field(dims, formulation, 5)
    for dag in (False, True):
        ref = MODS[formulation].apply(U, psi, 0.1, 1.0, bc, dagger=dag)
        for prec, links, bound in ((lq.F64, 18, 1e-13), (lq.F64, 12, 1e-13), (lq.F32, 12, 4e-6),
                                   (lq.F32, 18, 4e-6), (lq.Q16, 12, 1e-4), (lq.Q16, 18, 1e-4)):
            out = lq.apply(g, formulation, 0.1, psi, op=lq.OP_MDAG if dag else lq.OP_M,
                           precision=prec, links=links).cpu().numpy()
            assert np.abs(out - ref).max() <= bound * np.abs(ref).max(), (prec, links, dag)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("formulation", [synth.WILSON, synth.STAGGERED_WILSON])
def test_batches_are_bitwise_single_systems(formulation, dims, monkeypatch):
    """Three systems in one, two and four per thread (and, Wilson with 18-real links, four across
    the lanes) give each the bits it has alone."""
    U, g = _gauge(dims)
    chis = np.stack([synth.z2_source(dims, formulation, 70 + s) for s in range(3)])
    ms = [0.3, 0.4, 0.5]
    for prec in (lq.F32, lq.Q16):
        opts = lq.solve_opts(precision=prec, links=18, poll_interval=8)
        monkeypatch.setenv("LQ_LAUNCH", "1,1")
        alone = [lq.cg_solve_batch(g, formulation, [m], chis[k:k + 1], [1e-8], opts=opts)[0][0]
                 for k, m in enumerate(ms)]
        for K in (1, 2, 4) + ((8,) if formulation == synth.WILSON else ()):
            monkeypatch.setenv("LQ_LAUNCH", f"{K},0")
            x, infos = lq.cg_solve_batch(g, formulation, ms, chis, [1e-8] * 3, opts=opts)
            assert all(i["status"] == lq.OK and i["true_residual"] <= 1e-8 for i in infos)
            for k in range(3):
                assert torch.equal(x[k], alone[k]), (prec, K, k)


def test_even_odd_halves_of_other_blocks_than_their_lattice():
    """32768 sites are cut into blocks of 256 and their even-odd halves into blocks of 64: the
    preconditioned solve meets the whole lattice's residual, and the timing entry point holds the
    halves' larger number of partials."""
    dims = (16, 16, 8, 16)
    U, g = _gauge(dims, eo=1)
    chi = synth.z2_source(dims, synth.WILSON, 3)
    for prec in (lq.F64, lq.Q16):
        x, info = lq.cg_solve_batch(g, synth.WILSON, [0.2], chi[None], [1e-9],
                                    opts=lq.solve_opts(precision=prec, evenodd=1))
        x = x[0].cpu().numpy()
        r = wilson.apply(U, chi - wilson.apply(U, x, 0.2), 0.2, dagger=True)
        b = wilson.apply(U, chi, 0.2, dagger=True)
        assert np.linalg.norm(r) <= 1.01e-9 * np.linalg.norm(b)
        for kernel in (3, 4):
            assert lq.time_dslash(g, synth.WILSON, 0.2, precision=prec, kernel=kernel, reps=2) > 0
