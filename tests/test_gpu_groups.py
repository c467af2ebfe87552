"""Batches whose groups of systems per thread are full, partial or have one active system, and
staggered batches on either side of the line between the stencil's two forms (needs an MI355X).

Above 16384 sites the stencils run in blocks of 256 sites with the systems-per-thread count and the
block order that LQ_LAUNCH asks for.  16 x 16 x 8 x 16 has whole x-y planes of site blocks, so the
tiled orders -3 and -4 apply as well.  Whatever the group, a system's solution has the bits it has
alone, with one system per thread in the plain order.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

lq = pytest.importorskip("paper_1312_3265_amd")
torch = pytest.importorskip("torch")

W, SW = synth.WILSON, synth.STAGGERED_WILSON
DIMS = (16, 16, 8, 16)
FEATURES = lq.FEAT_CORNERS | lq.FEAT_F32 | lq.FEAT_Q16 | lq.FEAT_EO
_GAUGE = {}
_ALONE = {}


def _gauge(dims):
    if dims not in _GAUGE:
        _GAUGE[dims] = lq.Gauge(lq.Lattice(dims, (1, 1, 1, -1)),
                                synth.gauge_field(dims, "near_identity", 41, 0.436), FEATURES)
    return _GAUGE[dims]


def _system(dims, formulation, k):
    return synth.z2_source(dims, formulation, 90 + k), 0.2 + 0.05 * k


def _opts(precision, eo):
    return lq.solve_opts(precision=precision, evenodd=eo, poll_interval=8)


def _alone(dims, formulation, precision, eo, k, monkeypatch):
    key = (dims, formulation, precision, eo, k)
    if key not in _ALONE:
        monkeypatch.setenv("LQ_LAUNCH", "1,0")
        chi, m = _system(dims, formulation, k)
        x, infos = lq.cg_solve_batch(_gauge(dims), formulation, [m], chi[None], [1e-8],
                                     opts=_opts(precision, eo))
        assert infos[0]["status"] == lq.OK and infos[0]["true_residual"] <= 1e-8
        _ALONE[key] = x[0]
    return _ALONE[key]


@pytest.mark.parametrize("precision", [lq.F32, lq.Q16])
@pytest.mark.parametrize("formulation", [W, SW])
@pytest.mark.parametrize("K", [2, 4])
def test_pool_slots_are_bitwise_single_systems(K, formulation, precision, monkeypatch):
    """A resident pool of four slots with one loaded (an inner one of its group), with one in each
    group of two, and with three: the empty slots' systems are not computed, or not used."""
    refs = [_alone(DIMS, formulation, precision, 0, k, monkeypatch) for k in range(4)]
    monkeypatch.setenv("LQ_LAUNCH", f"{K},2")
    pool = lq.Batch(_gauge(DIMS), formulation, 4, opts=_opts(precision, 0))
    for slots in ((1,), (2,), (0, 3), (1, 2, 3)):
        for k in slots:
            chi, m = _system(DIMS, formulation, k)
            pool.load(k, chi, m, 1e-8)
        done = set()
        while len(done) < len(slots):
            for k, st in enumerate(pool.step(8)):
                assert st != lq.SLOT_FAILED
                if st == lq.SLOT_DONE and k not in done:
                    x, info = pool.fetch(k)
                    assert torch.equal(x, refs[k]), (slots, k)
                    done.add(k)


def _schedules(dims, formulation, precision, eo, n, launches, monkeypatch):
    refs = [_alone(dims, formulation, precision, eo, k, monkeypatch) for k in range(n)]
    chis, ms = zip(*(_system(dims, formulation, k) for k in range(n)))
    for K, w in launches:
        monkeypatch.setenv("LQ_LAUNCH", f"{K},{w}")
        x, infos = lq.cg_solve_batch(_gauge(dims), formulation, list(ms), np.stack(chis), [1e-8] * n,
                                     opts=_opts(precision, eo))
        assert all(i["status"] == lq.OK for i in infos), (K, w)
        for k in range(n):
            assert torch.equal(x[k], refs[k]), (K, w, k)


@pytest.mark.parametrize("precision", [lq.F32, lq.Q16])
@pytest.mark.parametrize("formulation,n", [(W, 5), (SW, 5), (SW, 9)])
def test_every_group_and_order_is_bitwise_single_systems(formulation, n, precision, monkeypatch):
    """Five systems leave a partial last group for two and four per thread; staggered Wilson takes
    groups of three (3 + 2, and 3 + 3 + 3 of nine) where four per thread are asked for."""
    _schedules(DIMS, formulation, precision, 0, n,
               [(K, w) for K in (1, 2, 4) for w in (0, 2, -1, -3, -4)], monkeypatch)


@pytest.mark.parametrize("precision", [lq.F32, lq.Q16])
@pytest.mark.parametrize("dims", [DIMS, (16, 16, 8, 32)])
def test_every_even_odd_group_and_order_is_bitwise_single_systems(dims, precision, monkeypatch):
    """The halves of the first lattice are cut into blocks of 64 sites, those of the second into
    blocks of 256."""
    _schedules(dims, W, precision, 1, 5, [(K, w) for K in (1, 2, 4) for w in (0, 1, 4, -1)],
               monkeypatch)


@pytest.mark.parametrize("precision,n", [(lq.F64, 2), (lq.F64, 3), (lq.F32, 2), (lq.F32, 3),
                                         (lq.Q16, 4), (lq.Q16, 5)])
def test_split_and_one_thread_staggered_stencils_are_bitwise_equal(precision, n, monkeypatch):
    """Up to 16384 sites the staggered stencil splits a site's terms over wavefronts while the
    launch has at most 512 blocks of 64 sites (16-bit 1024), and keeps one thread per site beyond:
    the systems of a batch on either side of that line have the bits of one system, which is
    always split."""
    dims = (16, 16, 8, 8)
    launches = [(1, 0), (1, 2)] + ([] if precision == lq.F64 else [(2, 0), (4, 2)])
    _schedules(dims, SW, precision, 0, n, launches, monkeypatch)
