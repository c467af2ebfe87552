"""Lattices whose FP64 arrays pass 4 GiB (needs an MI355X with 100 GB free).

The links are diag(1, -1, -1) on every bond, so that a link entry stored over another one shows;
fields are constant per colour.  Then C_mu psi = +-psi, D_st psi = 0 and Gamma_55 psi = phi psi with
phi = (-1)^(x2 + x4) (the four signs of a colour multiply to 1), so M psi = (m + 1 - phi) psi.
"""
import pytest

import synth

pytestmark = pytest.mark.gpu

lq = pytest.importorskip("paper_1312_3265_amd")
torch = pytest.importorskip("torch")


def _gauge(dims):
    L1, L2, L3, L4 = dims
    U = torch.zeros((L4, L3, L2, L1, 4, 3, 3), dtype=torch.complex128, device="cuda")
    for a, s in enumerate((1.0, -1.0, -1.0)):
        U[..., a, a] = s
    return lq.Gauge(lq.Lattice(dims), U, features=0)


def _free():
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.skipif(not torch.cuda.is_available() or _free() < 100 << 30, reason="needs 100 GB")
def test_plaquette_and_on_the_fly_apply_at_33_million_sites():
    """Nine slabs of links pass 4 GiB, the six that 12-real links read do not."""
    dims = (64, 64, 64, 128)
    g = _gauge(dims)
    assert abs(g.plaquette() - 1.0) <= 1e-13 and g.su3_deviation() == 0.0
    m = 0.25
    c = torch.tensor([1.0, 2.0 + 1.0j, -3.0], dtype=torch.complex128, device="cuda")
    psi = c.expand(dims[3], dims[2], dims[1], dims[0], 3).contiguous()
    out = lq.apply(g, synth.STAGGERED_WILSON, m, psi, g55=lq.G55_ONTHEFLY)
    x2 = torch.arange(dims[1], device="cuda")
    for t in range(dims[3]):
        phi = 1.0 - 2.0 * ((x2 + t) % 2)
        ref = (m + 1.0 - phi)[None, :, None, None] * psi[t]
        assert float((out[t] - ref).abs().max()) <= 1e-12
    del out, psi, g
    _free()


@pytest.mark.skipif(not torch.cuda.is_available() or _free() < 100 << 30, reason="needs 100 GB")
def test_an_operator_past_4_gib_is_refused():
    """An FP64 Wilson field of 23 million sites takes 4.4 GB: its last components were dropped or
    went over others."""
    dims = (64, 64, 64, 88)
    g = _gauge(dims)
    assert abs(g.plaquette() - 1.0) <= 1e-13
    psi = torch.ones((dims[3], dims[2], dims[1], dims[0], 4, 3), dtype=torch.complex128, device="cuda")
    with pytest.raises(lq.LQError) as e:
        lq.apply(g, synth.WILSON, 0.25, psi)
    assert e.value.code == lq.ERR_ARG
    del psi, g
    _free()
