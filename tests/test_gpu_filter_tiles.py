"""The filter's passes over all elements at the edges of their tiles (64 tetrahedra; 64, 32,
16 or 8 hexahedra): element counts of less than one tile, whole tiles and a remainder, in the
plain call (dyadic index of every element against the oracle, untouched elements bit for bit)
and with the stage update fused in (one filtered RK4 step against the oracle, FP64)."""
import numpy as np
import pytest

from oracle import entropy_filter as ef
from oracle import fr as ofr
from oracle import rk as ork
from paper_2408_16509_amd import inputs

from helpers import oracle_blocks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
FP = ef.FilterParams()


@pytest.mark.parametrize("kind,n,order", [("tet", (1, 1, 1), 4), ("tet", (2, 4, 4), 4), ("tet", (3, 3, 4), 4),
                                          ("hex", (3, 3, 3), 1), ("hex", (4, 4, 4), 2), ("hex", (4, 4, 5), 3),
                                          ("hex", (3, 3, 3), 4)])
def test_filter_at_tile_edges(kind, n, order):
    from paper_2408_16509_amd import frmi
    mesh = inputs.hex_box(n) if kind == "hex" else inputs.kuhn_split(inputs.hex_box(n), permute_seed=5)
    b, = bl = oracle_blocks(mesh, order)
    x = b.xsol
    ic = np.moveaxis(inputs.shock(x[..., 0], x[..., 1], x[..., 2]), 0, 1).copy()
    smin = ef.smin_neighbourhood(bl, [ic], FP)[0]
    uo, ko, _ = ef.filter_block(b, ic, smin, FP)
    ctx = frmi.Context(mesh, system=0, order=order, riemann=1)
    u = ctx.pack64(ic.ravel())
    k = torch.zeros(len(ko), dtype=torch.int32, device="cuda")
    ctx.filter(u, u.clone(), mode=0, k=k)
    got = ctx.unpack64(u).cpu().numpy().reshape(ic.shape)
    assert np.array_equal(k.cpu().numpy(), ko)
    assert np.array_equal(got[ko == 0], ic[ko == 0])
    assert np.linalg.norm(got - uo) <= 1e-12 * np.linalg.norm(uo)
    # one RK4 step from the oracle's filtered state, the filter on every stage and the result
    dt = 1e-3
    sm = ef.smin_neighbourhood(bl, [uo], FP)[0]
    flt = lambda s: ef.filter_block(b, s, sm, FP)[0]
    prm = ofr.Params(riemann=1)
    want = flt(ork.rk4_step(lambda s: ofr.rhs(bl, [flt(s[0]) if s[0] is not uo else s[0]], prm), [uo], dt)[0])
    u = ctx.pack64(uo.ravel())
    ctx.rk_step(u, dt, 1, filter_mode=0)
    got = ctx.unpack64(u).cpu().numpy().reshape(ic.shape)
    assert np.linalg.norm(got - want) <= 1e-10 * np.linalg.norm(want - uo)
    ctx.close()
