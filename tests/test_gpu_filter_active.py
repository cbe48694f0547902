"""The filter's passes over all elements with elements to treat in every one of them: a filtered
shock whose energy is disturbed in part of the elements, the last one (in the last, partial tile)
among them.  The plain call against the oracle (dyadic index of every element, fallbacks among
them, untouched elements bit for bit, states to 1e-12), then one RK4 step from the filtered state
with the stage updates fused in, candidates in each of its four passes, FP64 within 1e-10 and the
FP32 form within 1e-4 of the oracle's increment, the bounds of the other filter tests.  (The
oracle's own response to disturbing its right-hand sides by 1e-14 is below 1e-13 of the increment, and
to 1e-6 below 1e-5 where the FP32 form is compared: no decision sits on an edge.)"""
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

# kind, cells, order, every how many elements disturbed, by how much, seed, step, FP32 form as well
CASES = [("tet", (1, 1, 1), 4, 3, 0.4, 1, 5e-3, True), ("tet", (2, 4, 4), 4, 3, 0.4, 1, 5e-3, True),
         ("tet", (3, 3, 4), 4, 3, 0.4, 2, 5e-3, True), ("hex", (5, 13, 1), 1, 1, 0.5, 6, 0.1, True),
         ("hex", (4, 4, 5), 2, 3, 0.4, 7, 4e-2, True), ("hex", (3, 17, 1), 3, 3, 0.4, 3, 2e-2, True),
         ("hex", (3, 3, 3), 4, 3, 0.4, 1, 2e-2, True), ("hex", (5, 13, 1), 4, 3, 0.4, 1, 2e-2, False)]


@pytest.mark.parametrize("kind,n,order,every,amp,seed,dt,reduced", CASES)
def test_filter_at_work(kind, n, order, every, amp, seed, dt, reduced):
    from paper_2408_16509_amd import frmi
    mesh = inputs.hex_box(n) if kind == "hex" else inputs.kuhn_split(inputs.hex_box(n), permute_seed=5)
    b, = bl = oracle_blocks(mesh, order)
    x = b.xsol
    base = np.moveaxis(inputs.shock(x[..., 0], x[..., 1], x[..., 2]), 0, 1).copy()
    base = ef.filter_block(b, base, ef.smin_neighbourhood(bl, [base], FP)[0], FP)[0]
    disturbed = np.arange(len(base)) % every == (len(base) - 1) % every
    st = base.copy()
    st[disturbed, 4] *= 1 + amp * np.random.default_rng(seed).uniform(-1, 1, size=(disturbed.sum(), st.shape[2]))
    smin = ef.smin_neighbourhood(bl, [base], FP)[0]
    uo, ko, _ = ef.filter_block(b, st, smin, FP)
    assert (ko != 0).any() and ko[-1] != 0
    # the step of the oracle, and how many elements each of its filter passes treats
    sm, prm, treated = ef.smin_neighbourhood(bl, [uo], FP)[0], ofr.Params(riemann=1), []

    def flt(s):
        out, k, _ = ef.filter_block(b, s[0], sm, FP)
        treated.append(((k != 0).sum(), k[-1] != 0))
        return [out]
    want, = ork.rk4_step(lambda s: ofr.rhs(bl, s, prm), [uo], dt, stage_post=flt)
    assert len(treated) == 4 and all(c > 0 for c, _ in treated) and any(last for _, last in treated)

    forms = [({}, 1e-10)]
    if reduced:
        forms.append((dict(precision=frmi.FR_FP32, u_ref=(1.0, 0.0, 0.0, 0.0, 2.5)), 1e-4))
    for kw, tol in forms:
        ctx = frmi.Context(mesh, system=0, order=order, riemann=1, elem_order=1, **kw)
        u = ctx.pack64(st.ravel())
        k = torch.full((len(ko),), 7, dtype=torch.int32, device="cuda")
        stats = ctx.filter(u, ctx.pack64(base.ravel()), mode=0, k=k, stats=True)
        got = ctx.unpack64(u).cpu().numpy().reshape(st.shape)
        assert np.array_equal(k.cpu().numpy(), ko)
        assert stats.n_troubled == (ko != 0).sum() and stats.n_fallback == (ko < 0).sum()
        assert np.array_equal(got[ko == 0], st[ko == 0])
        assert np.linalg.norm(got - uo) <= 1e-12 * np.linalg.norm(uo)
        u = ctx.pack64(uo.ravel())
        ctx.rk_step(u, dt, 1, filter_mode=0)
        got = ctx.unpack64(u).cpu().numpy().reshape(st.shape)
        ctx.close()
        err = np.linalg.norm(got - want) / np.linalg.norm(want - uo)
        print(kind, n, order, "fp32" if kw else "fp64", "treated", [int(c) for c, _ in treated], f"error {err:.1e}", flush=True)
        assert err <= tol
