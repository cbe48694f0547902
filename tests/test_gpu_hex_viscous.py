"""Navier--Stokes on hexahedra: the gradient kernel's point and end tables at every order (columns
split over threads that do not divide the points, ends that do not fill the threads), the three
LDG switches and both geometries, on element counts below, at and above one 64-element block,
against the oracle.  FP64 at 1e-12 of well-conditioned states, the FP32 deviation form within its
stated 1e-5."""
import numpy as np
import pytest

from oracle import fr as ofr
from paper_2408_16509_amd import inputs

from helpers import oracle_blocks, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [(1, 1, 1), (4, 4, 4), (5, 13, 1)])
@pytest.mark.parametrize("order,curved", [(1, False), (2, False), (3, False), (4, False), (2, True), (4, True)])
@pytest.mark.parametrize("riemann,beta", [(1, 0.5), (0, -0.5), (1, 0.0), (0, 0.3)])
def test_hex_navier_stokes(n, order, curved, riemann, beta):
    from paper_2408_16509_amd import frmi
    kw = dict(perturb=0.1, perturb_seed=3, permute_seed=4)
    mesh = inputs.curved_hex_box(n, q=2, amp=0.1, permute_seed=4) if curved else inputs.hex_box(n, **kw)
    b, = bl = oracle_blocks(mesh, order)
    u = np.moveaxis(inputs.random_state(b.xsol.shape[:2], 11, vel=0.1, amp=0.02), 0, 1).copy()
    want = ofr.rhs(bl, [u], ofr.Params(system=1, riemann=riemann, ldg_beta=beta))
    for prec, tol in ((frmi.FR_FP64, 1e-12), (frmi.FR_FP32, 1e-5)):
        ctx = frmi.Context(mesh, system=1, order=order, riemann=riemann, ldg_beta=beta, precision=prec,
                           u_ref=(1.0, 0.0, 0.0, 0.0, 2.5))
        r = ctx.new_native()
        ctx.rhs(ctx.pack(u.ravel()), r)
        got = ctx.unpack_rhs(r).cpu().numpy().reshape(u.shape)
        ctx.close()
        err, per_var = rel_err([got], want)
        assert err <= tol and np.all(per_var <= tol), (err, per_var)
