"""The embedded pair's stage and norm kernels at the edges of their launches: padded blocks
(65 and 513 elements), the element count at which the block size changes (512), both state types,
against the oracle integrating the same problem.  Bounds of the other adaptive tests: FP64 norm
and step to 1e-9 and the state's change to 1e-10, FP32 form 1e-4."""
import numpy as np
import pytest

from oracle import fr as ofr
from oracle import rk_adaptive as ra
from paper_2408_16509_amd import inputs

from helpers import oracle_blocks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MACH = 0.3


@pytest.mark.parametrize("n", [(5, 13, 1), (8, 8, 8), (9, 19, 3)])
@pytest.mark.parametrize("fp32", [False, True])
def test_adaptive_at_block_edges(n, fp32):
    from paper_2408_16509_amd import frmi
    mesh = inputs.hex_box(n)
    b, = bl = oracle_blocks(mesh, 2)
    u0 = np.moveaxis(inputs.tgv(b.xsol[..., 0], b.xsol[..., 1], b.xsol[..., 2], mach=MACH), 0, 1).copy()
    prm = ofr.Params(system=0, riemann=0)
    t_end, dt0, tol = 0.02, 0.01, 1e-6
    (uo,), so = ra.integrate(lambda s: ofr.rhs(bl, s, prm), [u0], t_end, dt0, ra.Controller(atol=tol, rtol=tol))
    kw = dict(precision=frmi.FR_FP32, u_ref=(1.0, 0.0, 0.0, 0.0, 1.0 / (1.4 * MACH ** 2) / 0.4)) if fp32 else {}
    ctx = frmi.Context(mesh, system=0, order=2, riemann=0, **kw)
    ug = ctx.pack64(u0.ravel())
    sg = ctx.rk_adaptive(ug, t_end, dt0, atol=tol, rtol=tol)
    got = ctx.unpack64(ug).cpu().numpy()
    ctx.close()
    err = np.linalg.norm(got - uo.ravel()) / np.linalg.norm(uo - u0)
    assert sg.t == t_end
    if fp32:
        assert abs(sg.accepted - so.accepted) <= 1 and err <= 1e-4, err
        return
    assert (sg.accepted, sg.rejected, sg.n_rhs) == (so.accepted, so.rejected, so.n_rhs)
    assert abs(sg.last_norm - so.steps[-1][1]) <= 1e-9 * so.steps[-1][1]
    assert err <= 1e-10, err
