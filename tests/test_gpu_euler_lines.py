"""The Euler divergence with its directions side by side, the forms whose partners' traces come
from hex_trace on curved p = 4 elements: below and past the mesh size at which the other form
takes over.  Copies of a small curved box; every copy has to give the oracle's residual, FP64
1e-12 and FP32 1e-5 of well-conditioned states as in the other element tests."""
import numpy as np
import pytest

from oracle import fr as ofr
from paper_2408_16509_amd import inputs

from helpers import oracle_blocks, rel_err
from test_gpu_euler_rk32 import UREF, _copies

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _check(mesh, order, riemann, prec, tol, counts):
    from paper_2408_16509_amd import frmi
    b, = bl = oracle_blocks(mesh, order)
    u = np.moveaxis(inputs.random_state(b.xsol.shape[:2], 11, vel=0.1, amp=0.02), 0, 1).copy()
    want = ofr.rhs(bl, [u], ofr.Params(system=0, riemann=riemann))[0]
    for k in counts:
        ctx = frmi.Context(_copies(mesh, k), system=0, order=order, riemann=riemann, precision=prec, u_ref=UREF)
        r = ctx.new_native()
        ctx.rhs(ctx.pack(np.tile(u, (k, 1, 1)).ravel()), r)
        got = ctx.unpack_rhs(r).cpu().numpy().reshape((k,) + u.shape)
        ctx.close()
        worst = max(rel_err([got[i]], [want])[0] for i in range(k))
        assert worst <= tol, (k, worst)


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("riemann", [0, 1])
def test_curved_p4_either_side_of_the_line(fp32, riemann):
    from paper_2408_16509_amd import frmi
    mesh = inputs.curved_hex_box((5, 3, 1), q=2, amp=0.1)
    below = 256 * (8 if fp32 else 4) // 15
    _check(mesh, 4, riemann, frmi.FR_FP32 if fp32 else frmi.FR_FP64, 1e-5 if fp32 else 1e-12, (1, below, below + 5))
