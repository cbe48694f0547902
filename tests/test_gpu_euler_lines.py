"""The Euler divergence with its directions side by side: the forms whose partners' traces come
from hex_trace on curved p = 4 elements, below and past the mesh size at which the other form
takes over, and the forms whose line lies elsewhere.  Copies of a small box; every copy has to
give the oracle's residual, FP64 1e-12 and FP32 1e-5 of well-conditioned states as in the other
element tests."""
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


@pytest.mark.parametrize("order,curved,fp32,blocks", [(1, False, True, 768), (2, False, False, 768), (2, True, True, 768),
                                                      (1, True, False, 300), (1, True, True, 300), (2, True, False, 800)])
def test_lines_past_one_block_per_cu(order, curved, fp32, blocks):
    """The forms that run side by side on larger meshes: at their line, just past it (or past
    256 blocks, where there is no line)."""
    from paper_2408_16509_amd import frmi
    n = (5, 13, 1)
    mesh = inputs.curved_hex_box(n, q=order, amp=0.1) if curved else inputs.hex_box(n, perturb=0.1, perturb_seed=3,
                                                                                    permute_seed=4)
    at = blocks * (32 if order == 1 else 16) // 65
    _check(mesh, order, 1, frmi.FR_FP32 if fp32 else frmi.FR_FP64, 1e-5 if fp32 else 1e-12, (at, at + 1))
