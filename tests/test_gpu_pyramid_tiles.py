"""Pyramids at the edges of the 16-element blocks of the matrix-core kernels (6, 48, 54 and 192
elements) and in both one-sided LDG directions, against the oracle; the two-sided switch (the
general kernels) at the same sizes.  FP64 at 1e-12 of well-conditioned states, the FP32
deviation form within its stated 1e-5."""
import numpy as np
import pytest

from oracle import fr as ofr
from paper_2408_16509_amd import inputs

from helpers import oracle_blocks, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [(1, 1, 1), (2, 2, 2), (3, 3, 1), (4, 4, 2)])
@pytest.mark.parametrize("system,riemann,beta", [(0, 1, 0.5), (1, 0, 0.5), (1, 1, -0.5), (1, 0, 0.0)])
def test_pyramids_at_block_edges(n, system, riemann, beta):
    from paper_2408_16509_amd import frmi
    mesh = inputs.pyramid_box(n, apex_perturb=0.1, perturb_seed=3, permute_seed=4, rotate_seed=5)
    b, = bl = oracle_blocks(mesh, 4)
    s = inputs.random_state(b.xsol.shape[:2], 11, vel=0.1, amp=0.02)
    u = np.moveaxis(s, 0, 1).copy()
    want = ofr.rhs(bl, [u], ofr.Params(system=system, riemann=riemann, ldg_beta=beta))
    for prec, tol in ((frmi.FR_FP64, 1e-12), (frmi.FR_FP32, 1e-5)):
        ctx = frmi.Context(mesh, system=system, order=4, riemann=riemann, ldg_beta=beta, precision=prec,
                           u_ref=(1.0, 0.0, 0.0, 0.0, 2.5))
        r = ctx.new_native()
        ctx.rhs(ctx.pack(u.ravel()), r)
        got = ctx.unpack_rhs(r).cpu().numpy().reshape(u.shape)
        ctx.close()
        err, per_var = rel_err([got], want)
        assert err <= tol and np.all(per_var <= tol), (err, per_var)
