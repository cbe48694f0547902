"""Device buffers of a Navier--Stokes context: what its kernels read, and no more.  Bytes taken at
setup against the arrays of each form (traces, viscous flux or gradient, gradient traces, common
fluxes; geometry and connectivity beside them), 48 MB allowed for the allocator's granularity;
the right-hand side on these contexts is covered by the parity tests of every form."""
import numpy as np
import pytest

from paper_2408_16509_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind,beta,fp32,words", [
    # pyramids, 55 points and 85 flux points: one-sided: traces, S_i.f_v, common fluxes
    ("pyr", 0.5, True, 5 * 85 + 12 * 55 + 5 * 85),
    # two-sided: traces, gradient, its traces
    ("pyr", 0.0, True, 5 * 85 + 15 * 55 + 15 * 85),
    # tetrahedra, 35 and 60: one-sided: S_i.f_v, common fluxes; two-sided: gradient
    ("tet", 0.5, False, 12 * 35 + 5 * 60), ("tet", 0.3, False, 15 * 35),
    # curved FP64 tetrahedra: the gradient whatever the switch; stored metric 10 x 35 + 3 x 60
    ("curved_tet", -0.5, False, 15 * 35 + 530)])
def test_buffers_of_each_form(kind, beta, fp32, words):
    from paper_2408_16509_amd import frmi
    n = (16, 16, 16) if kind == "curved_tet" else (20, 20, 20)
    mesh = {"pyr": lambda: inputs.pyramid_box(n), "tet": lambda: inputs.kuhn_split(inputs.hex_box(n)),
            "curved_tet": lambda: inputs.curved_tet_box(n, q=2, amp=0.1)}[kind]()
    kw = dict(precision=frmi.FR_FP32, u_ref=(1.0, 0, 0, 0, 2.5)) if fp32 else {}
    # what a process takes at its first context and launch (code, queues) is not the context's
    small = frmi.Context(inputs.hex_box((2, 2, 2)), order=1)
    small.rhs(small.pack(np.tile([1.0, 0, 0, 0, 2.5], (64, 1)).reshape(8, 8, 5).transpose(0, 2, 1).ravel()), small.new_native())
    small.close()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    ctx = frmi.Context(mesh, system=1, order=4, ldg_beta=beta, **kw)
    took = free0 - torch.cuda.mem_get_info()[0]
    E = ctx.layout.e_pad[0]
    ctx.close()
    most = E * (words * (4 if fp32 else 8) + 200) + (48 << 20)
    assert took <= most, (took, most)
