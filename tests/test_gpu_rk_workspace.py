"""The integrators' shared workspace: the FP32 form's kept increments double as the filtered
hexahedra's FP64 accumulator and the embedded pair's first FP64 increment as RK4's accumulator, so a
context that alternates between them gives the bits of fresh contexts (padding lanes included), holds
no more than these need, and allocates nothing for RK4 once the embedded pair has run (so that an RK4
call can then be captured)."""
import numpy as np
import pytest

from paper_2408_16509_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

UREF = (1.0, 0.0, 0.0, 0.0, 2.5)


def _context(kind, fp32, n=(3, 5, 3)):
    from paper_2408_16509_amd import frmi
    mesh = inputs.hex_box(n)
    if kind == "mixed":
        mesh = inputs.concat([mesh, inputs.kuhn_split(inputs.hex_box((2, 2, 3), lo=(3.0, -3.1, -3.2), hi=(
            3.0 + 2 * np.pi, -3.1 + 2 * np.pi, -3.2 + 2 * np.pi)))], permute_seed=2)
    kw = dict(precision=frmi.FR_FP32, u_ref=UREF) if fp32 else {}
    return frmi.Context(mesh, order=4 if kind == "mixed" else 3, riemann=1, **kw)


def _shock(ctx):
    lay, x, out, off = ctx.layout, ctx.sol_points(), [], 0
    for i in range(lay.n_types):
        n, s = lay.n_elem[i], lay.n_sp[i]
        p = x[off:off + n * s].reshape(n, s, 3)
        out.append(np.moveaxis(inputs.shock(p[..., 0], p[..., 1], p[..., 2]), 0, 1).ravel())
        off += n * s
    u = ctx.pack64(np.concatenate(out))
    ctx.filter(u, u.clone(), mode=0)
    return u


@pytest.mark.parametrize("kind", ["hex", "mixed"])
@pytest.mark.parametrize("fp32", [False, True])
def test_alternating_integrators_equal_fresh_contexts(kind, fp32):
    calls = [lambda c, u: c.rk_step(u, 1e-3, 2, filter_mode=0), lambda c, u: c.rk_step(u, 1e-5, 2),
             lambda c, u: c.rk_adaptive(u, 2e-5, 1e-5, atol=1e-2, rtol=1e-2, fac_max=1.0),
             lambda c, u: c.rk_step(u, 1e-3, 1, filter_mode=0),
             lambda c, u: c.rk_adaptive(u, 1e-5, 1e-5, atol=1e-2, rtol=1e-2), lambda c, u: c.rk_step(u, 1e-5, 1)]
    one = _context(kind, fp32)
    u = _shock(one)
    pads = [(one.layout.native_offset[i], one.layout.n_sp[i], one.layout.e_pad[i], one.layout.n_elem[i])
            for i in range(one.layout.n_types)]
    assert any(e > n for _, _, e, n in pads)
    for i, call in enumerate(calls):
        fresh = _context(kind, fp32)
        want = u.clone()
        call(fresh, want)
        call(one, u)
        assert torch.equal(u, want), i
        fresh.close()
        for o, s, e, n in pads:
            pad = u[o:o + s * 5 * e].view(s, 5, e)[:, :, n:]
            assert torch.equal(pad, torch.tensor([1.0, 0, 0, 0, 1], dtype=torch.float64, device="cuda")[None, :, None]
                               .expand_as(pad)), i
    one.close()


@pytest.mark.parametrize("fp32", [False, True])
def test_rk4_captured_after_the_embedded_pair(fp32):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx = _context("hex", fp32)
        u0 = _shock(ctx)
        ctx.rk_adaptive(u0, 1e-5, 1e-5, atol=1e-2, rtol=1e-2)
        u, want = u0.clone(), u0.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ctx.rk_step(u, 1e-5, 2)
    for _ in range(4):                   # replays with eager work and synchronizations between
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            ctx.rk_step(want, 1e-5, 2)
        torch.cuda.synchronize()
        assert torch.equal(u, want)
    ctx.close()


def test_workspace_per_value():
    """Device memory that the integrators take at their first call, per native value: FP32 filtered 28
    bytes (stage 4, increments 4 + 12, the filter's FP64 stage state 8), FP64 RK4 and embedded pair
    together 40 (stage 8, increments 8 + 8 + 16); 64 MB beside them for per-element arrays and the
    allocator's granularity."""
    for fp32, calls, per in ((True, [lambda c, u: c.rk_step(u, 1e-9, 1, filter_mode=0)], 28),
                             (False, [lambda c, u: c.rk_step(u, 1e-9, 1),
                                      lambda c, u: c.rk_adaptive(u, 1e-9, 1e-9, atol=1e-2, rtol=1e-2)], 40)):
        ctx = _context("hex", fp32, (40, 40, 40))
        x = ctx.sol_points()
        w = np.empty((len(x), 5))
        w[:] = (1.0, 0.1, 0.0, 0.0, 2.6)
        u = ctx.pack64(w.reshape(-1, 64, 5).transpose(0, 2, 1).ravel())
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        for f in calls:
            f(ctx, u)
        torch.cuda.synchronize()
        took = free0 - torch.cuda.mem_get_info()[0]
        assert took <= per * ctx.layout.native_len + (64 << 20), (fp32, took / ctx.layout.native_len)
        ctx.close()
