"""Canonical <-> native layout (fr_pack, fr_unpack, fr_pack64, fr_unpack64, fr_unpack_rhs):
data movement, so every comparison is bit for bit.  Element counts off the multiples of the
32-element tiles, every number of points per element (one or several chunks per tile), both
element orders and a context of two blocks."""
import numpy as np
import pytest

from paper_2408_16509_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MESHES = {
    "hex": lambda: inputs.hex_box((3, 5, 7), permute_seed=3),
    "one_hex": lambda: inputs.hex_box((1, 1, 1)),
    "tet": lambda: inputs.kuhn_split(inputs.hex_box((2, 3, 3)), permute_seed=3),
    "pyr": lambda: inputs.pyramid_box((2, 3, 2), permute_seed=3),
    "mixed": lambda: inputs.concat([inputs.hex_box((3, 3, 4)), inputs.kuhn_split(inputs.hex_box(
        (3, 3, 4), lo=(3.0, -np.pi, -np.pi), hi=(3.0 + 2 * np.pi, np.pi, np.pi)))], permute_seed=3),
}


@pytest.mark.parametrize("mname,order", [("hex", 1), ("hex", 2), ("hex", 3), ("hex", 4), ("one_hex", 4), ("tet", 4),
                                         ("pyr", 4), ("mixed", 4)])
@pytest.mark.parametrize("elem_order", [1, 2])
def test_layout_round_trip(mname, order, elem_order):
    from paper_2408_16509_amd import frmi
    mesh = MESHES[mname]()
    ref = (1.0, 0.0, 0.0, 0.0, 2.5)
    for prec in (frmi.FR_FP64, frmi.FR_FP32):
        ctx = frmi.Context(mesh, order=order, precision=prec, u_ref=ref, elem_order=elem_order)
        lay = ctx.layout
        c = np.random.default_rng(7).normal(size=lay.canon_len) + 3.0
        want = c.copy()                 # what the native form holds, canonical order, per block
        nat64, nat = ctx.pack64(c), ctx.pack(c)
        assert np.array_equal(ctx.unpack64(nat64).cpu().numpy(), c)
        got, rhs = ctx.unpack(nat).cpu().numpy(), ctx.unpack_rhs(nat).cpu().numpy()
        for i in range(lay.n_types):
            n, s, E = lay.n_elem[i], lay.n_sp[i], lay.e_pad[i]
            o, no = lay.canon_offset[i], lay.native_offset[i]
            b = slice(o, o + n * 5 * s)
            if prec == frmi.FR_FP32:
                r = np.array(ref)[None, :, None]
                dev = (c[b].reshape(n, 5, s) - r).astype(np.float32)
                want[b] = (dev.astype(np.float64) + r).ravel()
                assert np.array_equal(rhs[b], dev.astype(np.float64).ravel())
            else:
                assert np.array_equal(rhs[b], c[b])
            if elem_order == 1:         # the native rows [pt][var][E], element order as given
                rows = nat64[no:no + s * 5 * E].cpu().numpy().reshape(s, 5, E)
                assert np.array_equal(rows[:, :, :n], c[b].reshape(n, 5, s).transpose(2, 1, 0))
                assert np.array_equal(rows[:, :, n:], np.broadcast_to(
                    np.array([1.0, 0, 0, 0, 1])[None, :, None], (s, 5, E - n)))
        assert np.array_equal(got, want)
        ctx.close()
