"""The byte model of the kernels that run (no GPU): each array of a form counted once, written out
here from the kernels' arguments."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("sfx,d", [("", 8), ("_f32", 4)])
def test_straight_tetrahedra_both_precisions(sfx, d):
    nsp, nfp, geo = 35, 60, 10 * d + 4 * 2 * 4
    # state in; S_i.f_v (4 values x 3 directions) and the formed pairs' common fluxes out
    assert bench.kernel_bytes_per_elem("tet_grad" + sfx, nsp, nfp) == d * (5 * nsp + 12 * nsp + 5 * (nfp // 2)) + geo
    # state, S_i.f_v and every flux point's common flux in; R out
    assert bench.kernel_bytes_per_elem("tet_div_ns" + sfx, nsp, nfp) == d * (5 * nsp + 12 * nsp + 5 * nfp + 5 * nsp) + geo


@pytest.mark.parametrize("d,sfx", [(8, ""), (4, "_f32")])
@pytest.mark.parametrize("p", [1, 3, 4])
def test_hexahedra_with_stored_viscous_fluxes(d, sfx, p):
    nsp, nfp = (p + 1) ** 3, 6 * (p + 1) ** 2
    b = lambda name: bench.kernel_bytes_per_elem(f"{name}{sfx}_p{p}", nsp, nfp)
    # state, partner traces on half of the faces; tau and energy flux (9), f_v.n (4) on half of the faces
    assert b("hex_grad_vf") == d * (5 * nsp + 5 * nfp // 2 + 9 * nsp + 4 * nfp // 2 + 24) + 48
    # both traces of every pair, one f_v.n, both slots of the common flux
    assert b("hex_face_vf") == d * (5 * nfp + 4 * nfp // 2 + 5 * nfp + 24) + 48
    assert b("hex_div_vf") == d * (5 * nsp + 9 * nsp + 5 * nfp + 5 * nsp + 24)
    # curved: stored metric for the 24 corner words
    for fam, metric in (("hex_grad_vf", 10 * nsp + 3 * nfp // 2), ("hex_face_vf", 3 * nfp // 2), ("hex_div_vf", 10 * nsp)):
        assert bench.kernel_bytes_per_elem(f"{fam}_cur{sfx}_p{p}", nsp, nfp) == b(fam) - 24 * d + d * metric
