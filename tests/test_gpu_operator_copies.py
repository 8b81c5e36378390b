"""Copies of complex64 operators in caller numbering on both sides of the row
length up to which they are read in place (3,200 vertices): a mesh in another
numbering gives the same entries but for the rounding of other blocks' orders
of summation (complex64: 2e-5 of the largest entry)."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2206_00708_amd")


@pytest.mark.parametrize("n", [3199, 3200, 3201])
def test_copies_around_the_line(n):
    cx = B.Context(0)
    xyz, tri = synth.fibonacci_sphere(n)
    perm = np.random.default_rng(n).permutation(n)
    small = B.Mesh(cx, *synth.icosphere(0))
    got = []
    for x, t in ((xyz, tri), (xyz[perm], np.argsort(perm)[tri].astype(np.int32))):
        m = B.Mesh(cx, x, t)
        p = B.Problem(cx, m, small, 1.0, 1.5, precision=B.C64_MIXED)
        p.assemble_operators()
        got.append(p.operator(0, "K"))
        p.close()
        m.close()
    i = torch.from_numpy(perm).cuda()
    want = got[0][i[:, None], i[None, :]]
    assert (got[1] - want).abs().max() < 2e-5 * want.abs().max()
