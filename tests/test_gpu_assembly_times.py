"""Times of the assembly of two small meshes side by side."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2206_00708_amd")


def test_parts_hold_no_wait_for_the_other_mesh():
    """1,856 triangles outside, 80 inside, one singular Gauss point: nearly all
    of the time is the exterior's regular pairs, and the singular part of the
    interior mesh, which ends long before, is not the wait for them."""
    cx = B.Context(0)
    me, mi = B.Mesh(cx, *synth.fibonacci_sphere(930)), B.Mesh(cx, *synth.icosphere(1))
    p = B.Problem(cx, me, mi, 300.0, 3.0, singular_gauss=1)
    part = []
    for _ in range(8):
        p.assemble_operators()
        p.assemble_projection()
        _, st, _ = p.solve(np.array([[0.0, 0.0, 1.0]]), tol=1e-2, maxit=5)
        assert st["t_assembly_ms"] >= 0.9 * st["t_regular_ms"] / 2
        part.append(st["t_singular_ms"] / st["t_regular_ms"])
    assert np.median(part) < 0.5, part
    for h in (p, me, mi, cx):
        h.close()
