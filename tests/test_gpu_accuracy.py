"""Rounding errors of the FP64 and mixed results: each at most what plain
evaluation in the same precision leaves, where the reference has a smaller
one."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2206_00708_amd")


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _mesh(seed, level=2):
    xyz, tri = synth.icosphere(level)
    rng = np.random.default_rng(seed)
    return synth.jitter_on_sphere(xyz @ synth.random_rotation(rng).T, tri, 0.02, rng), tri


@pytest.mark.parametrize("seed", [1, 2])
def test_singular_double_layer(orc, seed):
    """K and T of the pairs that share vertices.  Their (x - y).n is mostly
    cancellation, exact for coincident pairs.  The Gauss-Legendre weights of
    the library are within 1.2e-15 (four points: 1.1e-15, over four coordinates
    of which one or two dominate: 1.9e-15), the oracle, which subtracts rounded
    points, within 1.3e-15 of extended precision: 3.2e-15 together."""
    xyz, tri = _mesh(seed)
    cx = B.Context(0)
    m = B.Mesh(cx, xyz, tri)
    p = B.Problem(cx, m, m, 2.0, 3.0)
    p.assemble_operators(2)
    ref = orc.assemble(xyz, tri, 2.0, which=2, ops="KT")
    for op in "KT":
        assert _rel(p.operator(0, op).cpu().numpy(), ref[op]) < 3.5e-15, op
    for h in (p, m, cx):
        h.close()
