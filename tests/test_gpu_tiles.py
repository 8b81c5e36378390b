"""Regular-pair tiles at the edges of their block tables, against the oracle:
runs of corners up to the longest a block holds (a pole shared by `n`
triangles of one block), blocks in Morton order (a valence above 12), a last
block of a few triangles, and the three phase forms of the quadrature."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2206_00708_amd")


def _globe(n, rings, rng):
    """A sphere of n meridians and `rings` parallels between two poles of valence n."""
    th = np.pi * np.arange(1, rings + 1) / (rings + 1)
    ph = 2 * np.pi * np.arange(n) / n
    ring = np.stack([np.sin(th)[:, None] * np.cos(ph), np.sin(th)[:, None] * np.sin(ph),
                     np.repeat(np.cos(th)[:, None], n, axis=1)], axis=2).reshape(-1, 3)
    x = np.concatenate([[[0, 0, 1.0]], ring, [[0, 0, -1.0]]])
    x = x * (1.0 + 0.02 * rng.standard_normal((len(x), 1)))
    at = lambda r, j: 1 + r * n + j % n   # noqa: E731
    tri = [(0, at(0, j), at(0, j + 1)) for j in range(n)]
    for r in range(rings - 1):
        for j in range(n):
            tri += [(at(r, j), at(r + 1, j), at(r + 1, j + 1)), (at(r, j), at(r + 1, j + 1), at(r, j + 1))]
    tri += [(len(x) - 1, at(rings - 1, j + 1), at(rings - 1, j)) for j in range(n)]
    return x, np.array(tri, dtype=np.int32)


# FP64 at the operator tolerance of the parity tests; the mixed form at its first-order
# bound n u with n = 324 terms and u = 2^-24
@pytest.mark.parametrize("n,rings,k,prec,tol", [(5, 3, 0.4, "C128", 1e-12), (7, 4, 2.0, "C128", 1e-12),
                                                (8, 5, 1.0, "C128", 1e-12), (12, 4, 1.5, "C128", 1e-12),
                                                (12, 1, 6.0, "C128", 1e-12), (13, 4, 1.5, "C128", 1e-12),
                                                (12, 4, 1.5, "C64_MIXED", 2e-5), (7, 4, 9.0, "C64_MIXED", 2e-5)])
def test_operators_globe(orc, n, rings, k, prec, tol):
    x, tri = _globe(n, rings, np.random.default_rng(n))
    ctx = B.Context(0)
    m = B.Mesh(ctx, x, tri)
    p = B.Problem(ctx, m, m, k, 1.3 * k, 1.0, 1.0, getattr(B, prec))
    p.assemble_operators()
    for mesh, kk in ((0, k), (1, 1.3 * k)):
        ref = orc.assemble(x, tri, kk)
        for op in "VKTD":
            got = p.operator(mesh, op).cpu().numpy()
            err = np.abs(got - ref[op]).max() / np.abs(ref[op]).max()
            assert err < tol, (mesh, op, err)


# the three phase forms of a complex wavenumber, set by k and by the damping; the mixed form beside them
@pytest.mark.parametrize("k,kim,prec,tol", [(0.5, 0.2, "C128", 1e-12), (0.2, 0.5, "C128", 1e-12),
                                            (1.3, 0.4, "C128", 1e-12), (0.3, 1.3, "C128", 1e-12),
                                            (0.3, 4.0, "C128", 1e-12), (6.0, 0.1, "C128", 1e-12),
                                            (0.3, 1.3, "C64_MIXED", 2e-5)])
def test_absorbing_operators_globe(orc, k, kim, prec, tol):
    x, tri = _globe(10, 6, np.random.default_rng(3))
    ctx = B.Context(0)
    m = B.Mesh(ctx, x, tri)
    p = B.Problem(ctx, m, m, k, k, 1.0, 1.0, getattr(B, prec))
    p.set_k_int_imag(kim)
    p.assemble_operators()
    ref = orc.assemble(x, tri, k + 1j * kim)
    for op in "VKTD":
        got = p.operator(1, op).cpu().numpy()
        err = np.abs(got - ref[op]).max() / np.abs(ref[op]).max()
        assert err < tol, (op, err)
