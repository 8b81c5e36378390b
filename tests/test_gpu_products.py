"""Products at the edges of their launch shapes: the block GEMM with chunks of
one stage, an odd and an even number of stages at each tile width and stage
depth, vectors off 16-byte boundaries, and the dense inverse-mass apply for
vectors that do not fit a compute unit's LDS."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2206_00708_amd")
N = pytest.importorskip("paper_2206_00708_amd._native")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _problem(ctx, ne, ni, prec, mode=0):
    me, mi = B.Mesh(ctx, *synth.fibonacci_sphere(ne)), B.Mesh(ctx, *synth.fibonacci_sphere(ni))
    p = B.Problem(ctx, me, mi, 2.0, 3.0, 1.0, 1.5, precision=prec)
    p.set_mass_apply(mode)
    p.assemble_operators()
    p.assemble_projection()
    return p


_CHILD = """
import sys, numpy as np, torch
sys.path.insert(0, %r); sys.path.insert(0, %r)
import paper_2206_00708_amd as B
from test_gpu_products import _problem, _rel
ctx = B.Context(0)
rng = np.random.default_rng(5)
for ne, ni in %r:
    p = _problem(ctx, ne, ni, B.C64_MIXED)
    for R in (1, 5, 16, 17, 33, 64):
        X = rng.standard_normal((R, p.n)) + 1j * rng.standard_normal((R, p.n))
        Y = p.mtf_matvec_batch(torch.from_numpy(X), strong=False).cpu().numpy()
        err = max(_rel(Y[r], p.mtf_matvec(torch.from_numpy(X[r]), strong=False).cpu().numpy()) for r in range(R))
        print(ne, ni, R, err, flush=True)
t = B.tune_table()
print({k: t[k] for k in t if k.startswith("gemm-ops")})
"""


# rows of 2 x 32, 2 x 64, 2 x 96 and 2 x 192 floats: chunks of 1 to 12 stages
_SIZES = ((20, 42), (162, 92))


@pytest.mark.parametrize("nke,nki,kst", [(1, 1, 32), (8, 3, 32), (3, 5, 32), (1, 2, 64), (8, 3, 64)])
def test_gemm_shapes(tmp_path, nke, nki, kst):
    """Against the single-vector mixed product, at the bound of the batch test
    for two FP32 summation orders.  The shapes are set by a table file."""
    cls = lambda n: round(4 * np.log2(n))   # noqa: E731
    f = tmp_path / "tune.txt"
    f.write_text("".join(f"gemm-ops:c{c}:e{cls(ne)}:i{cls(ni)} {nke} {nki} {kst}\n"
                         for c in (32, 64, 128) for ne, ni in _SIZES))
    out = subprocess.run([sys.executable, "-c", _CHILD % (ROOT, os.path.join(ROOT, "tests"), _SIZES)],
                         capture_output=True, text=True, timeout=100, env=dict(os.environ, BEMTX_TUNE_FILE=str(f)))
    assert out.returncode == 0, out.stderr[-2000:]
    lines = out.stdout.strip().splitlines()
    used = eval(lines[-1])
    assert len(used) == 6 and all(v == [nke, nki, kst] for v in used.values()), used
    assert len(lines) == 13 and all(float(s.split()[3]) < 2e-6 for s in lines[:12]), lines


@pytest.mark.parametrize("prec,nrhs", [(B.C128, 0), (B.C64_MIXED, 0), (B.C64_MIXED, 3)])
def test_vectors_off_16_byte_boundaries(prec, nrhs):
    """Device vectors that begin 8 bytes into a 16-byte unit: the same bits."""
    p = _problem(B.Context(0), 92, 42, prec)
    n, R = p.n, max(nrhs, 1)
    x = torch.randn(2 * n * R, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    got = []
    for off in ((0, 0), (1, 0), (0, 1), (1, 1)):
        bx, by = (torch.zeros(2 * n * R + 2, dtype=torch.float64, device="cuda") for _ in range(2))
        vx, vy = bx[off[0]:off[0] + 2 * n * R], by[off[1]:off[1] + 2 * n * R]
        vx.copy_(x)
        torch.cuda.synchronize()
        a, b = ctypes.c_void_p(vx.data_ptr()), ctypes.c_void_p(vy.data_ptr())
        code = (N.load().bem_mtf_matvec_batch(p._h, a, b, nrhs, 1, 1) if nrhs
                else N.load().bem_mtf_matvec(p._h, a, b, 1, 1))
        assert code == B.OK
        got.append(vy.clone())
        assert by.count_nonzero() == vy.count_nonzero()   # nothing written beside the result
    assert got[0].abs().max() > 0 and all(torch.equal(got[0], g) for g in got[1:])


@pytest.mark.parametrize("ne,ni", [(4500, 92), (4700, 92)])   # the first fit LDS, the second do not
def test_dense_mass_apply_either_side_of_lds(ne, ni):
    """The dense inverse against the sparse apply, both FP64, at the bound of
    their comparison at 2,562 + 1,962 vertices."""
    ctx = B.Context(0)
    y = []
    for mode in (1, 2):
        p = _problem(ctx, ne, ni, B.C128, mode)
        assert p.mass_apply_sparse() == (mode == 2)
        x = np.random.default_rng(9).standard_normal((2, p.n))
        y.append(p.mtf_matvec(torch.from_numpy(x[0] + 1j * x[1]), strong=True).cpu().numpy())
        del p
    assert _rel(y[0], y[1]) < 1e-13


def _rosette(n, points):
    """A sphere of about `points` vertices of valence up to 7, one of valence n."""
    from scipy.spatial import ConvexHull
    x = synth.fibonacci_sphere(points)[0]
    h = np.sqrt(4 * np.pi / points)
    a = max(n / (2 * np.pi), 1.0) * h
    ph = 2 * np.pi * np.arange(n) / n + 0.01
    ring = np.stack([np.sin(a) * np.cos(ph), np.sin(a) * np.sin(ph), 0 * ph + np.cos(a)], axis=1)
    x = np.concatenate([x[np.arccos(np.clip(x[:, 2], -1, 1)) > a + 0.8 * h], [[0, 0, 1.0]], ring])
    return x, synth.orient_outward(x, ConvexHull(x).simplices.astype(np.int32))


# the widths of the sparse apply's rows (6, 8, 11 and 15 neighbours) at their ends, in patches of one vertex
# per thread and of two
@pytest.mark.parametrize("n", [6, 7, 8, 9, 11, 12, 15])
@pytest.mark.parametrize("points", [162, 2562])
def test_sparse_mass_row_widths(n, points):
    """Sparse against dense, both FP64: areas of a mesh's vertices differ by up
    to a factor of about 10, so rounding (1e-16 by 36 steps) stays below 1e-12."""
    ctx = B.Context(0)
    y = []
    xyz, tri = synth.icosphere(2 if points == 162 else 4) if n == 6 else _rosette(n, points)
    assert np.bincount(tri.ravel()).max() == n
    m = B.Mesh(ctx, xyz, tri)
    for mode in (1, 2):
        p = B.Problem(ctx, m, m, 2.0, 3.0, 1.0, 1.5, precision=B.C128)
        p.set_mass_apply(mode)
        p.assemble_operators()
        p.assemble_projection()
        assert p.mass_apply_sparse() == (mode == 2)
        x = np.random.default_rng(9).standard_normal((2, p.n))
        y.append(p.mtf_matvec(torch.from_numpy(x[0] + 1j * x[1]), strong=True).cpu().numpy())
    assert _rel(y[1], y[0]) < 1e-12


@pytest.mark.parametrize("ne,ni,R", [(642, 642, 64), (1500, 700, 37), (2600, 2000, 64)])
def test_sparse_mass_several_vectors_a_workgroup(ne, ni, R):
    """Runs that are one vector times powers of two: the same bits but for the exponent."""
    p = _problem(B.Context(0), ne, ni, B.C64_MIXED, 2)
    assert p.mass_apply_sparse()
    x = np.random.default_rng(3).standard_normal((2, p.n))
    scale = 2.0 ** (np.arange(R) % 9 - 4)
    X = scale[:, None] * (x[0] + 1j * x[1])
    Y = p.mtf_matvec_batch(torch.from_numpy(X), strong=True).cpu().numpy()
    assert np.abs(Y[0]).max() > 0 and all(np.array_equal(Y[r] / scale[r], Y[0] / scale[0]) for r in range(R))
    # one vector alone: the FP32 sums of another tile width, times at most 2 by M^-1
    one = p.mtf_matvec_batch(torch.from_numpy(X[:1]), strong=True).cpu().numpy()
    assert _rel(Y[0], one[0]) < 4e-6


# rows within and beyond half of the LDS and the whole (complex128 rows of 16 n bytes, complex64 of 8 n), and
# an odd number of complex64 entries
@pytest.mark.parametrize("prec,n", [(B.C128, 2048), (B.C128, 2049), (B.C128, 5200), (B.C128, 5601), (B.C128, 10100),
                                    (B.C64_MIXED, 41), (B.C64_MIXED, 2049), (B.C64_MIXED, 10101),
                                    (B.C64_MIXED, 11201)])
def test_operator_in_caller_numbering(prec, n):
    """The same mesh in another numbering: the same entries, but for the
    rounding of other blocks' orders of summation."""
    ctx = B.Context(0)
    xyz, tri = synth.fibonacci_sphere(n)
    perm = np.random.default_rng(n).permutation(n)
    inv = np.argsort(perm)
    got = []
    for x, t in ((xyz, tri), (xyz[perm], inv[tri].astype(np.int32))):
        m = B.Mesh(ctx, x, t)
        small = B.Mesh(ctx, *synth.icosphere(0))
        p = B.Problem(ctx, m, small, 1.0, 1.5, 1.0, 1.5, precision=prec)
        p.assemble_operators()
        got.append(p.operator(0, "K"))
        del p
    i = torch.from_numpy(perm).cuda()
    want = got[0][i[:, None], i[None, :]]
    tol = 1e-12 if prec == B.C128 else 2e-5
    assert (got[1] - want).abs().max() < tol * want.abs().max()


# tiles of 16 waves (240 tile pairs) and of four (272), tiles of one vertex, one tile
@pytest.mark.parametrize("ne,ni", [(959, 960), (961, 1000), (65, 129), (33, 64)])
@pytest.mark.parametrize("prec,tol", [(B.C128, 1e-13), (B.C64_MIXED, 2e-6)])
def test_matvec_against_its_operators(ne, ni, prec, tol):
    """The weak product against the copied operators and the projection; mixed
    at the bound of two FP32 summation orders."""
    from scipy.sparse import csr_matrix
    p = _problem(B.Context(0), ne, ni, prec)
    rng = np.random.default_rng(7)
    x = rng.standard_normal(p.n) + 1j * rng.standard_normal(p.n)
    ve, we, vi, wi = np.split(x, [ne, 2 * ne, 2 * ne + ni])
    op = {(m, o): p.operator(m, o).to(torch.complex128).cpu().numpy() for m in (0, 1) for o in "VKTD"}
    rp, col, val = p.projection()
    P = csr_matrix((val, col, rp), shape=(ni, ne))
    r = 1.0 / 1.5
    ref = np.concatenate([-op[0, "K"] @ ve + op[0, "V"] @ we + 0.5 * (P.T @ vi),
                          op[0, "D"] @ ve + op[0, "T"] @ we + 0.5 * r * (P.T @ wi),
                          -0.5 * (P @ ve) - op[1, "K"] @ vi + op[1, "V"] @ wi,
                          -0.5 / r * (P @ we) + op[1, "D"] @ vi + op[1, "T"] @ wi])
    y = p.mtf_matvec(torch.from_numpy(x), strong=False).cpu().numpy()
    assert _rel(y, ref) < tol
