"""Device memory limits of a context: a call that does not fit returns
BEM_E_OOM and leaves the context usable.  Expected values are the same calls'
results in a context without a limit, bit for bit (the kernels and their order
are the same)."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2206_00708_amd")

E_OOM = -5
PAIR = (synth.icosphere(2), synth.fibonacci_sphere(130))


def _operators(p):
    return [p.operator(m, op).cpu().numpy() for m in (0, 1) for op in "VKTD"]


def _assembled(cx, pair=PAIR):
    me, mi = B.Mesh(cx, *pair[0]), B.Mesh(cx, *pair[1])
    p = B.Problem(cx, me, mi, 2.0, 3.0, 1.0, 1.5)
    try:
        p.assemble_operators()
        return _operators(p), cx.bytes_in_use()
    finally:
        for h in (p, me, mi):
            h.close()


@pytest.fixture(scope="module")
def unlimited():
    assert torch.cuda.is_available(), "GPU tests need a device"
    small = (synth.icosphere(1), synth.icosphere(1))
    cx = B.Context(0)
    want, used = _assembled(cx)
    want_small, _ = _assembled(cx, small)
    cx.close()
    return want, used, small, want_small


@pytest.mark.parametrize("short", [1, 1 << 18, 1 << 20, 12 << 20])
def test_assembly_over_the_budget_leaves_the_context_usable(unlimited, short):
    """An assembly whose memory is `short` bytes below what it takes without a
    limit either succeeds or fails whole; after a failure the context
    assembles another problem."""
    want, used, small, want_small = unlimited
    cx = B.Context(0, hbm_budget_bytes=used - short)
    try:
        got, _ = _assembled(cx)
        assert all(np.array_equal(g, w) for g, w in zip(got, want))
    except B.BemError as e:
        assert e.code == E_OOM, e
    got, _ = _assembled(cx, small)
    assert all(np.array_equal(g, w) for g, w in zip(got, want_small))
    assert cx.bytes_in_use() <= used - short
    cx.trim()
    assert cx.bytes_in_use() == 0
    cx.close()


def test_assembly_fits_where_one_region_does(unlimited):
    """The budget of the operators, the tables and the larger of the two
    scratch regions is enough.  The regions hold 36,864 bytes per pair of the
    meshes' blocks of 16 triangles: 20 blocks of 320, 16 of 256 triangles."""
    want, used, _, _ = unlimited
    assert len(PAIR[0][1]) == 320 and len(PAIR[1][1]) == 256
    spare = 16 * 17 // 2 * 36864
    cx = B.Context(0, hbm_budget_bytes=used - spare)
    for _ in range(2):   # the second one with the blocks that the first has released
        got, in_use = _assembled(cx)
        assert in_use <= used - spare
        assert all(np.array_equal(g, w) for g, w in zip(got, want))
    cx.close()


def test_footprint_counts_one_region():
    """The footprint that admission works with: operators, dense inverse
    masses, the larger scratch region, Krylov basis and work vectors,
    Hessenberg and triangular factors, partial sums, bound of the couplings."""
    cx = B.Context(0)
    me, mi = B.Mesh(cx, *PAIR[0]), B.Mesh(cx, *PAIR[1])
    p = B.Problem(cx, me, mi, 2.0, 3.0, 1.0, 1.5)
    ne, ni, maxit = 162, 130, 50
    n = 2 * (ne + ni)
    want = (4 * (ne * 192 + ni * 160) * 16 + (ne * ne + ni * ni) * 8 + 20 * 21 // 2 * 36864
            + ((maxit + 1) * n + 8 * n) * 16 + 2 * maxit * (maxit + 1) * 16
            + (n + 1023) // 1024 * 2 * (maxit + 1) * 16 + 64 * (ne + ni) * 8)
    assert p.footprint(1, maxit) == want
    for h in (p, me, mi):
        h.close()
    cx.close()


def test_field_and_winding_fit_where_one_region_does():
    """A field of one right-hand side needs, beside its points, the unknowns,
    368 bytes per triangle of one region and 16 bytes per point and chunk of
    it (13 chunks of the 5,120 triangles for 40,000 points); a winding number
    8 bytes per point and chunk (40 for 256 points).  In allocation sizes:
    2, 1/2, 1/4, 2 and 10 MB, and 1/8 MB.  The sums run in another order than
    without a limit (1e-12 of the largest value)."""
    ext, inte, _ = synth.make_pair(7, 4, "ico", 0.02, (1.0, 0.9, 0.8), int_level=4)
    rng = np.random.default_rng(4)
    pts = torch.as_tensor(rng.uniform(1.5, 3.0, (80000, 3)), device="cuda")
    region = torch.arange(80000, device="cuda", dtype=torch.int32) % 2
    n = 2 * (len(ext[0]) + len(inte[0]))
    x = torch.as_tensor(rng.standard_normal((2, n)) + 1j * rng.standard_normal((2, n)), device="cuda")
    d = synth.plane_wave_directions(2, rng)

    def base():
        cx = B.Context(0)
        me, mi = B.Mesh(cx, *ext), B.Mesh(cx, *inte)
        b = cx.bytes_in_use()
        for h in (me, mi, cx):
            h.close()
        return b

    def run(budget, call):
        cx = B.Context(0, hbm_budget_bytes=budget)
        me, mi = B.Mesh(cx, *ext), B.Mesh(cx, *inte)
        p = B.Problem(cx, me, mi, 3.0, 4.0)
        out = call(p, me).cpu().numpy()
        for h in (p, me, mi, cx):
            h.close()
        return out

    tables = base()
    for call, mb in ((lambda p, m: p.field(d, x, pts, region), 14.75), (lambda p, m: m.winding(pts[:256]), 0.125)):
        want = run(0, call)
        got = run(tables + int(mb * (1 << 20)), call)
        assert np.max(np.abs(got - want)) < 1e-12 * max(1.0, np.max(np.abs(want)))
