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
