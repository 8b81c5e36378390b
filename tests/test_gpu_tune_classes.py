"""Size classes of the mat-vec's tuned tile edge: 1,920 + 1,920 and 1,921 +
1,921 vertices are of one class, the first pair too small to be timed (240
pairs of 128-column tiles), the second one (272) not."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

B = pytest.importorskip("paper_2206_00708_amd")


def _product(cx, n):
    m = B.Mesh(cx, *synth.fibonacci_sphere(n))
    p = B.Problem(cx, m, m, 2.0, 3.0)
    p.assemble_operators()
    p.assemble_projection()
    rng = np.random.default_rng(n)
    p.mtf_matvec(torch.as_tensor(rng.standard_normal(p.n) + 1j * rng.standard_normal(p.n)))
    for h in (p, m):
        h.close()


def test_small_pair_leaves_its_class_to_be_timed():
    assert torch.cuda.is_available(), "GPU tests need a device"
    assert round(4 * np.log2(1920)) == round(4 * np.log2(1921)) == 44
    key = "mtf-c128:e44:i44"
    cx = B.Context(0)
    before = key in B.tune_table()
    _product(cx, 1920)
    assert (key in B.tune_table()) == before
    assert B.tune_table()[key + ":small"] == [64]
    _product(cx, 1921)
    assert key in B.tune_table()
    cx.close()
