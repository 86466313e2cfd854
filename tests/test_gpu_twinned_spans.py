"""The twinned iteration kernel at the edges of its decomposition: row spans of
124 cells (whole, one cell over, several even ones), wavefronts of 2 and blocks
of 8 rows, marches that end inside a span of planes, and the buffer an
iteration count ends in.  Against the FP64 oracle with the bar of
test_gpu_twinned.py: every half rounds each value a few times in float32 (a
contraction, so errors do not grow), 1e-5 relative."""
import numpy as np
import pytest

from test_gpu_twinned import ALL_WALLS, rel, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (123, 5, 4), (124, 8, 16), (125, 9, 17), (126, 7, 33), (249, 10, 6),
                                   (372, 4, 5), (11, 131, 70), (250, 37, 46)])
@pytest.mark.parametrize("iters", [1, 2, 3])
def test_twinned_spans_match_oracle(shape, iters):
    print(f"[twinned] {shape} iters={iters}", flush=True)
    got, want, st, _, r_or, g = run(*shape, 0.9, iters, seed=sum(shape))
    g.close()
    assert rel(got, want) <= 1e-5
    assert st["iters"] == iters
    assert st["resid"] == pytest.approx(r_or, rel=1e-4)


def test_twinned_solve_is_reproducible():
    """Iterates and float64 residual have one fixed order."""
    a = run(125, 12, 9, 1.0, 4, bc=ALL_WALLS, seed=2)
    b = run(125, 12, 9, 1.0, 4, bc=ALL_WALLS, seed=2)
    a[-1].close()
    b[-1].close()
    assert np.array_equal(a[0], b[0]) and a[2] == b[2]
