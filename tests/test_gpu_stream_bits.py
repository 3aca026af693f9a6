"""Streamed FP64 column launches (512 and 1024 lines of 2048 points, blended modes) end
bitwise as a workgroup per tile does (256 lines, below the streamed launch's least tile
count).  FP64 has one schedule of that shape, so the two are compared over grids:
on states, metrics and layers that do not depend on x a row transform returns every
column alike, and all columns that no layer in x touches have to agree."""
import numpy as np
import pytest

from paper_1909_02894_amd import workloads as W

pytestmark = pytest.mark.gpu
N2 = 2048


@pytest.mark.parametrize("kind", ["layer", "curved"])
@pytest.mark.parametrize("n1", [512, 1024])
def test_streamed_fp64_columns_same_bits(n1, kind):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_02894_amd import dirac as D
    rng = np.random.default_rng(5)
    col = rng.standard_normal((N2, 1, 2)) + 1j * rng.standard_normal((N2, 1, 2))
    y = -20.0 + np.arange(N2)[:, None] * (40.0 / N2)
    phi, dphi = -0.1 * np.exp(-y ** 2 / 9), 0.1 * np.exp(-y ** 2 / 9) * 2 * y / 9

    def solve(width):
        print(f"[stream bits] {width}x{N2} {kind}", flush=True)
        kw, steps = dict(pml_width=16), 1          # the x layer rounds its own columns: one step
        if kind == "curved":
            one = np.ones((1, width))
            z = np.zeros((N2, width))
            kw, steps = dict(metric=D.METRIC_FIELDS, spin=D.SPIN_PAPER,
                             fields=(phi * one, z, z, dphi * one, z, z)), 3
        s = D.Solver(width, N2, 20.0, 20.0, 0.002, 1.0, 0.7, D.FP64, **kw)
        s.set_schedule(1, 16, 2, 2)
        s.set_initial_spinor(np.repeat(col, width, axis=1))
        s.step_n(steps)
        out = s.get_spinor()
        s.close()
        lo = 17 if kind == "layer" else 0          # the seam's neighbours hold the layer
        inner = out[:, lo:width - 16 if kind == "layer" else width]
        assert np.array_equal(inner, np.repeat(inner[:, :1], inner.shape[1], axis=1))
        return inner[:, 0]

    assert np.array_equal(solve(n1), solve(256))
