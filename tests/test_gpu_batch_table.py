"""The batch's instance table goes to the device as launch arguments, 16 to 25 instances at a
time, or as a copy when it is long; with two column counts per lane one launch covers both
lists.  Around the chunks' edges every instance looked at equals a single-grid run of the
region form bit for bit, over calls of 1, 2 and 3 steps."""
import numpy as np
import pytest

from gpu_helpers import C64, C128
from paper_2411_18341_amd import phx
from test_gpu_rk4_pair import case, states

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [C64, C128])
@pytest.mark.parametrize("has_v", [False, True])
@pytest.mark.parametrize("count", [1, 17, 24, 25, 26, 51, 97, 151, 160])
def test_table_chunks(count, has_v, precision):
    import torch
    rng = np.random.default_rng(count)
    grids = [(int(rng.integers(1, 150)), int(rng.integers(1, 60))) for _ in range(count)]
    fields = []
    for k, (nx, ny) in enumerate(grids):
        ph, q = case(nx, ny, (0, 1), True, has_v, seed=k, precision=precision)
        fields.append((ph, q))
    b = phx.Batch(grids, [phx.config_from_physics(ph, precision=precision)], precision=precision, with_v=has_v)
    for k, (_, q) in enumerate(fields):
        for t, f in ((b.psi, q[0][0]), (b.n, q[1][0]), (b.P, q[3][0])) + (((b.V, q[2]),) if has_v else ()):
            b.view(t, k).copy_(torch.from_numpy(np.ascontiguousarray(f)))
    look = sorted({0, count - 1} | {k for e in (15, 16, 24, 25, 48, 50, 144, 150) for k in (e - 1, e) if 0 <= k < count})
    want = {k: states(*fields[k], (8, 4), (1, 2, 3), precision=precision) for k in look}
    for i, steps in enumerate((1, 2, 3)):
        b.step(steps)
        torch.cuda.synchronize()
        for k in look:
            assert np.array_equal(b.view(b.psi, k).cpu().numpy().astype(np.complex128), want[k][i][0][0]), (k, i)
            assert np.array_equal(b.view(b.n, k).cpu().numpy().astype(np.float64), want[k][i][1][0]), (k, i)
