"""Noisy steps where the increment is drawn in the step: the shape and the band height the
library picks are not slower than the region form with a pass for the increments (up to 5 %,
the spread between runs), also where the grid has slightly more waves than the device has
SIMDs, and in calls of one step; the tall one-column shapes take the library's height."""
import time

import pytest

from gpu_helpers import C64
from test_gpu_pairs_pay import solver
from test_gpu_step_walk import end_state, same

pytestmark = pytest.mark.gpu


def noisy(n, bc, tile):
    return solver(n, n, C64, bc, True, False, tile=tile, noise=1.0)


def call_us(s, steps):
    import torch
    best = float("inf")
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(20):
            s.step(steps)
        torch.cuda.synchronize()
        best = min(best, 1e6 * (time.perf_counter() - t) / 20)
    s.close()
    return best


@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
@pytest.mark.parametrize("n,steps", [(1100, 1), (1500, 1), (1100, 16), (1400, 16), (1500, 16), (2048, 16)])
def test_default_shape_pays(n, steps, bc):
    default, region = call_us(noisy(n, bc, (0, 0)), steps), call_us(noisy(n, bc, (8, 4)), steps)
    print(f"default {default:.1f} region {region:.1f}")
    assert default <= 1.05 * region


@pytest.mark.parametrize("rows", [88, 112])
def test_tall_one_column_shapes(rows):
    tall, picked = call_us(noisy(2048, (0, 0), (1, rows)), 16), call_us(noisy(2048, (0, 0), (1, 64)), 16)
    assert tall <= 1.1 * picked


@pytest.mark.parametrize("nx,ny", [(1100, 1024), (1400, 1400), (1536, 1025)])
def test_calls_of_one_step_bitwise(nx, ny):
    kw = dict(noise=0.6, seed=5)
    assert same(end_state("driven", nx, ny, (0, 0), C64, (0, 0), calls=(1, 1, 3), **kw),
                end_state("driven", nx, ny, (0, 0), C64, (2, 0), calls=(5,), **kw))


def test_overflow_of_the_increment_is_reported():
    """An increment that is not finite sets the flag in the step that adds it."""
    from paper_2411_18341_amd import phx
    s = solver(256, 64, C64, (0, 0), True, False, tile=(2, 0), noise=1e300)
    s.step(2)
    assert s.observables()["nonfinite"] > 0
    with pytest.raises(phx.PhxError):
        s.step(1)
    s.close()
