"""The one-step streaming walk and the forms chosen around it.

The walks give the same bits for every band height and column count: bands of 8 rows (small
grids), of the height the library picks, and taller ones; single steps and pairs of steps
with the drive; the Wiener increment drawn in the step or in the pass after it, with zero
boundaries.  In imaginary time the restoring scale is summed by the waves themselves (up to
512 of them) or by a pass."""
import numpy as np
import pytest

import oracle
from gpu_helpers import C64, C128, TOL, GpuRun, oracle_physics, quantize, rel_l2
from paper_2411_18341_amd import phx
from test_gpu_drive import OMEGA, drive_profile, quantize_e
from test_gpu_rk4 import workload

pytestmark = pytest.mark.gpu


def end_state(kind, nx, ny, bc, precision, tile, calls=(3, 2), drive=False, **kw):
    ph, psi, n, V, P = workload(kind, nx, ny, bc, seed=nx + ny)
    if kw.get("imag_time"):
        n = P = None
    q = quantize(precision, psi, n, V, P)
    if drive:
        kw.update(E=quantize_e(precision, drive_profile(ph, 3)), drive_omega=OMEGA)
    run = GpuRun(ph, *q, precision=precision, kernel=phx.PHX_KERNEL_STEP, tile_wx=tile[0], tile_rows=tile[1], **kw)
    for k in calls:
        run.step(k)
    out = run.state()
    run.close()
    return out


def same(a, b):
    return np.array_equal(a[0], b[0]) and (a[1] is None or np.array_equal(a[1], b[1]))


@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", [(2, 1), (118, 7), (120, 8), (122, 9), (250, 65)])
def test_wide_band_heights_bitwise(nx, ny, bc):
    region = end_state("driven_v", nx, ny, bc, C64, (8, 4))
    for rows in (8, 13, 40, 64):
        assert same(region, end_state("driven_v", nx, ny, bc, C64, (2, rows))), rows


@pytest.mark.parametrize("precision", [C64, C128])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("nx,ny", [(1, 1), (55, 39), (56, 40), (57, 41), (170, 90)])
def test_one_column_bitwise(nx, ny, bc, precision):
    region = end_state("driven_v", nx, ny, bc, precision, (8, 4))
    assert same(region, end_state("driven_v", nx, ny, bc, precision, (1, 40)))


@pytest.mark.parametrize("graph_steps", [-1, 2])
@pytest.mark.parametrize("precision,nx,ny", [(C64, 1449, 1448), (C64, 1447, 1449), (C128, 1448, 1450), (C64, 61, 33)])
def test_drive_pairs_bitwise(precision, nx, ny, graph_steps):
    """Around 2^21 cells, from which driven runs take two steps per launch; 40 rows: single."""
    kw = dict(drive=True, calls=(4, 3), graph_steps=graph_steps)
    assert same(end_state("driven_v", nx, ny, (1, 0), precision, (1, 40), **kw),
                end_state("driven_v", nx, ny, (1, 0), precision, (1, 64), **kw))


@pytest.mark.parametrize("bc", [(1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("kind", ["driven", "driven_v"])
def test_noise_in_step_zero_boundaries(kind, bc):
    for nx, ny in ((2, 3), (120, 40), (122, 81)):
        kw = dict(noise=0.6, seed=5)
        assert same(end_state(kind, nx, ny, bc, C64, (8, 4), **kw), end_state(kind, nx, ny, bc, C64, (2, 0), **kw))


@pytest.mark.parametrize("precision", [C64, C128])
@pytest.mark.parametrize("nx,ny,tile", [(3, 2, (1, 64)), (57, 41, (1, 64)), (448, 510, (1, 64)), (448, 640, (1, 64)),
                                        (450, 1100, (1, 40)), (120, 1030, (2, 8)), (1200, 520, (2, 8))])
def test_imag_scale_forms(nx, ny, tile, precision):
    """Wave counts up to and beyond 512, odd and even calls, direct launches and replays."""
    if precision == C128 and tile[0] == 2:
        pytest.skip("two columns per lane: complex64")
    ph, psi, n, V, P = workload("conservative", nx, ny, (0, 1), seed=2)
    q = quantize(precision, psi, None, V, None)
    run = GpuRun(ph, q[0], None, q[2], None, precision=precision, imag_time=True, kernel=phx.PHX_KERNEL_STEP,
                 tile_wx=tile[0], tile_rows=tile[1], graph_steps=4)
    want = q[0]
    for k in (1, 6, 5, 8):
        run.step(k)
        want = oracle.rk4_imag(oracle_physics(ph), want, V=q[2], dt=ph.dt, steps=k)
    got = run.state()[0]
    assert run.observables()["nonfinite"] == 0
    run.close()
    assert rel_l2(got, want) <= TOL[precision]


@pytest.mark.parametrize("bc", [(0, 0), (1, 1)])
@pytest.mark.parametrize("nx,ny", [(720, 724), (725, 728), (1144, 1143), (1146, 1146), (1024, 1024), (1000, 1301),
                                   (1311, 1500), (1537, 1702), (999, 2011)])
def test_pair_heights_bitwise(nx, ny, bc):
    """Grids on which the two-step walk with one column per lane ends inside a chunk, and
    around the sizes from which it is the default."""
    region = end_state("driven", nx, ny, bc, C64, (8, 4), calls=(4, 3))
    assert same(region, end_state("driven", nx, ny, bc, C64, (1, 64), calls=(4, 3)))
    assert same(region, end_state("driven", nx, ny, bc, C64, (0, 0), calls=(4, 3)))
