"""Two RK4 steps per launch (the wide form with the library's band height, and the
one-column form).

The same arithmetic per cell as the other whole-step forms, so the state equals the
region form's bit for bit: over strip seams (112 output columns, 48 with one column per lane), bands of 20 rows,
grids narrower than a strip's halo, every boundary mix, with and without reservoir and
potential, and for every remainder of the step count (pairs, single steps, graph
replays, an odd count that needs a copy)."""
import numpy as np
import pytest

from gpu_helpers import C64, C128, GpuRun, quantize
from paper_2411_18341_amd import build, inputs, phx

gpu = pytest.mark.gpu


def case(nx, ny, bc, reservoir, has_v, seed=0, precision=C64):
    rng = np.random.default_rng(700 + seed)
    ph = inputs.Physics(nx=nx, ny=ny, dx=0.2, dy=0.25, bc_x=bc[0], bc_y=bc[1], reservoir=reservoir, g=0.01,
                        g_r=0.02 if reservoir else 0.0, R=0.01 if reservoir else 0.0, gamma_c=0.15,
                        gamma_r=0.225 if reservoir else 0.0, dt=0.02)
    psi = inputs.random_state((1, ny, nx), seed, 0.5)
    n = rng.uniform(0, 5, (1, ny, nx)) if reservoir else None
    P = rng.uniform(0, 3, (1, ny, nx)) if reservoir else None
    V = rng.standard_normal((ny, nx)) if has_v else None
    return ph, quantize(precision, psi, n, V, P)


def states(ph, q, tile, calls, graph_steps=0, precision=C64):
    run = GpuRun(ph, *q, precision=precision, kernel=phx.PHX_KERNEL_STEP, tile_wx=tile[0], tile_rows=tile[1],
                 graph_steps=graph_steps)
    out = []
    for k in calls:
        run.step(k)
        out.append(run.state())
    run.close()
    return out


def same(a, b):
    return all(np.array_equal(p[0], q[0]) and (p[1] is None or np.array_equal(p[1], q[1])) for p, q in zip(a, b))


@gpu
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("reservoir", [False, True])
@pytest.mark.parametrize("has_v", [False, True])
def test_pair_edges(has_v, reservoir, bc):
    for nx, ny in ((112, 20), (114, 21), (110, 19), (226, 41), (336, 33), (2, 1), (2, 7), (8, 3), (16, 50), (128, 64)):
        ph, q = case(nx, ny, bc, reservoir, has_v, seed=nx)
        calls = (4, 3)
        assert same(states(ph, q, (8, 4), calls), states(ph, q, (2, 0), calls)), (nx, ny)


@gpu
@pytest.mark.parametrize("precision", [C64, C128])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (0, 1), (1, 0)])
@pytest.mark.parametrize("kind", [(False, False), (True, False), (False, True), (True, True)])
def test_pair_one_column_edges(kind, bc, precision):
    for nx, ny in ((48, 20), (49, 21), (47, 19), (97, 41), (145, 33), (1, 1), (3, 7), (9, 3), (17, 50), (64, 64)):
        ph, q = case(nx, ny, bc, *kind, seed=nx, precision=precision)
        calls = (4, 3)
        assert same(states(ph, q, (8, 4), calls, precision=precision),
                    states(ph, q, (1, 64), calls, precision=precision)), (nx, ny)


@gpu
@pytest.mark.parametrize("tile", [(2, 0), (1, 64)])
@pytest.mark.parametrize("graph_steps", [-1, 2, 4, 6])
def test_pair_step_counts(graph_steps, tile):
    ph, q = case(300, 150, (0, 1), True, False, seed=3)
    calls = (1, 2, 3, 4, 5, 6, 7, 9, 13, 4, 1, 3)
    assert same(states(ph, q, (8, 4), calls, graph_steps), states(ph, q, tile, calls, graph_steps))


@gpu
def test_pair_reports_nonfinite():
    ph, q = case(240, 60, (0, 0), True, False, seed=4)
    q[0][0, 30, 100] = np.nan
    run = GpuRun(ph, *q, precision=C64, kernel=phx.PHX_KERNEL_STEP, tile_wx=2, tile_rows=0)
    run.step(4)
    assert run.observables()["nonfinite"] > 0
    with pytest.raises(phx.PhxError):
        run.step(1)
    run.close()


@gpu
@pytest.mark.parametrize("precision,nx,ny", [(C64, 1254, 1254), (C64, 1256, 1253), (C64, 1915, 1916), (C64, 1916, 1916),
                                             (C64, 2049, 1900), (C128, 887, 886), (C128, 890, 888)])
def test_default_shape_bitwise(nx, ny, precision):
    """Around the sizes from which the default is the one-column and the wide walk."""
    ph, q = case(nx, ny, (0, 1), True, False, seed=6, precision=precision)
    run = GpuRun(ph, *q, precision=precision)
    run.step(5)
    default = [run.state()]
    run.close()
    assert same(states(ph, q, (8, 4), (5,), precision=precision), default)


@pytest.mark.parametrize("unit", ["rk4_stream_pair_f2.hip", "rk4_stream_pair_d1.hip", "dp_walk_d1.hip"])
def test_wide_stores_keep_their_data(unit):
    """No store of more than 64 bits has its data rewritten by the next instruction."""
    asm = build.device_asm(unit)
    assert "buffer_store_dwordx4" in asm
    assert build.store_data_hazards(asm) == []


@gpu
@pytest.mark.parametrize("precision", [C64, C128])
@pytest.mark.parametrize("bc", [(0, 0), (1, 1), (1, 0)])
def test_batch_pairs_bitwise(bc, precision):
    """Batches of even and odd widths around the strips of both column counts: after 4, 3
    and 1 batched steps each instance equals a single-grid run of the region form."""
    grids = [(112, 20), (114, 33), (49, 21), (97, 5), (2, 9), (1, 1), (226, 105), (130, 230)]
    import torch
    runs, fields = [], []
    for k, (nx, ny) in enumerate(grids):
        ph, q = case(nx, ny, bc, True, False, seed=50 + k, precision=precision)
        fields.append(q)
        runs.append(states(ph, q, (8, 4), (4, 3, 1), precision=precision))
    b = phx.Batch(grids, [phx.config_from_physics(ph, precision=precision)], precision=precision)
    for k, q in enumerate(fields):
        for t, f in ((b.psi, q[0][0]), (b.n, q[1][0]), (b.P, q[3][0])):
            b.view(t, k).copy_(torch.from_numpy(np.ascontiguousarray(f)))
    for i, steps in enumerate((4, 3, 1)):
        b.step(steps)
        torch.cuda.synchronize()
        for k in range(len(grids)):
            assert np.array_equal(b.view(b.psi, k).cpu().numpy().astype(np.complex128), runs[k][i][0][0]), (k, i)
            assert np.array_equal(b.view(b.n, k).cpu().numpy().astype(np.float64), runs[k][i][1][0]), (k, i)
