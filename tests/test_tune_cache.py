"""The cache of tuned shapes: one record per set of terms of the step and per revision of the
shapes; a record that the library refuses is measured again and leaves the solver usable; a
shape from the cache keeps the solver's progress."""
import json

import pytest

from paper_2411_18341_amd import phx


def config(**kw):
    return phx.make_config(64, 48, 0.2, g=0.01, dt=0.01, **kw)


def test_keys_are_distinct():
    cfgs = [config(), config(noise=0.5), config(drive=True), config(imag_time=True), config(reservoir=True),
            config(integrator=phx.PHX_RK45), config(precision=phx.PHX_C128), config(components=2),
            config(bc_x=phx.PHX_BC_ZERO), config(bc_y=phx.PHX_BC_ZERO), config(kernel=phx.PHX_KERNEL_STEP)]
    keys = [phx.tune_key(c, v, "dev") for c in cfgs for v in (False, True)]
    assert len(set(keys)) == len(keys)
    assert phx.tune_key(config(noise=0.5), False) == phx.tune_key(config(noise=0.7, seed=3), False)


def test_records_of_another_revision_are_not_used(tmp_path, monkeypatch):
    monkeypatch.setenv("PHX_TUNE_CACHE", str(tmp_path / "tune.json"))
    cfg = config()
    record = {"tile_wx": 3, "tile_rows": 64}
    old = f"dev|k{cfg.kernel}|p{cfg.precision}|64x48|c1|r0|v0|bc00"  # as written without a revision
    (tmp_path / "tune.json").write_text(json.dumps({old: record}))
    assert phx.cached_shape(cfg, False, "dev") is None
    (tmp_path / "tune.json").write_text(json.dumps({phx.tune_key(cfg, False, "dev"): record}))
    assert phx.cached_shape(cfg, False, "dev") == (3, 64)
    monkeypatch.setattr(phx, "TUNE_REVISION", phx.TUNE_REVISION + 1)
    assert phx.cached_shape(cfg, False, "dev") is None


def stored(tmp_path, monkeypatch, s, shape):
    import torch
    monkeypatch.setenv("PHX_TUNE_CACHE", str(tmp_path / "tune.json"))
    phx.store_shape(s.cfg, False, phx.phx_tune_result(phx.PHX_KERNEL_STEP, *shape, 5, 10.0, 12.0),
                    torch.cuda.get_device_name(s.psi.device))


@pytest.mark.gpu
def test_a_refused_record_is_measured_again(tmp_path, monkeypatch):
    import torch
    s = phx.Solver(config(imag_time=True), torch.ones((1, 48, 64), dtype=torch.complex64, device="cuda:0"))
    stored(tmp_path, monkeypatch, s, (8, 4))  # imaginary time has no region form
    r = s.autotune(reps=2)
    assert not r["cached"] and r["tile_wx"] in (1, 2)
    s.step(3)
    s.observables()
    s.close()


@pytest.mark.gpu
def test_a_cached_shape_keeps_the_progress(tmp_path, monkeypatch):
    import torch
    psi = []
    for tune in (False, True):
        s = phx.Solver(config(noise=0.5, gamma_c=0.2, seed=4), torch.ones((1, 48, 64), dtype=torch.complex64, device="cuda:0"))
        s.step(3)
        if tune:
            stored(tmp_path, monkeypatch, s, (1, 64))
            assert s.autotune(reps=2)["cached"]
        assert s.info()["steps_accepted"] == 3
        s.step(2)
        torch.cuda.synchronize()
        psi.append(s.psi.clone())
        s.close()
    assert torch.equal(psi[0], psi[1])
