"""Which plans run as teams of 64 samples (tiles of 64) and which of the small ones run one lane per
sample (tiles of 256, one workgroup each): by the horizon, and beyond three opponents by the teams
that LDS keeps resident.  Both kinds choose the same samples and leave the same bits (against
plans of two samples per lane)."""

import numpy as np
import pytest

import parity as PY
from paper_2607_25388_amd import inputs

pytestmark = pytest.mark.gpu

TEAM, ONE = 64, 256


@pytest.fixture(scope="module")
def planner():
    import paper_2607_25388_amd.sgtp as sg
    p = sg.Planner(max_agents_total=384, max_races=126, max_K=1 << 16)
    p.enable_path_integral()
    yield p
    p.close()


def _plan(planner, track, races, params, K, opt):
    import paper_2607_25388_amd.sgtp as sg
    planner.upload_track(0, track)
    rts = [sg.race_from_inputs(r, 0, K, params["N"], params["n_tail"]) for r in races]
    return planner.plan(params, rts, 1, opt, trace=True), rts


@pytest.mark.parametrize("model,n,R,K,N,tile", [
    (0, 3, 1, 128, 1, TEAM), (0, 1, 1, 65536, 7, ONE), (0, 1, 1, 65536, 8, TEAM), (1, 1, 1, 65536, 12, ONE),
    (1, 1, 1, 65536, 13, TEAM), (0, 3, 1, 16384, 5, ONE), (0, 3, 1, 16384, 6, TEAM), (1, 3, 126, 128, 9, ONE),
    (1, 3, 126, 128, 12, TEAM), (0, 10, 1, 4000, 4, ONE), (0, 10, 1, 4000, 5, TEAM), (0, 3, 1, 16384, 64, TEAM)])
def test_horizon(planner, model, n, R, K, N, tile):
    _check(planner, inputs.make_fourier_track(300.0, 10.0, 1000), 8.0, dict(inputs.default_params(N, 1), model=model),
           n, R, K, tile)


@pytest.mark.parametrize("ds,n,K,tile", [(0.5, 16, 3072, TEAM), (0.2, 16, 2048, TEAM), (0.2, 16, 2049, ONE),
                                         (0.2, 16, 3072, ONE), (0.1, 2, 16640, TEAM)])
def test_resident_teams(planner, ds, n, K, tile):
    """16 vehicles: three teams per CU with 0.5 m nodes (46 KB), two with 0.2 m nodes (58 KB); up to
    three opponents the second round stays."""
    params = dict(inputs.default_params(40, 3 if n > 4 else 1), max_moves=64)
    _check(planner, inputs.make_fourier_track(300.0, 10.0, 1000, ds=ds), 8.0, params, n, 1, K, tile)


def _check(planner, track, spacing, params, n, R, K, tile):
    import torch
    import paper_2607_25388_amd.sgtp as sg
    races = [inputs.make_race(track, n, params["N"], spacing, n >= 4, 3000 + r, 2000 + r) for r in range(R)]
    out = []
    for spl in (1, 2):
        plan, rts = _plan(planner, track, races, params, K, sg.plan_options(samples_per_lane=spl, persistent=2 - spl))
        info = plan.info()
        if spl == 1:
            assert info["tiles"] == info["grid"] == n * R * -(-K // tile), info
        print(f"case {n} {R} {K} {params['N']} {info}", flush=True)
        plan.run()
        u = plan.run()
        torch.cuda.synchronize()
        out.append([plan.choices().tobytes(), u.cpu().numpy().tobytes()] + [t.cpu().numpy().tobytes()
                   for rt in rts for t in (rt.u_nom, rt.traj) if t is not None])
        plan.close()
    assert out[0] == out[1]
    assert planner.status() == 0


@pytest.mark.parametrize("K", [700, 30000, 65536])
def test_path_integral_of_few_opponents_stays_with_teams(planner, K):
    """Its sums are taken over 128 samples, whatever the horizon."""
    import paper_2607_25388_amd.sgtp as sg
    track = inputs.make_fourier_track(300.0, 10.0, 1000)
    params = dict(inputs.default_params(2, 1), update=1)
    plan, _ = _plan(planner, track, [inputs.make_race(track, 1, 2, 8.0, False, 3000, 2000)], params, K, sg.plan_options())
    assert plan.info()["tiles"] == -(-K // TEAM)
    plan.close()


@pytest.mark.parametrize("model,K", [(0, 32768), (0, 32769), (0, 49153), (1, 32769)])
def test_two_samples_per_lane_around_one_wave_per_simd(planner, model, K):
    """256 workgroups read ahead, 260 do not: the same choices as one sample per lane."""
    import torch
    import paper_2607_25388_amd.sgtp as sg
    track = inputs.make_fourier_track(300.0, 10.0, 1000)
    params = dict(inputs.default_params(12, 1), model=model)
    race = inputs.make_race(track, 4, 12, 8.0, True, 3000, 2000)
    out = []
    for spl in (1, 2):
        plan, rts = _plan(planner, track, [race], params, K, sg.plan_options(persistent=0, samples_per_lane=spl))
        plan.run()
        u = plan.run()
        torch.cuda.synchronize()
        out.append((plan.choices().tobytes(), u.cpu().numpy().tobytes(), rts[0].u_nom.cpu().numpy().tobytes()))
        plan.close()
    assert out[0] == out[1]


@pytest.mark.parametrize("n,R,K", [(1, 1, 262144), (1, 1, 262145), (4, 8, 8300), (2, 9, 20000)])
def test_kinematic_point_footprint_at_five_workgroups_per_cu(planner, n, R, K):
    """Beyond 1024 workgroups the kernel with fewer registers runs: the bits of the persistent one."""
    import torch
    import paper_2607_25388_amd.sgtp as sg
    track = inputs.make_fourier_track(300.0, 10.0, 1000)
    params = dict(inputs.default_params(10, 1), model=1)
    races = [inputs.make_race(track, n, 10, 8.0, n >= 4, 3000 + r, 2000 + r) for r in range(R)]
    p = sg.Planner(max_agents_total=n * R, max_races=R, max_K=K)
    try:
        out = []
        for persistent in (0, 1):
            plan, rts = _plan(p, track, races, params, K, sg.plan_options(persistent=persistent))
            assert plan.info()["tiles"] == n * R * -(-K // ONE)
            plan.run()
            u = plan.run()
            torch.cuda.synchronize()
            out.append([plan.choices().tobytes(), u.cpu().numpy().tobytes()] + [r.u_nom.cpu().numpy().tobytes() for r in rts])
            plan.close()
        assert out[0] == out[1]
    finally:
        p.close()
