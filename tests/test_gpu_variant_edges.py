"""The kernels of small launches against the one-lane kernel of large ones, bit for bit, with the
variant of both sides made sure of: a list of more than 65536 samples always runs one lane per
sample, and a plan's number of tiles tells its variant (64 samples per tile: four waves for 64
samples, 128: a pair of lanes per sample, 256: one lane)."""

import numpy as np
import pytest

import parity as PY
from paper_2607_25388_amd import inputs

pytestmark = pytest.mark.gpu

OUT = ("cost", "viol", "flags", "x_final", "noise")
K_LARGE = 100000  # more than TEAM_MAX_SAMPLES, more than 1536 waves
TEAM, PAIR, ONE = 64, 128, 256


@pytest.fixture(scope="module")
def planner():
    import paper_2607_25388_amd.sgtp as sg
    p = sg.Planner(max_agents_total=10, max_races=1, max_K=K_LARGE)
    yield p
    p.close()


def _tile_samples(planner, track, race, params, K):
    """Samples per tile of a plan of the race with K samples a vehicle."""
    import paper_2607_25388_amd.sgtp as sg
    plan = planner.plan(params, [PY.build(planner, track, race, params, K)], 1, sg.plan_options(persistent=0),
                        trace=False)
    tiles = plan.info()["tiles"]
    plan.close()
    fits = [s for s in (TEAM, PAIR, ONE) if tiles == race.n_agents * -(-K // s)]
    assert len(fits) == 1, (tiles, K)
    return fits[0]


def _both(planner, track, race, params, K, variant, agent):
    assert _tile_samples(planner, track, race, params, K) == variant
    assert _tile_samples(planner, track, race, params, K_LARGE) == ONE
    return [PY.gpu_rollout(planner, params, PY.build(planner, track, race, params, k), agent, 1) for k in (K, K_LARGE)]


def _same_bits(small, large, K, keep=slice(None)):
    for nm in OUT:
        a, b = small[nm][keep], large[nm][:K][keep]
        assert np.array_equal(np.ascontiguousarray(a).view(np.uint8), np.ascontiguousarray(b).view(np.uint8)), nm


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("name,agent,K,N", [("c1", 0, 2048, 20), ("c1", 1, 1001, 21), ("c2", 1, 2048, 40),
                                            # horizons shorter than the controls' look-ahead, of its
                                            # length, and one, two and three steps past the ring
                                            ("c1", 0, 300, 1), ("c2", 1, 513, 2), ("c2", 0, 129, 3),
                                            ("c1", 1, 700, 4), ("c2", 2, 1000, 5), ("c2", 0, 333, 6),
                                            ("c2", 1, 900, 7),
                                            # the longest horizon the library takes
                                            ("c2", 2, 2048, 64),
                                            # one sample; a vehicle's last team with one sample
                                            ("c2", 0, 1, 9), ("c2", 1, 65, 9)])
def test_teams_match_one_lane(planner, model, name, agent, K, N):
    track, race, params, _, _ = PY.workload(name)
    race = inputs.make_race(track, race.n_agents, N, 10.0, False, 3000, 2000)
    params = dict(params, N=N, n_tail=inputs.n_tail_from_fraction(0.3, N), model=model)
    if K > 64:
        _same_bits(*_both(planner, track, race, params, K, TEAM, agent), K)
    else:  # (one tile whatever the variant)
        small = PY.gpu_rollout(planner, params, PY.build(planner, track, race, params, K), agent, 1)
        large = PY.gpu_rollout(planner, params, PY.build(planner, track, race, params, K_LARGE), agent, 1)
        _same_bits(small, large, K)
    assert planner.status() == 0


@pytest.mark.parametrize("model,n,N,n_disc,variant", [(0, 2, 40, 1, PAIR), (0, 2, 20, 3, PAIR), (0, 4, 25, 3, PAIR),
                                                      (0, 1, 30, 1, PAIR), (1, 2, 40, 1, ONE), (1, 4, 25, 3, ONE),
                                                      (0, 6, 20, 1, ONE)])
def test_fallback_where_the_rings_do_not_fit(planner, model, n, N, n_disc, variant):
    """4 cm nodes and 80 moves a step make the staged window 1536 rows (48 KiB): with the teams' rings
    (8.2 KB and more) the tables no longer fit in 58 KiB of LDS, without them they do.  The plan is
    built again without teams: a pair of lanes per sample for the dynamic model and at most three
    opponents, one lane (the kernel that reads rows ahead) otherwise."""
    track = inputs.make_fourier_track(300.0, 10.0, 1000, ds=0.04)
    race = inputs.make_race(track, n, N, 10.0, False, 3001, 2001)
    params = dict(inputs.default_params(N, n_disc), model=model, max_moves=80)
    K = 1100
    for agent in {0, n - 1}:
        small, large = _both(planner, track, race, params, K, variant, agent)
        _same_bits(small, large, K)
    r = PY.oracle_for(track, params).rollout_cost(race, n - 1, 1, K)
    PY.check_choice(small["choice"], r, params, f"fallback {model} {n} {N}")


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("fine", [False, True])
def test_tight_corners_and_samples_far_inside(planner, model, fine):
    """A circle of 4 m radius whose cars are headed across its centre: the normals of the rows cross,
    so a point beyond the centre lies behind rows that follow and ahead of rows before."""
    track = inputs.make_circle_track(4.0, 6.0, ds=2 * np.pi * 4.0 / (400 if fine else 50))
    N, K = 30, 1500
    params = dict(inputs.default_params(N, 1), model=model)
    race = inputs.make_race(track, 3, N, 3.0, False, 3002, 2002)
    race.x[:, 2] += np.array([1.5, 1.2, 2.0])
    race.x[:, 3] = [12.0, 6.0, 20.0]
    race.u_nom[:, :, 1] = 0.05
    for agent in range(3):
        small, large = _both(planner, track, race, params, K, TEAM, agent)
        _same_bits(small, large, K)


def test_give_up_leaves_the_other_samples_the_one_lane_bits(planner):
    """Poll bound of one: the samples whose wait gave up are scored non-finite, every other keeps the
    bits of the one-lane kernel."""
    import paper_2607_25388_amd.sgtp as sg
    track, race, params, _, _ = PY.workload("c2")
    K = 4096
    ref = _both(planner, track, race, params, K, TEAM, 1)[1]
    planner.set_poll_limit(1)
    try:
        g = PY.gpu_rollout(planner, params, PY.build(planner, track, race, params, K), 1, 1)
        st = planner.status()
    finally:
        planner.set_poll_limit(1 << 22)
    gave_up = (g["flags"] & 16) > 0
    assert bool(st & sg.SGTP_STATUS_WAIT_GAVE_UP) == bool(gave_up.any())
    assert np.all(np.isinf(g["viol"][gave_up])) and not np.any(g["flags"][gave_up] & 7)
    _same_bits(g, ref, K, ~gave_up)
    assert planner.status() == 0
