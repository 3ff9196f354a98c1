"""The throughput variant of the sweep (one lane per sample, several waves per SIMD) against
the small-launch variant (64 samples on the four waves of a workgroup, both vehicle models,
up to and beyond three opponents), bit for bit, where its own code differs: the batched raceline walk
(fine nodes: many nodes per step; few moves allowed: the walk's limit; the end of an open
track: the window's limit), the screening of the opponents in groups (every remainder of a
group), the clip without its NaN test (a NaN and an infinite nominal control) and the
proposal's samples."""

import numpy as np
import pytest

import parity as PY
from paper_2607_25388_amd import inputs

pytestmark = pytest.mark.gpu

OUT = ("cost", "viol", "flags", "x_final", "noise")
K_LARGE, K_SMALL = 100000, 1500  # more than 1536 waves against one workgroup per 64 samples


@pytest.fixture(scope="module")
def planner():
    import paper_2607_25388_amd.sgtp as sg
    p = sg.Planner(max_agents_total=10, max_races=1, max_K=K_LARGE)
    yield p
    p.close()


def _case(name):
    n, N, over, track = 3, 40, {}, inputs.make_fourier_track(300.0, 10.0, 1000)
    if name == "fine_nodes":
        track = inputs.make_fourier_track(300.0, 10.0, 1000, ds=0.1)
        n, N = 2, 30
    elif name == "two_moves":
        over = dict(max_moves=2)
    elif name == "one_move":
        over = dict(max_moves=1)
    elif name == "open_end":
        track = inputs.make_straight_track(120.0, 10.0, vref=40.0)
    elif name.startswith("kinematic"):
        n, N, over = int(name[9:]), 17, dict(model=1)
    elif name.startswith("vehicles"):
        n, N = int(name[8:]), 25
    params = dict(inputs.default_params(N, 3), **over)
    race = inputs.make_race(track, n, N, 6.0, n >= 4, 3000, 2000)
    if name == "open_end":
        for j in range(n):
            nd = track.nodes[track.n - 60 + 12 * j]
            race.x[j] = [nd[0], nd[1], 0.0, 40.0, 0.0, 0.0]
            race.s_abs[j] = nd[7]
    race.u_nom[:, :, 0] = 1.0
    if name == "nan_nominal":
        race.u_nom[1, 7, 0] = np.nan
    elif name == "inf_nominal":
        race.u_nom[1, 5, 1] = np.inf
    return track, race, params


@pytest.mark.parametrize("name", ["plain", "fine_nodes", "two_moves", "one_move", "open_end", "nan_nominal",
                                  "inf_nominal", "proposal", "vehicles1", "vehicles2", "vehicles4", "vehicles5",
                                  "vehicles6", "vehicles7", "vehicles10", "kinematic1", "kinematic3",
                                  "kinematic6"])
def test_throughput_variant_matches_small_launch_variant(planner, name):
    import torch
    track, race, params = _case(name)
    agent = min(1, race.n_agents - 1)
    got = {}
    for K in (K_SMALL, K_LARGE):
        rt = PY.build(planner, track, race, params, K)
        if name == "proposal":
            g = torch.Generator().manual_seed(3)
            q = torch.rand((race.n_agents, params["N"], 4), generator=g) * torch.tensor([2.0, 0.2, 1.0, 0.05])
            rt.prop, rt.K_prop = q.cuda().contiguous(), 777
        print(f"case {name} K {K}", flush=True)
        got[K] = PY.gpu_rollout(planner, params, rt, agent, 1, want_noise=True)
    for nm in OUT:
        a, b = got[K_SMALL][nm], got[K_LARGE][nm][:K_SMALL]
        assert np.array_equal(np.ascontiguousarray(a).view(np.uint8), np.ascontiguousarray(b).view(np.uint8)), nm
    flags = got[K_SMALL]["flags"]
    if name in ("one_move", "open_end"):
        assert np.any(flags & 8)  # the limit was met
    if name == "nan_nominal":
        assert np.all(flags & 16)
    assert planner.status() == 0
