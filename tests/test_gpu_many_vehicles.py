"""Direct planning calls over more vehicles than a small copy of their descriptors holds (16 KB, about
150 vehicles): the same bits as a plan of the same races, call after call with other races in
between (the ring of descriptor images)."""

import pytest

from paper_2607_25388_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,n", [(1, 2), (40, 3), (45, 3), (24, 16)])
def test_direct_calls_match_plans(R, n):
    import torch
    import paper_2607_25388_amd.sgtp as sg
    K, N = 70, 9
    track = inputs.make_fourier_track(300.0, 10.0, 1000)
    params = inputs.default_params(N, 1)
    planner = sg.Planner(max_agents_total=R * n, max_races=R, max_K=1024)
    try:
        planner.upload_track(0, track)

        def races(seed):
            return [sg.race_from_inputs(inputs.make_race(track, n, N, 6.0, n >= 4, seed + r, 2000 + r), 0, K, N,
                                        params["n_tail"]) for r in range(R)]
        print(f"case {R} {n}", flush=True)
        for seed in range(3000, 3010):  # more calls than the ring has images
            a, b = races(seed), races(seed)
            u = planner.plan_step(params, a, 1)
            plan = planner.plan(params, b, 1, sg.plan_options(persistent=0, use_graph=0), trace=False)
            v = plan.run()
            torch.cuda.synchronize()
            assert torch.equal(u.view(torch.int32), v.view(torch.int32))
            for x, y in zip(a, b):
                assert torch.equal(x.u_nom.view(torch.int32), y.u_nom.view(torch.int32))
            plan.close()
        # one after the other without a wait between
        many = [races(seed) for seed in range(4000, 4012)]
        us = [planner.plan_step(params, r, 0).clone() for r in many]
        torch.cuda.synchronize()
        for seed, u in zip(range(4000, 4012), us):
            w = planner.plan_step(params, races(seed), 0)
            torch.cuda.synchronize()
            assert torch.equal(u.view(torch.int32), w.view(torch.int32))
    finally:
        planner.close()
