"""Timed workloads of the planner and of its proposal network.

listed() names the workloads, draw() gives more of the same ranges, prepare() makes the
inputs and the handles that a program keeps (planner context, tracks, plan, network,
trainer), run() is one pass through the public entry points, work() the bytes and FLOPs
that a pass cannot do without, exact() the results in float64 written without this
package's planner or network.

Kinds
  plan      closed-loop planning steps of a set of races through a plan object (the graph
            replay a racing program runs at every control interval)
  call      the same through the direct calls plan_step() and advance(), no plan kept
  response  one best response with its per-sample outputs (inspection, parity checks)
  forward   the proposal network on a batch of feature rows
  train     Adam steps of the proposal network on sampled minibatches, then its weights
  gemm      the network's BF16 matrix product on its own
"""

from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2607_25388_amd import inputs, learned
from paper_2607_25388_amd import race_eval
from paper_2607_25388_amd import sgtp as sg


def listed():
    return [
        # one game of the paper's own setup (3 kinematic cars, K = 128, H = 12, 2 sweeps): the
        # smallest planning call, launch and latency bound
        dict(name="race_paper", kind="plan", scale="small", races=1, vehicles=3, K=128, N=12, L=2, discs=1,
             update=0, persistent=0, spl=1, prop=0.0),
        # a two-car race on the short track, planned by direct calls without a plan object
        dict(name="race_call", kind="call", scale="full", races=1, vehicles=2, K=1024, N=20, L=3, discs=1,
             update=0, persistent=0, spl=1, prop=0.0),
        # the mid-scale race: 3 vehicles, latency of one on-line planner
        dict(name="race_mid", kind="plan", scale="full", races=1, vehicles=3, K=16384, N=40, L=5, discs=3,
             update=0, persistent=0, spl=1, prop=0.0),
        # the large field: 10 vehicles on a staggered grid at full K
        dict(name="field_large", kind="plan", scale="full", races=1, vehicles=10, K=65536, N=50, L=5, discs=3,
             update=0, persistent=0, spl=1, prop=0.0),
        # the batched workload: 256 uneven races (2-10 vehicles, K 4096-65536, N 20/40/50)
        dict(name="batch_256", kind="plan", scale="mixed", races=256, vehicles=0, K=0, N=50, L=5, discs=3,
             update=0, persistent=0, spl=2, prop=0.0),
        # closed-loop evaluation at the paper's scale: every vehicle of 42 trials plans its own
        # game (default plan options, as race_eval runs it)
        dict(name="eval_small", kind="plan", scale="small", races=126, vehicles=3, K=128, N=12, L=2, discs=1,
             update=0, persistent=1, spl=1, prop=0.0),
        # the path-integral ablation in the full-size evaluation
        dict(name="eval_mppi", kind="plan", scale="full", races=126, vehicles=3, K=4096, N=40, L=5, discs=3,
             update=1, persistent=1, spl=1, prop=0.0),
        # 32 races planned with the learned proposal inside the step (K/4 samples, 7/8 proposed)
        dict(name="learned_32", kind="plan", scale="full", races=32, vehicles=0, K=4096, N=50, L=5, discs=3,
             update=0, persistent=0, spl=1, prop=0.875),
        # one best response with every per-sample output, ragged K and odd horizon
        dict(name="response", kind="response", scale="full", vehicles=4, K=5000, N=33, discs=3, noise=False),
        # the network over a data set's features
        dict(name="forward_65536", kind="forward", rows=65536),
        # the training loop at the batch the proposal is trained with
        dict(name="train_4096", kind="train", batch=4096, M=200000, N=50, steps=32),
        # the network's product at a size where the matrix cores count
        dict(name="gemm_16384", kind="gemm", M=16384, N=1024, K=1024, ta=False, tb=False, bias=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: sizes over their logarithm, odd ones among them."""
    kind = rng.choice(["plan", "plan", "plan", "plan", "call", "response", "forward", "train", "gemm"])
    if kind in ("plan", "call"):
        scale = rng.choice(["small", "full", "full"])
        N = rng.randint(8, 20) if scale == "small" else rng.randint(18, 50)
        vehicles = rng.randint(2, 4) if scale == "small" else rng.randint(2, 10)
        races = 1 if kind == "call" or rng.random() < 0.5 else _log(rng, 2, 126)
        K = _log(rng, 64, 4096) if scale == "small" else _log(rng, 512, 65536)
        cap = 150e6 if races == 1 else 600e6  # sample-steps of a sweep
        K = max(64, min(K, int(cap / (races * vehicles * N))))
        update = 1 if rng.random() < 0.2 else 0
        prop = 0.0 if update or rng.random() < 0.7 else round(rng.uniform(0.3, 1.0), 3)
        return dict(kind=kind, scale=scale, races=races, vehicles=vehicles, K=K, N=N, L=rng.randint(1, 5),
                    discs=1 if scale == "small" else rng.choice([1, 3]), update=update,
                    persistent=rng.choice([0, 1]) if kind == "plan" else 0,
                    spl=rng.choice([1, 1, 2]) if kind == "plan" else 1, prop=prop if kind == "plan" else 0.0)
    if kind == "response":
        return dict(kind=kind, scale="full", vehicles=rng.randint(1, 8), K=_log(rng, 100, 65536),
                    N=rng.randint(15, 50), discs=rng.choice([1, 3]), noise=rng.random() < 0.3)
    if kind == "forward":
        return dict(kind=kind, rows=_log(rng, 3, 65536))
    if kind == "train":
        return dict(kind=kind, batch=_log(rng, 256, 16384), M=_log(rng, 20000, 400000), N=rng.randint(20, 50),
                    steps=rng.randint(8, 32))
    return dict(kind="gemm", M=_log(rng, 64, 65536), N=_log(rng, 64, 1024), K=_log(rng, 48, 1024),
                ta=rng.random() < 0.3, tb=rng.random() < 0.3, bias=rng.random() < 0.5)


# ---- inputs -------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _track(scale, N):
    """The raceline a program has loaded: the batched workload's track for the horizon, or
    one of the evaluation's small-scale loops."""
    if scale == "small":
        sc = race_eval.SCALES["small"]
        return inputs.make_fourier_track(sc["length"], sc["width"], 1106, **sc["track"])
    key = 20 if N <= 30 else 40 if N <= 45 else 50
    length, width = inputs.TRACK_FOR_N[key]
    return inputs.make_fourier_track(length, width, 1000 + key)


def _params(case):
    if case["scale"] == "small":
        p = inputs.small_scale_params(case["N"])
    else:
        p = inputs.default_params(case["N"], case["discs"])
    p["update"] = case.get("update", 0)
    return p


def _specs(case):
    """(track, vehicles, K, N) of every race."""
    if case["scale"] == "mixed":
        return [(_track("full", s["N"]), s["n_agents"], s["K"], s["N"])
                for s in inputs.batched_races(case["races"])]
    out = []
    for r in range(case["races"]):
        n = case["vehicles"] or 2 + r % 4
        out.append((_track(case["scale"], case["N"]), n, case["K"], case["N"]))
    return out


def _races(case, seed):
    """Races of the case whose tensors are slices of one buffer per field."""
    specs, small = _specs(case), case["scale"] == "small"
    rng = np.random.default_rng(seed)
    made, tracks = [], []
    for r, (tr, n, K, N) in enumerate(specs):
        if not any(tr is t for t in tracks):
            tracks.append(tr)
        made.append(inputs.make_race(tr, n, N, 2.0 if small else (8.0 if n >= 5 else 10.0), n >= 5,
                                     int(rng.integers(1 << 31)), int(rng.integers(1 << 31))))
    nt = sum(s[1] for s in specs)
    cells = [s[1] * s[3] for s in specs]
    rows = [s[1] * (s[3] + 1) for s in specs]
    buf = dict(x=torch.tensor(np.concatenate([m.x for m in made]), device="cuda"),
               s_abs=torch.tensor(np.concatenate([m.s_abs for m in made]), device="cuda"),
               v_scale=torch.tensor(np.concatenate([m.v_scale for m in made]), dtype=torch.float32, device="cuda"),
               u_nom=torch.zeros((sum(cells), 2), dtype=torch.float32, device="cuda"),
               traj=torch.zeros((sum(rows), 8), dtype=torch.float64, device="cuda"),
               prop=torch.zeros((sum(cells), 4), dtype=torch.float32, device="cuda"))
    races, a, c, t = [], 0, 0, 0
    for (tr, n, K, N), m, nc, nr in zip(specs, made, cells, rows):
        prop = buf["prop"][c:c + nc].view(n, N, 4) if case.get("prop", 0.0) > 0.0 else None
        tid = next(i for i, t in enumerate(tracks) if t is tr)
        races.append(sg.RaceTensors(n, m.ego, tid, N, inputs.n_tail_from_fraction(0.3, N), K,
                                    int(m.seed), 0, buf["x"][a:a + n], buf["s_abs"][a:a + n],
                                    buf["v_scale"][a:a + n], buf["u_nom"][c:c + nc].view(n, N, 2),
                                    buf["traj"][t:t + nr].view(n, N + 1, 8), prop,
                                    int(case.get("prop", 0.0) * K)))
        a, c, t = a + n, c + nc, t + nr
    return races, tracks, buf, nt


def _features(rows, gen):
    """Feature rows with the layout and ranges of sgtp_features."""
    X = torch.randn((rows, 50), generator=gen, device="cuda")
    X[:, :6] *= torch.tensor([0.4, 0.1, 0.2, 0.1, 0.2, 0.4], device="cuda")
    X[:, 2] += 0.8
    for m in range(4):
        here = torch.rand((rows, 1), generator=gen, device="cuda") < 0.9 - 0.2 * m
        f = X[:, 6 + 6 * m:12 + 6 * m]
        f *= torch.tensor([0.8, 0.5, 0.1, 0.3, 0.1, 0.0], device="cuda")
        f[:, 5] = 1.0
        f *= here
    X[:, 30:] *= 0.3
    return X


def prepare(case, seed):
    kind = case["kind"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if kind in ("plan", "call"):
        params = _params(case)
        races, tracks, buf, nt = _races(case, seed)
        planner = sg.Planner(max_agents_total=nt, max_races=len(races), max_K=max(r.K for r in races))
        for i, tr in enumerate(tracks):
            planner.upload_track(i, tr)
        if case["update"] == 1:
            planner.enable_path_integral()
        state = dict(case=case, params=params, races=races, buf=buf, planner=planner)
        if kind == "plan":
            opts = sg.plan_options(persistent=case["persistent"], samples_per_lane=case["spl"], include_advance=1)
            state["plan"] = planner.plan(params, races, case["L"], opts, trace=False)
            if case["prop"] > 0.0:
                state["mlp"] = sg.Mlp(nt, seed=int(seed) % 1000)
                state["plan"].set_proposal(state["mlp"])
        return state
    if kind == "response":
        one = dict(case, races=1)
        races, tracks, buf, nt = _races(one, seed)
        r, tr = races[0], tracks[0]
        # a nominal that follows the raceline, as a running planner's warm start does
        i = np.floor(np.mod(r.s_abs.cpu().numpy(), tr.length) / tr.ds).astype(int)
        v = r.x[:, 3].cpu().numpy()
        u = np.zeros((r.n_agents, r.N, 2), np.float32)
        for t in range(r.N):
            k = (i + np.round(v * 0.05 * t / tr.ds).astype(int)) % tr.n
            u[:, t, 1] = np.arctan(2.6 * tr.nodes[k, 3])
        r.u_nom.copy_(torch.tensor(u))
        planner = sg.Planner(max_agents_total=nt, max_races=1, max_K=r.K)
        planner.upload_track(0, tr)
        return dict(case=case, params=_params(case), race=r, planner=planner, track=tr)
    if kind == "forward":
        mlp = sg.Mlp(case["rows"], seed=int(seed) % 1000)
        return dict(case=case, mlp=mlp, X=_features(case["rows"], gen))
    if kind == "train":
        params = inputs.default_params(case["N"], 3)
        X = _features(case["M"], gen)
        W = torch.randn((50, 2 * case["N"]), generator=gen, device="cuda") * 0.3
        U = (torch.tanh(X @ W) + 0.3 * torch.randn((case["M"], 2 * case["N"]), generator=gen, device="cuda"))
        U = U.view(case["M"], case["N"], 2) * torch.tensor([3.0, 0.15], device="cuda")
        mlp = sg.Mlp(case["batch"], seed=int(seed) % 1000)
        data = learned.Dataset(X, U.contiguous(), None, None)
        tr = learned.Trainer(mlp, data, params, batch=case["batch"], lr=1e-3, seed=int(seed))
        return dict(case=case, mlp=mlp, data=data, trainer=tr, params=params, seed=int(seed))
    M, N, K = case["M"], case["N"], case["K"]
    A = (torch.randn((K, M) if case["ta"] else (M, K), generator=gen, device="cuda")).to(torch.bfloat16)
    B = (torch.randn((N, K) if case["tb"] else (K, N), generator=gen, device="cuda")).to(torch.bfloat16)
    bias = torch.randn(N, generator=gen, device="cuda") if case["bias"] else None
    return dict(case=case, A=A, B=B, bias=bias)


# ---- one pass -----------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "plan":
        u = state["plan"].run()
        b = state["buf"]
        return dict(u=u, x=b["x"], s=b["s_abs"], u_nom=b["u_nom"], traj=b["traj"])
    if kind == "call":
        b, p = state["buf"], state["planner"]
        u = p.plan_step(state["params"], state["races"], case["L"])
        p.advance(state["params"], state["races"], u)
        for r in state["races"]:
            r.plan_step += 1
        return dict(u=u, x=b["x"], s=b["s_abs"], u_nom=b["u_nom"], traj=b["traj"])
    if kind == "response":
        out = state["planner"].rollout_cost(state["params"], state["race"], 0, 1, want_noise=case["noise"])
        return {k: v for k, v in out.items() if v is not None}
    if kind == "forward":
        return state["mlp"].forward(state["X"])
    if kind == "train":
        for _ in range(case["steps"]):
            loss = state["trainer"].step()
        return dict(loss=loss, weights=state["mlp"].get_params())
    M, N, K = case["M"], case["N"], case["K"]
    return sg.gemm_bf16(state["A"], (1, M) if case["ta"] else (K, 1), state["B"], (1, K) if case["tb"] else (N, 1),
                        M, N, K, bias=state["bias"])


# ---- what a pass cannot do without ----------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("plan", "call", "response"):
        # FLOPs of a sample and step: rollout, projection and tracking cost, and the disc pairs
        # of every opponent
        base = 460.0 if case["scale"] != "small" else 260.0
        flops = nbytes = 0.0
        sweeps = 1.0 if kind == "response" else None
        specs = _specs(dict(case, races=1)) if kind == "response" else _specs(case)
        for tr, n, K, N in specs:
            per = base + 7.0 * case["discs"] ** 2 * (n - 1)
            vehicles = 1.0 if sweeps else (case["L"] + 1.0) * n + 1.0
            flops += vehicles * K * N * per
            nbytes += n * (48 + 8 + 4 + 8 * N * 2) + (0 if kind == "response" else n * (48 + 8 + 64 * (N + 1)))
            if kind == "response":
                nbytes += K * (4 + 1 + 4 + 48 + (8 * N if case["noise"] else 0))
        return dict(bytes=nbytes, flops=flops)
    params = 50 * 256 + 256 + 256 * 256 + 256 + 256 * 200 + 200
    if kind == "forward":
        return dict(bytes=4.0 * (case["rows"] * 250 + params),
                    flops=2.0 * case["rows"] * (50 * 256 + 256 * 256 + 256 * 200))
    if kind == "train":
        s, B = case["steps"], case["batch"]
        return dict(bytes=4.0 * s * (B * (50 + 2 * case["N"]) + 6 * params),
                    flops=float(s) * B * learned.TRAIN_FLOP_PER_ROW)
    M, N, K = case["M"], case["N"], case["K"]
    return dict(bytes=2.0 * (M * K + K * N) + 4.0 * M * N, flops=2.0 * M * N * K)


# ---- results in float64 ---------------------------------------------------------------

def _philox(c, key):
    """Philox4x32-10 on int64 tensors holding 32-bit words; c: four tensors."""
    m32 = 0xFFFFFFFF

    def mul(a, b):  # 32 x 32 -> (high, low)
        lo = (b & 0xFFFF) * a
        hi = (b >> 16) * a
        t = hi + (lo >> 16)
        return t >> 16, ((t & 0xFFFF) << 16) | (lo & 0xFFFF)

    k0, k1 = key & m32, (key >> 32) & m32
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c


def _net(P, X):
    """Outputs of the network with packed parameters P (float64 leaves) on X."""
    o, parts = 0, []
    for i, j in ((50, 256), (256, 256), (256, 200)):
        parts.append((P[o:o + i * j].view(i, j), P[o + i * j:o + i * j + j]))
        o += i * j + j
    h = X
    for n, (W, b) in enumerate(parts):
        h = h @ W + b
        if n < 2:
            h = 0.5 * h * (1.0 + torch.tanh(0.7978845608 * (h + 0.044715 * h ** 3)))
    return h


def _exact_train(st):
    case, M, B, N = st["case"], st["case"]["M"], st["case"]["batch"], st["case"]["N"]
    P = torch.tensor(sg.mlp_init(st["seed"] % 1000), dtype=torch.float64, device="cuda")
    m, v = torch.zeros_like(P), torch.zeros_like(P)
    sig = torch.tensor([st["params"]["sigma_a"], st["params"]["sigma_d"]], dtype=torch.float64, device="cuda")
    row = torch.arange(min(B, M), device="cuda")
    loss = None
    for t in range(case["steps"]):
        zero = torch.zeros_like(row)
        r = _philox([row, zero + t, zero, zero], st["seed"])[0]
        i = ((r >> 16) * M + (((r & 0xFFFF) * M) >> 16)) >> 16
        X, U = st["data"].X[i].double(), st["data"].U[i].double()
        Pg = P.clone().requires_grad_(True)
        o = _net(Pg, X).view(-1, 50, 4)[:, :N]
        mu = o[..., :2] * torch.tensor([4.0, 0.2], dtype=torch.float64, device="cuda")
        ls = torch.log(sig) + torch.clamp(o[..., 2:], -4.0, 1.0)
        loss = (0.5 * ((U - mu) * torch.exp(-ls)) ** 2 + ls).sum() / U.shape[0]
        g, = torch.autograd.grad(loss, Pg)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        P = P - 1e-3 * (m / (1 - 0.9 ** (t + 1))) / (torch.sqrt(v / (1 - 0.999 ** (t + 1))) + 1e-8)
    return dict(loss=loss.detach().view(1), weights=P)


class _Line:
    """A closed raceline in float64: normal-interpolated polyline and its Frenet frame."""

    def __init__(self, tr):
        self.n, self.length, self.psi_lap = tr.n, tr.length, tr.psi_lap
        nd = torch.tensor(tr.nodes, dtype=torch.float64, device="cuda")
        self.x, self.y, self.psi, self.s = nd[:, 0], nd[:, 1], nd[:, 2], nd[:, 7]
        self.wl, self.wr, self.v = nd[:, 4], nd[:, 5], nd[:, 6]
        self.nx, self.ny = -torch.sin(self.psi), torch.cos(self.psi)

    def at(self, col, i):
        lap = torch.div(i, self.n, rounding_mode="floor")
        val = col[i - lap * self.n]
        if col is self.s:
            val = val + lap * self.length
        elif col is self.psi:
            val = val + lap * self.psi_lap
        return val

    def ahead(self, i, X, Y):
        return (X - self.at(self.x, i)) * self.at(self.ny, i) - (Y - self.at(self.y, i)) * self.at(self.nx, i)

    def foot(self, i, X, Y):
        g = lambda c: (self.at(c, i), self.at(c, i + 1))  # noqa: E731
        (ax, bx), (ay, by), (anx, bnx), (any_, bny) = g(self.x), g(self.y), g(self.nx), g(self.ny)
        rx, ry, dx, dy, dnx, dny = X - ax, Y - ay, bx - ax, by - ay, bnx - anx, bny - any_
        C = rx * any_ - ry * anx
        Bq = (rx * dny - ry * dnx) - (dx * any_ - dy * anx)
        A = -(dx * dny - dy * dnx)
        den = -Bq - torch.copysign(torch.sqrt(torch.clamp(Bq * Bq - 4 * A * C, min=0.0)), Bq)
        t = torch.clamp(torch.where(den != 0, 2 * C / den, torch.zeros_like(C)), 0.0, 1.0)
        nx, ny = anx + t * dnx, any_ + t * dny
        d = ((X - ax - t * dx) * nx + (Y - ay - t * dy) * ny) / torch.sqrt(nx * nx + ny * ny)
        mix = lambda c: g(c)[0] + t * (g(c)[1] - g(c)[0])  # noqa: E731
        return mix(self.s), d, mix(self.wl), mix(self.wr)

    def find(self, X, Y):  # one point: the enclosing segment of smallest |d|
        i = torch.arange(self.n, device="cuda")
        inside = (self.ahead(i, X, Y) >= 0) & (self.ahead(i + 1, X, Y) <= 0)
        d = torch.where(inside, self.foot(i, X, Y)[1].abs(), torch.full_like(X + self.x, math.inf))
        return int(torch.argmin(d))

    def walk(self, i, X, Y):
        for _ in range(16):
            i = i + (self.ahead(i + 1, X, Y) > 0).long()
        for _ in range(16):
            i = i - (self.ahead(i, X, Y) < 0).long()
        return i

    def sample(self, s):  # node values at arc length s (0-d tensors)
        i = torch.floor(s / (self.length / self.n)).long()
        t = (s - self.at(self.s, i)) / (self.at(self.s, i + 1) - self.at(self.s, i))
        return [self.at(c, i) + t * (self.at(c, i + 1) - self.at(c, i)) for c in (self.x, self.y, self.psi, self.v)]


def _rollout(p, x0, u):
    """States [N + 1][6][..] of the dynamic single-track model under controls u [N][2][..]."""
    L = p["lf"] + p["lr"]
    Ff, Fr = p["mu"] * p["m"] * p["g"] * p["lr"] / L, p["mu"] * p["m"] * p["g"] * p["lf"] / L

    def f(s, a, de):
        psi, vy, om = s[2], s[4], s[5]
        vx = torch.clamp(s[3], min=0.0)
        vh = torch.clamp(vx, min=p["v_eps"])
        af = de - torch.atan((vy + p["lf"] * om) / vh)
        ar = -torch.atan((vy - p["lr"] * om) / vh)
        Fyf = Ff * torch.sin(p["C"] * torch.atan(p["B"] * af))
        Fyr = Fr * torch.sin(p["C"] * torch.atan(p["B"] * ar))
        return torch.stack([vx * torch.cos(psi) - vy * torch.sin(psi), vx * torch.sin(psi) + vy * torch.cos(psi), om,
                            a - Fyf * torch.sin(de) / p["m"] + vy * om,
                            (Fyr + Fyf * torch.cos(de)) / p["m"] - vx * om,
                            (p["lf"] * Fyf * torch.cos(de) - p["lr"] * Fyr) / p["Iz"]])

    s, out, h = x0, [x0], p["dt"]
    for a, de in u:
        k1 = f(s, a, de)
        k2 = f(s + 0.5 * h * k1, a, de)
        k3 = f(s + 0.5 * h * k2, a, de)
        k4 = f(s + h * k3, a, de)
        s = s + h / 6 * (k1 + 2 * k2 + 2 * k3 + k4)
        s = torch.cat([s[:3], torch.clamp(s[3:4], min=0.0), s[4:]])
        out.append(s)
    return out


def _exact_response(st):
    p, r, line, K, N = st["params"], st["race"], _Line(st["track"]), st["race"].K, st["race"].N
    x, un = r.x.clone(), r.u_nom.double()
    lo, hi = (torch.tensor([p[a], p[b]], device="cuda", dtype=torch.float64).view(2, 1)
              for a, b in (("a_min", "d_min"), ("a_max", "d_max")))
    n, offs = r.n_agents, p["disc_off"][:p["n_disc"]]
    seg, s0 = [], []
    for j in range(n):
        i = line.find(x[j, 0], x[j, 1])
        s = line.foot(torch.tensor([i], device="cuda"), x[j, 0], x[j, 1])[0]
        lap = int(torch.round((r.s_abs[j] - s) / line.length))
        seg.append(i + lap * line.n)
        s0.append(s + lap * line.length)

    def track(j, states, i):  # s, d, clearance rows of every state after the first
        out = []
        for s in states[1:]:
            i = line.walk(i, s[0], s[1])
            out.append(line.foot(i, s[0], s[1]))
        return out

    def clip(j, z):
        sig = torch.tensor([p["sigma_a"], p["sigma_d"]], device="cuda", dtype=torch.float64).view(2, 1)
        return [torch.maximum(torch.minimum(un[j, t].view(2, 1) + sig * z[t], hi), lo) for t in range(N)]

    def start(j, k):
        return x[j].view(6, 1).expand(6, k)

    # the samples' Gaussian pairs: one Philox call for two steps
    k = torch.arange(K, device="cuda")
    z = []
    for t in range(N):
        if t % 2 == 0:
            w = _philox([k, torch.zeros_like(k) + t // 2, torch.zeros_like(k) + (1 << 16),
                         torch.zeros_like(k) + r.plan_step], r.seed)
        a, b = w[2 * (t % 2)], w[2 * (t % 2) + 1]
        u1, u2 = (2 * (a >> 9) + 1).double() * 2.0 ** -24, (b >> 8).double() * 2.0 ** -24
        rho = torch.sqrt(-2 * torch.log(u1))
        z.append(torch.stack([rho * torch.cos(2 * math.pi * u2), rho * torch.sin(2 * math.pi * u2)]))
    u = clip(0, z)
    X = _rollout(p, start(0, K), u)
    F = track(0, X, torch.full((K,), seg[0], device="cuda"))
    cost, sr, bd = torch.zeros(K, dtype=torch.float64, device="cuda"), s0[0][0], None
    lam = float(r.v_scale[0])
    for t in range(N):
        sr = sr + p["dt"] * lam * line.sample(sr)[3]
        xr, yr, pr, vr = line.sample(sr)
        e = X[t + 1]
        ep = e[2] - pr
        ep = ep - 2 * math.pi * torch.round(ep / (2 * math.pi))
        Q, R, S = p["Q"], p["R"], p["S"]
        cost += Q[0] * (e[0] - xr) ** 2 + Q[1] * (e[1] - yr) ** 2 + Q[2] * ep ** 2 + Q[3] * (e[3] - lam * vr) ** 2
        cost += R[0] * u[t][0] ** 2 + R[1] * u[t][1] ** 2
        if t:
            cost += S[0] * (u[t][0] - u[t - 1][0]) ** 2 + S[1] * (u[t][1] - u[t - 1][1]) ** 2
        _, d, wl, wr = F[t]
        b = torch.minimum(wr + d, wl - d)
        bd = b if bd is None else torch.minimum(bd, b)
    tail = lambda f: sum(g[1] for g in f[N - r.n_tail:]) / r.n_tail  # noqa: E731
    cap = max(p["g_safe"], p["d_col"])
    obs = torch.full_like(cost, math.inf)
    for j in range(1, n):
        Y = _rollout(p, start(j, 1), clip(j, torch.zeros((N, 2, 1), dtype=torch.float64, device="cuda")))
        G = track(j, Y, torch.tensor([seg[j]], device="cuda"))
        g = torch.full_like(cost, cap)
        for t in range(1, N + 1):
            for a in offs:
                for b in offs:
                    qx = X[t][0] + a * torch.cos(X[t][2]) - Y[t][0] - b * torch.cos(Y[t][2])
                    qy = X[t][1] + a * torch.sin(X[t][2]) - Y[t][1] - b * torch.sin(Y[t][2])
                    g = torch.minimum(g, torch.sqrt(qx * qx + qy * qy))
        ds0, dsN = s0[0] - s0[j], F[-1][0] - G[-1][0]
        alpha = 1 / (1 + ds0.abs() / (p["s_contest"] + p["eps_alpha"]))
        block = p["w_block"] if p["s_role"] < float(ds0) < p["s_contest"] else 0.0
        game = -p["w_contest"] * (dsN.abs() < p["s_contest"]) - p["w_long"] * alpha * dsN
        game = game - block / (1 + (tail(F) - tail(G)).abs())
        cost += p["w_game"] * (game + p["w_safety"] * torch.clamp(p["g_safe"] - g, min=0.0) ** 2)
        obs = torch.minimum(obs, g)
    viol = torch.clamp(p["m_bd"] - bd, min=0.0) + torch.clamp(p["d_col"] - obs, min=0.0)
    out = dict(cost=cost, flags=None, viol=viol, x_final=X[-1].T.contiguous(), choice=None)
    if st["case"]["noise"]:
        out["noise"] = torch.stack(z).permute(2, 0, 1).contiguous()
    return out


def exact(case, seed):
    """Float64 results.  A planning step has none: it adopts the argmin over samples whose
    costs lie closer together than float32 tells apart, and every later number follows it."""
    if case["kind"] in ("plan", "call"):
        return None
    st = prepare(case, seed)
    if case["kind"] == "response":
        return _exact_response(st)
    if case["kind"] == "forward":
        P = torch.tensor(sg.mlp_init(int(seed) % 1000), dtype=torch.float64, device="cuda")
        return _net(P, st["X"].double())
    if case["kind"] == "train":
        return _exact_train(st)
    A, B = st["A"].double(), st["B"].double()
    C = (A.T if case["ta"] else A).contiguous() @ (B.T if case["tb"] else B).contiguous()
    return C if st["bias"] is None else C + st["bias"].double()
