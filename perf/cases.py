"""The work that a user has this framework do, as cases for timing and comparison.

Every kind below goes through the public entry points of paper_2101_01160_amd:

  md           LJSystem.step and .state: Lennard-Jones MD of one system or of a
               batch of replicas, with the fused coarse-graining attached
               (s_cg > 0) or without it, then the state read out
  cg_pair      mdlg_coarse_grain: one coarse-graining event of two snapshots
  cg_series    mdlg_coarse_grain_series: all pairs of a stored trajectory at
               several coarse-graining times and lattice drifts
  neq          mdlg_neq_mdlg: ensemble occupations and collision operator
  vacf         mdlg_vacf: velocity autocorrelation sums
  hist         mdlg_displacement_hist: displacement histograms
  mlp_forward  SurrogateMLP.forward: the equilibrium of B parameter points
  mlp_train    SurrogateMLP.train_step: Adam steps, then the parameters read

Sizes are those of the benchmark's workloads and of the tests.
"""
import math

import numpy as np
import torch

import paper_2101_01160_amd as m

RC, SKIN, DT = 2.5, 0.5, 1e-4
LAGS = (1, 2, 3, 4, 6, 8, 10, 13, 16, 20)  # coarse-graining times of the surrogate data, in snapshots
MLP_DIMS = (6, 256, 256, 256, 49)


def _md(name, n, n_rep, phi, kT, lx, s_cg, steps, n_min=0, force_bits=64, cell_acc=False, shear=0.0):
    """n: particles of a replica (of the largest one, where n_min > 0: sizes then run from n_min to n)."""
    return {"name": name, "kind": "md", "n": n, "n_min": n_min, "n_rep": n_rep, "phi": phi, "kT": kT, "lx": lx,
            "s_cg": s_cg, "steps": steps, "force_bits": force_bits, "cell_acc": cell_acc, "shear": shear}


def listed():
    return [
        # the system that the smoke run and most tests step: 512 particles, latency and launches only
        _md("md_512", 512, 1, 0.0784, 20.0, 32, 50, 400),
        # the benchmark's default workload, eight coarse steps and the state
        _md("md_1m", 1 << 20, 1, 0.0784, 20.0, 1024, 50, 400),
        # the precision workload: 2^22 particles with FP32 pair forces
        _md("md_4m_fp32", 1 << 22, 1, 0.0784, 20.0, 2048, 50, 100, force_bits=32),
        # the non-equilibrium workload's MD: an ensemble of 256 small boxes started as a shear wave, between
        # two stored snapshots (an uneven number of steps, no fused coarse-graining)
        _md("md_neq_256x998", 998, 256, 0.0784, 20.0, 25, 0, 391, shear=4.0),
        # dense replicas of uneven size, as the batched workload and the surrogate's training data have them
        _md("md_dense_batch", 131072, 24, 0.4, 5.0, 0, 50, 100, n_min=4096),
        # one event of two stored snapshots of the benchmark's system
        {"name": "cg_pair_1m", "kind": "cg_pair", "n": 1 << 20, "phi": 0.0784, "lx": 1024, "img": True, "u": 0.0,
         "field": "none"},
        # the surrogate's training data: ten coarse-graining times x sixteen drifts over every snapshot pair
        {"name": "cg_series_8x65536", "kind": "cg_series", "n": 65536, "n_rep": 8, "n_snap": 201, "n_lag": 10,
         "n_u": 16, "moments": True},
        # the non-equilibrium workload's analysis: 100 coarse steps of 256 replicas on a 25 x 25 lattice
        {"name": "neq_256x998", "kind": "neq", "n": 998, "n_rep": 256, "lx": 25, "n_snap": 101, "xi": True},
        # the paper sweep's autocorrelation: four systems of 99,856 particles, 601 snapshots, 51 spread lags
        {"name": "vacf_4x99856", "kind": "vacf", "n": 99856, "n_rep": 4, "n_snap": 601, "n_lag": 51},
        # the paper sweep's displacement histograms, one row's stored snapshots
        {"name": "hist_4x99856", "kind": "hist", "n": 99856, "n_rep": 4, "n_snap": 9, "n_lag": 1, "n_bin": 96},
        # the surrogate evaluated over a large set of parameter points
        {"name": "mlp_forward_65536", "kind": "mlp_forward", "B": 65536},
        # the surrogate's training: ten Adam steps of 2048 samples
        {"name": "mlp_train_2048", "kind": "mlp_train", "B": 2048, "steps": 10},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("md", "md", "md", "md", "cg_pair", "cg_series", "neq", "vacf", "hist", "mlp_forward", "mlp_train"))
    if kind == "md":
        total = _log_int(rng, 512, 1 << 21)
        n_rep = min(rng.choice((1, 1, 4, _log_int(rng, 2, 256))), total // 512)
        n = total // n_rep
        phi, kT = round(rng.uniform(0.05, 0.4), 4), round(rng.uniform(1.0, 20.0), 3)
        return {"kind": "md", "n": n, "n_min": max(512, n // 8) if n_rep > 1 and rng.random() < 0.5 else 0,
                "n_rep": n_rep, "phi": phi, "kT": kT, "lx": 0, "s_cg": rng.choice((0, 10, 25, 50, 50, 200)),
                "steps": rng.randint(100, 400), "force_bits": rng.choice((64, 64, 32)),
                "cell_acc": rng.random() < 0.25, "shear": 0.0}
    if kind == "cg_pair":
        return {"kind": "cg_pair", "n": _log_int(rng, 512, 1 << 22), "phi": round(rng.uniform(0.05, 0.4), 4),
                "lx": _log_int(rng, 7, 2048), "img": rng.random() < 0.5, "u": rng.choice((0.0, 0.2)),
                "field": rng.choice(("none", "n_event", "cell_acc"))}
    if kind == "cg_series":
        n_lag = rng.randint(1, 10)
        return {"kind": "cg_series", "n": _log_int(rng, 500, 65536), "n_rep": rng.randint(1, 8),
                "n_snap": rng.randint(40, 201), "n_lag": n_lag, "n_u": rng.randint(1, 16),
                "moments": rng.random() < 0.75}
    if kind == "neq":
        lx = rng.randint(7, 64)
        return {"kind": "neq", "n": _log_int(rng, 250, 4000), "n_rep": _log_int(rng, 4, 256), "lx": lx,
                "n_snap": rng.randint(3, 101) if lx < 33 else rng.randint(3, 33), "xi": rng.random() < 0.75}
    if kind == "vacf":
        n_snap = rng.randint(20, 601)
        return {"kind": "vacf", "n": _log_int(rng, 500, 99856), "n_rep": rng.randint(1, 4), "n_snap": n_snap,
                "n_lag": rng.randint(2, min(51, n_snap // 4))}
    if kind == "hist":
        return {"kind": "hist", "n": _log_int(rng, 500, 99856), "n_rep": rng.randint(1, 4),
                "n_snap": rng.randint(5, 64), "n_lag": rng.randint(1, 4), "n_bin": rng.choice((24, 96, 97, 1000))}
    if kind == "mlp_forward":
        return {"kind": "mlp_forward", "B": _log_int(rng, 1, 65536)}
    return {"kind": "mlp_train", "B": _log_int(rng, 32, 4096), "steps": 10}


# ------------------------------------------------------------------ inputs ---

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)


def _box(n, phi):
    return math.sqrt(n * math.pi / (4.0 * phi))


def _sizes(case):
    """Particles of each replica."""
    n, n_min, n_rep = case["n"], case.get("n_min", 0), case["n_rep"]
    if not n_min:
        return [n] * n_rep
    # spread over the logarithm, large and small ones in turn
    return [int(round(n_min * (n / n_min) ** ((0.5 + r * 0.6180339887498949) % 1.0))) for r in range(n_rep)]


def _gas(g, n, phi, kT, shear=0.0):
    """Positions of a gas without overlaps and Maxwellian velocities: a square grid with each site moved freely
    inside its own square less the particles' core."""
    L = _box(n, phi)
    nx = math.ceil(math.sqrt(n))
    ny = math.ceil(n / nx)
    k = torch.arange(n, device="cuda")
    site = torch.stack([(k % nx + 0.5) * (L / nx), (k // nx + 0.5) * (L / ny)], dim=1)
    half = max(0.05, (min(L / nx, L / ny) - 0.96) / 2)
    pos = torch.remainder(site + half * (2.0 * _rand(g, n, 2) - 1.0), L)
    pos[pos >= L] = 0.0
    vel = math.sqrt(kT) * _randn(g, n, 2)
    vel -= vel.mean(dim=0, keepdim=True)
    vel *= torch.sqrt((n - 1) * kT / (0.5 * (vel * vel).sum()))
    if shear:
        vel[:, 0] += shear * torch.sin(2.0 * math.pi * pos[:, 1] / L)
    return pos, vel, L


def _md_inputs(case, seed):
    g = _gen(seed)
    parts = [_gas(g, n, case["phi"], case["kT"], case["shear"]) for n in _sizes(case)]
    return torch.cat([p for p, _, _ in parts]), torch.cat([v for _, v, _ in parts]), [L for _, _, L in parts]


def _lattices(case, boxes):
    return [case["lx"] or max(7, round(L / 2.0)) for L in boxes]


def _wrap(x, L):
    """Wrapped positions and image counts of unwrapped ones."""
    img = torch.floor(x / L)
    pos = x - img * L
    pos[pos < 0.0] = 0.0
    pos[pos >= L] = math.nextafter(L, 0.0)
    return pos, img.to(torch.int32)


def _walk(g, n, n_snap, L, v_std, step_std):
    """A stored trajectory [n_snap][n][2]: ballistic motion v_std per snapshot plus a random step."""
    x, v = L * _rand(g, n, 2), v_std * _randn(g, n, 2)
    pos = torch.empty((n_snap, n, 2), dtype=torch.float64, device="cuda")
    img = torch.empty((n_snap, n, 2), dtype=torch.int32, device="cuda")
    for p in range(n_snap):
        pos[p], img[p] = _wrap(x, L)
        x = x + v
        if step_std:
            x = x + step_std * _randn(g, n, 2)
    return pos, img


def _series_inputs(case, seed):
    """Replicas of the surrogate's parameter range: dx ~ 2, ten MD steps between snapshots."""
    g = _gen(seed)
    rng = np.random.default_rng(seed)
    n, n_rep, P = case["n"], case["n_rep"], case["n_snap"]
    box = [_box(n, phi) for phi in rng.uniform(0.05, 0.4, n_rep)]
    lx = [max(7, round(L / 2.0)) for L in box]
    parts = [_walk(g, n, P, L, 10 * DT * math.sqrt(kT), 0.1 * 10 * DT * math.sqrt(kT))
             for L, kT in zip(box, rng.uniform(1.0, 20.0, n_rep))]
    r, th = 0.2 * np.sqrt(rng.uniform(0, 1, case["n_u"])), rng.uniform(0, 2 * math.pi, case["n_u"])
    u = np.stack([r * np.cos(th), r * np.sin(th)], axis=1)
    u[0] = 0.0
    origin = np.mod(0.5 + np.arange(P)[:, None] * np.array([0.7548776662466927, 0.5698402909980532]), 1.0)
    return {"offsets": np.arange(n_rep + 1) * n, "box": box, "lx": lx, "u": u, "origin": origin,
            "pos": torch.cat([p for p, _ in parts], dim=1), "img": torch.cat([i for _, i in parts], dim=1),
            "lags": LAGS[:case["n_lag"]]}


def _vacf_lags(case):
    """Spread evenly over the logarithm up to three quarters of the trajectory, 0 among them."""
    top = 3 * case["n_snap"] // 4
    lags = [0]
    for k in range(1, case["n_lag"]):
        lags.append(max(lags[-1] + 1, int(round(top ** (k / (case["n_lag"] - 1))))))
    return [min(l, case["n_snap"] - 1) for l in lags]


def _vacf_inputs(case, seed):
    """Velocities at kT = 20 that forget themselves over 100 snapshots."""
    g = _gen(seed)
    n, P = case["n"] * case["n_rep"], case["n_snap"]
    vel = torch.empty((P, n, 2), dtype=torch.float64, device="cuda")
    a = math.exp(-0.01)
    vel[0] = math.sqrt(20.0) * _randn(g, n, 2)
    for p in range(1, P):
        vel[p] = a * vel[p - 1] + math.sqrt(20.0 * (1 - a * a)) * _randn(g, n, 2)
    return vel


def _mlp_params(seed):
    rng = np.random.default_rng(seed)
    parts = []
    for fi, fo in zip(MLP_DIMS[:-1], MLP_DIMS[1:]):
        a = math.sqrt(6.0 / (fi + fo))
        parts += [rng.uniform(-a, a, fi * fo), np.zeros(fo)]
    return np.concatenate(parts).astype(np.float32)


def _mlp_x(g, B):
    """(phi, kT, dt_cg / dx, |u|, cos, sin) over the surrogate's parameter box."""
    u = 0.2 * torch.sqrt(_rand(g, B))
    th = 2.0 * math.pi * _rand(g, B)
    dt = torch.exp(math.log(5e-4) + math.log(20.0) * _rand(g, B))
    cols = [0.05 + 0.35 * _rand(g, B), 1.0 + 19.0 * _rand(g, B), dt, u, torch.cos(th), torch.sin(th)]
    return torch.stack(cols, dim=1).to(torch.float32).contiguous()


def _mlp_target(g, x):
    """Equilibria shaped like the measured ones: a narrow Gaussian over the lattice velocities about the drift."""
    c = torch.from_numpy(m.mdlg_velocity_table().astype(np.float64)).cuda()
    u = (x[:, 3:4] * x[:, 4:6]).double()
    d2 = ((c[None] - u[:, None]) ** 2).sum(dim=2)
    return torch.softmax(-d2 / (2.0 * (0.08 + 0.12 * _rand(g, x.shape[0], 1))), dim=1).to(torch.float32).contiguous()


def _batches(case, seed):
    g = _gen(seed)
    out = []
    for _ in range(case["steps"]):
        x = _mlp_x(g, case["B"])
        out.append((x, _mlp_target(g, x)))
    return out


def _zeros(shape, dtype):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "md":
        pos, vel, boxes = _md_inputs(case, seed)
        params = [m.lj_params(n, L, dt=DT, rc=RC, force_bits=case["force_bits"]) for n, L in zip(_sizes(case), boxes)]
        s["sys"] = m.LJSystem(pos, vel, params=params)
        if case["s_cg"]:
            s["acc"] = s["sys"].attach_cg(_lattices(case, boxes), case["s_cg"], cell_acc=case["cell_acc"])
    elif kind == "cg_pair":
        g = _gen(seed)
        L = _box(case["n"], case["phi"])
        pos, img = _walk(g, case["n"], 2, L, 0.3 * L / case["lx"], 0.3 * L / case["lx"])
        lx = case["lx"]
        if not case["img"]:  # two snapshots in one box: the steps that wrap are beyond the lattice velocities
            img = [None, None]
        s.update(L=L, pos=[pos[0].contiguous(), pos[1].contiguous()], img=[i if i is None else i.contiguous() for i in img],
                 counts=_zeros((50,), torch.int64), moments=_zeros((5,), torch.float64),
                 field=None if case["field"] == "none" else _zeros((49, lx, lx), torch.int32))
    elif kind == "cg_series":
        s.update(_series_inputs(case, seed))
        s["counts"] = _zeros((case["n_rep"], case["n_lag"], case["n_u"], 50), torch.int64)
        s["moments"] = _zeros((case["n_rep"], case["n_lag"], 5), torch.float64) if case["moments"] else None
    elif kind == "neq":
        n, lx, P = case["n"] * case["n_rep"], case["lx"], case["n_snap"]
        s["L"] = 4.0 * lx
        s["pos"], s["img"] = _walk(_gen(seed), n, P, s["L"], 0.8, 1.4)
        s["f"], s["ovf"] = _zeros((P - 1, 49, lx, lx), torch.int32), _zeros((P - 1,), torch.int64)
        s["xi"] = _zeros((P - 2, 49, lx, lx), torch.int32) if case["xi"] else None
    elif kind == "vacf":
        s["vel"], s["lags"] = _vacf_inputs(case, seed), _vacf_lags(case)
        s["offsets"] = np.arange(case["n_rep"] + 1) * case["n"]
        s["c"] = _zeros((case["n_rep"], case["n_lag"]), torch.float64)
    elif kind == "hist":
        n, n_rep = case["n"], case["n_rep"]
        L = _box(n, 0.0784)
        s["pos"], s["img"] = _walk(_gen(seed), n * n_rep, case["n_snap"], L, 1.1, 1.1)
        s.update(offsets=np.arange(n_rep + 1) * n, box=[L] * n_rep, lags=list(range(1, case["n_lag"] + 1)),
                 width=[48.0 * math.sqrt(l) / case["n_bin"] for l in range(1, case["n_lag"] + 1)],
                 hist=_zeros((n_rep, case["n_lag"], 2, case["n_bin"] + 2), torch.int64))
    elif kind == "mlp_forward":
        s["net"] = m.SurrogateMLP(_mlp_params(seed), case["B"])
        s["x"] = _mlp_x(_gen(seed), case["B"])
    else:
        s["net"] = m.SurrogateMLP(_mlp_params(seed), case["B"])
        s["batches"] = _batches(case, seed)
        s["loss"] = _zeros((1,), torch.float32)
    return s


# --------------------------------------------------------------------- run ---

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "md":
        s["sys"].step(case["steps"])
        pos, vel, img = s["sys"].state()
        if "acc" not in s:
            return [pos, vel, img]
        a = s["acc"]
        return [pos, vel, img, a.moments, a.counts] + ([a.cell_acc] if case["cell_acc"] else [])
    if kind == "cg_pair":
        field = {} if case["field"] == "none" else {case["field"]: s["field"]}
        m.mdlg_coarse_grain(case["lx"], s["L"], s["pos"][0], s["pos"][1], s["counts"], s["moments"],
                            img_prev=s["img"][0], img_cur=s["img"][1], u=(case["u"], 0.0), **field)
        return [s["moments"], s["counts"], s["field"]]
    if kind == "cg_series":
        m.mdlg_coarse_grain_series(s["offsets"], s["box"], s["lx"], s["pos"], s["img"], s["lags"], s["u"], s["counts"],
                                   s["moments"], lattice_offset=s["origin"])
        return [s["moments"], s["counts"]]
    if kind == "neq":
        m.mdlg_neq_mdlg(s["L"], case["lx"], s["pos"], s["img"], s["f"], s["ovf"], s["xi"])
        return [s["f"], s["ovf"], s["xi"]]
    if kind == "vacf":
        m.mdlg_vacf(s["offsets"], s["vel"], s["lags"], s["c"])
        return [s["c"]]
    if kind == "hist":
        m.mdlg_displacement_hist(s["offsets"], s["box"], s["pos"], s["img"], s["lags"], s["width"], case["n_bin"],
                                 s["hist"])
        return [s["hist"]]
    if kind == "mlp_forward":
        return [s["net"].forward(s["x"])]
    for x, r in s["batches"]:
        s["net"].train_step(x, r, 2e-3, s["loss"])
    return [s["net"].params(), s["loss"]]


# -------------------------------------------------------------------- work ---

def work(case):
    """Inputs read once, outputs written once, and the operations of the method itself."""
    kind = case["kind"]
    if kind == "md":
        # state in and out; per step the pairs inside the cutoff (half of pi rc^2 rho each, about 30 operations)
        # and the integration (12); per event the snapshot read and written and the lattice indices (40)
        n = sum(_sizes(case))
        pairs = 0.5 * math.pi * RC * RC * case["phi"] * 4.0 / math.pi
        events = case["steps"] // case["s_cg"] if case["s_cg"] else 0
        fields = 4 * 49 * sum(l * l for l in _lattices(case, [_box(k, case["phi"]) for k in _sizes(case)]))
        return {"bytes": 80.0 * n + 32.0 * n * min(1, events) + (fields if case["cell_acc"] and events else 0),
                "flops": n * (case["steps"] * (30.0 * pairs + 12.0) + 40.0 * events)}
    if kind == "cg_pair":
        return {"bytes": case["n"] * (48.0 if case["img"] else 32.0) + (0 if case["field"] == "none" else 4.0 * 49 * case["lx"] ** 2),
                "flops": 40.0 * case["n"]}
    if kind == "cg_series":
        n, P = case["n"] * case["n_rep"], case["n_snap"]
        pairs = n * sum(P - l for l in LAGS[:case["n_lag"]])
        return {"bytes": 24.0 * n * P, "flops": pairs * (10.0 * case["n_u"] + (16.0 if case["moments"] else 0.0))}
    if kind == "neq":
        n, P = case["n"] * case["n_rep"], case["n_snap"]
        field = 4.0 * 49 * case["lx"] ** 2
        return {"bytes": 24.0 * n * P + field * ((P - 1) + (P - 2 if case["xi"] else 0)), "flops": 12.0 * n * P}
    if kind == "vacf":
        n, P = case["n"] * case["n_rep"], case["n_snap"]
        return {"bytes": 16.0 * n * P, "flops": 4.0 * n * sum(P - l for l in _vacf_lags(case))}
    if kind == "hist":
        n, P = case["n"] * case["n_rep"], case["n_snap"]
        return {"bytes": 24.0 * n * P, "flops": 12.0 * n * sum(P - l for l in range(1, case["n_lag"] + 1))}
    per = 2.0 * sum(a * b for a, b in zip(MLP_DIMS[:-1], MLP_DIMS[1:]))
    if kind == "mlp_forward":
        return {"bytes": 4.0 * case["B"] * (6 + 49) + 2.0 * m.MLP_NPARAMS, "flops": per * case["B"]}
    return {"bytes": case["steps"] * (4.0 * case["B"] * (6 + 49) + 24.0 * m.MLP_NPARAMS),
            "flops": 3.0 * per * case["B"] * case["steps"]}


# ------------------------------------------------------------------- exact ---

class _Pairs:
    """Pairs within rc + skin of a batch of periodic boxes, for plain torch MD."""

    def __init__(self, sizes, boxes):
        rep = torch.repeat_interleave(torch.arange(len(sizes)), torch.tensor(sizes)).cuda()
        box = torch.tensor(boxes, dtype=torch.float64).cuda()
        side = torch.floor(box / (RC + SKIN)).long()
        base = torch.cumsum(side * side, 0) - side * side
        self.L, self.side, self.base = box[rep], side[rep], base[rep]
        self.cells = int((side * side).sum())

    def build(self, x):
        n = x.shape[0]
        c = torch.minimum((x / self.L[:, None] * self.side[:, None]).long(), self.side[:, None] - 1)
        cell = self.base + c[:, 1] * self.side + c[:, 0]
        count = torch.bincount(cell, minlength=self.cells)
        order = torch.argsort(cell)
        start = torch.cumsum(count, 0) - count
        me = torch.arange(n, device=x.device)
        found = []
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                other = self.base + ((c[:, 1] + dy) % self.side) * self.side + (c[:, 0] + dx) % self.side
                for k in range(int(count.max())):
                    i = me[(count[other] > k)]
                    j = order[start[other[i]] + k]
                    i, j = i[j > i], j[j > i]
                    d = self.near(x, i, j)
                    keep = (d * d).sum(dim=1) < (RC + SKIN) ** 2
                    found.append(torch.stack([i[keep], j[keep]]))
        self.i, self.j = torch.cat(found, dim=1)

    def near(self, x, i, j):
        d = x[i] - x[j]
        L = self.L[i][:, None]
        return d - L * torch.round(d / L)

    def force(self, x):
        d = self.near(x, self.i, self.j)
        r2 = (d * d).sum(dim=1)
        inv = 1.0 / r2
        s6 = inv * inv * inv
        f = torch.where(r2 < RC * RC, 24.0 * inv * s6 * (2.0 * s6 - 1.0), torch.zeros_like(r2))[:, None] * d
        return torch.zeros_like(x).index_add_(0, self.i, f).index_add_(0, self.j, -f)


def _exact_md(case, seed):
    x, v, boxes = _md_inputs(case, seed)
    sizes = _sizes(case)
    pairs = _Pairs(sizes, boxes)
    L = pairs.L[:, None]
    s_cg = case["s_cg"]
    true, snap = x.clone(), x.clone()  # unwrapped positions, and those of the last event
    moments = torch.zeros((len(sizes), 5), dtype=torch.float64)
    pairs.build(x)
    f = pairs.force(x)
    for k in range(1, case["steps"] + 1):
        v = v + 0.5 * DT * f
        x = x + DT * v
        true = true + DT * v
        x = torch.where(x >= L, x - L, torch.where(x < 0, x + L, x))
        if k % 20 == 0:
            pairs.build(x)
        f = pairs.force(x)
        v = v + 0.5 * DT * f
        if s_cg and k % s_cg == 0:
            for r, d in enumerate(torch.split(true - snap, sizes)):
                d2 = d * d
                row = [2.0 * d.shape[0], float(d2.sum()), float((d2 * d2).sum()), float(d[:, 0].sum()), float(d[:, 1].sum())]
                moments[r] += torch.tensor(row, dtype=torch.float64)
            snap = true.clone()
    if not s_cg:
        return [x, v, None]
    return [x, v, None, moments, None] + ([None] if case["cell_acc"] else [])


def _sums(d):
    """(samples, sum d^2, sum d^4, sum d_x, sum d_y) of displacements [..., 2]."""
    d2 = d * d
    return torch.stack([torch.tensor(float(d.numel()), dtype=torch.float64, device="cuda"), d2.sum(), (d2 * d2).sum(),
                        d[..., 0].sum(), d[..., 1].sum()])


def _encode(x):
    x = x.double()
    return torch.stack([x[:, 0] / 0.4, torch.log(x[:, 1]) / math.log(20.0), (torch.log(x[:, 2]) + 6.0) / 1.5,
                        5.0 * x[:, 3] * x[:, 4], 5.0 * x[:, 3] * x[:, 5], 5.0 * x[:, 3]], dim=1)


def _logits(theta, x):
    h, at = _encode(x), 0
    for k, (fi, fo) in enumerate(zip(MLP_DIMS[:-1], MLP_DIMS[1:])):
        w = theta[at:at + fi * fo].view(fi, fo)
        h = h @ w + theta[at + fi * fo:at + fi * fo + fo]
        at += fi * fo + fo
        if k < 3:
            h = torch.nn.functional.silu(h)
    return h


def exact(case, seed):
    kind = case["kind"]
    if kind == "md":
        return _exact_md(case, seed) if sum(_sizes(case)) * case["steps"] <= 5e8 else None
    if kind == "cg_pair":
        s = prepare(case, seed)
        d = s["pos"][1] - s["pos"][0]
        if case["img"]:
            d = d + s["L"] * (s["img"][1] - s["img"][0]).double()
        return [_sums(d), None, None]
    if kind == "cg_series":
        if not case["moments"]:
            return None
        s = _series_inputs(case, seed)
        out = []
        for r, L in enumerate(s["box"]):
            a, b = int(s["offsets"][r]), int(s["offsets"][r + 1])
            x = s["pos"][:, a:b] + L * s["img"][:, a:b].double()
            out.append(torch.stack([_sums(x[l:] - x[:-l]) for l in s["lags"]]))
        return [torch.stack(out), None]
    if kind == "vacf":
        vel, n = _vacf_inputs(case, seed), case["n"]
        c = [[(vel[l:, r * n:(r + 1) * n] * vel[:vel.shape[0] - l, r * n:(r + 1) * n]).sum() for l in _vacf_lags(case)]
             for r in range(case["n_rep"])]
        return [torch.tensor(c, dtype=torch.float64)]
    if kind == "mlp_forward":
        theta = torch.from_numpy(_mlp_params(seed)).cuda().double()
        return [torch.softmax(_logits(theta, _mlp_x(_gen(seed), case["B"])), dim=1)]
    if kind == "mlp_train":
        theta = torch.from_numpy(_mlp_params(seed)).cuda().double().requires_grad_()
        m1, m2 = torch.zeros_like(theta), torch.zeros_like(theta)
        loss = None
        for k, (x, r) in enumerate(_batches(case, seed), 1):
            r = r.double()
            loss = (torch.xlogy(r, r) - r * torch.log_softmax(_logits(theta, x), dim=1)).sum() / x.shape[0]
            (g,) = torch.autograd.grad(loss, theta)
            with torch.no_grad():
                m1 = 0.9 * m1 + 0.1 * g
                m2 = 0.999 * m2 + 0.001 * g * g
                theta -= 2e-3 * (m1 / (1 - 0.9 ** k)) / (torch.sqrt(m2 / (1 - 0.999 ** k)) + 1e-8)
        return [theta.detach(), loss.detach()]
    return None
