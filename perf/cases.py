"""Performance cases: the replans, rollouts, batches and served requests that users of the planner run.

A case is a dict of plain values; `kind` names the entry point:

  replan   one call of a `Plan`: n_iters CEM iterations from a start state, warm start shifted by one step;
  rollout  the rollout stage alone on controls the caller has written into the plan's candidate buffer;
  batch    one `Batch` replan of several uneven instances in one launch;
  serve    one burst of requests, one per robot, through a `Server` until every action is back.

Sizes are those of the named workloads (`mtp_workloads`), of the tests and of the benchmark, or odd sizes of
the same ranges.  Every input follows from the seed: task (goal, obstacles, targets), randomised models, start
state and the planner's Philox key.
"""
import math

import numpy as np
import torch

import mtp_workloads as W
import paper_2505_01059_amd as mtp

POINT_MASS, CHAIN, CONTACT = W.POINT_MASS, W.CHAIN, W.CHAIN_CONTACT
BSPLINE, AKIMA, LINEAR = W.BSPLINE, W.AKIMA, W.LINEAR


def _plan_case(name, dynamics, links, tensor, gauss, horizon, layers, width, elites, iters, interp=BSPLINE, degree=3,
               replicas=1, wor=0, dt=0.0, obstacles=20, kind="replan"):
    return {"name": name, "kind": kind, "dynamics": dynamics, "links": links, "tensor": tensor, "gauss": gauss,
            "horizon": horizon, "layers": layers, "width": width, "elites": elites, "iters": iters, "interp": interp,
            "degree": degree, "replicas": replicas, "wor": wor, "dt": dt, "obstacles": obstacles}


def listed():
    return [
        # the paper's navigation sizes: 256 candidates, 20 steps; a control loop at hundreds of Hz, all latency
        _plan_case("pm_paper", POINT_MASS, 0, 255, 1, 20, 5, 30, 16, 10, dt=0.05),
        # the point-mass workload of the benchmark and of the smoke test
        _plan_case("pm_small", POINT_MASS, 0, 256, 32, 50, 4, 8, 16, 10),
        # a point mass among the sizes of the uneven mix, ragged, Akima
        _plan_case("pm_ragged", POINT_MASS, 0, 3001, 340, 77, 6, 19, 52, 6, interp=AKIMA),
        # a short chain (three links), a few hundred candidates, quadratic B-spline
        _plan_case("chain3_small", CHAIN, 3, 500, 61, 32, 5, 12, 16, 4, degree=2),
        # the 7-link workload of the benchmark
        _plan_case("chain7", CHAIN, 7, 8192, 1024, 128, 8, 32, 128, 8, interp=AKIMA),
        # a 12-link chain of the uneven mix on its own, odd sizes
        _plan_case("chain12", CHAIN, 12, 3001, 375, 64, 9, 33, 52, 6),
        # ground contact, every candidate under three randomised models
        _plan_case("contact7_models", CONTACT, 7, 1024, 129, 96, 8, 32, 64, 4, replicas=3),
        # one eighth of the 24-link contact workload (its share on one of eight GPUs)
        _plan_case("contact24_share", CONTACT, 24, 8192, 512, 256, 12, 64, 512, 6),
        # the benchmark's default workload: 24 links, contact, 69632 candidates
        _plan_case("contact24", CONTACT, 24, 65536, 4096, 256, 12, 64, 512, 6),
        # evaluation of given controls: rollout and cost of 2003 candidates of the 12-link chain
        _plan_case("rollout12", CHAIN, 12, 1780, 223, 96, 8, 32, 32, 1, kind="rollout"),
        # many uneven instances in one launch: 32 of the mix
        {"name": "mix32", "kind": "batch", "first": 0, "instances": 32},
        # a burst of requests of 24 robots of the serving fleet
        {"name": "serve24", "kind": "serve", "first": 10000, "instances": 24},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["replan"] * 8 + ["rollout"] * 2 + ["batch", "serve"])
    if kind in ("batch", "serve"):
        first = rng.randrange(0, 200) if kind == "batch" else 10000 + rng.randrange(0, 400)
        return {"kind": kind, "first": first, "instances": _log_int(rng, 4, 32)}
    dynamics = rng.choice([POINT_MASS, CHAIN, CHAIN, CONTACT] if kind == "replan" else [POINT_MASS, CHAIN, CHAIN])
    if dynamics == POINT_MASS:
        links = 0
    elif dynamics == CHAIN:
        links = rng.choice([2, 3, 4, 7, 12, 24] if kind == "replan" else [2, 3, 4, 7, 12])
    else:
        links = rng.choice([4, 7, 24])
    replicas = rng.choice([1, 1, 2, 3]) if dynamics == CONTACT else 1
    total = _log_int(rng, 200, 2500 if kind == "rollout" else 40000 // replicas)
    # tensor : local about 8 : 1, as in the workloads
    gauss = max(1, total // rng.choice([8, 9, 17]))
    horizon = rng.choice([16, 20, 32, 50, 64, 96, 128, 256]) + rng.choice([0, 0, 1, 3])
    if kind == "rollout":
        horizon = min(horizon, 96)
    interp = rng.choice([BSPLINE, BSPLINE, AKIMA, LINEAR])
    wor = 1 if rng.random() < 0.1 else 0
    return {"kind": kind, "dynamics": dynamics, "links": links, "tensor": total - gauss, "gauss": gauss,
            "horizon": horizon, "layers": rng.randint(6, 12), "width": rng.randint(8, 64),
            "elites": min(max(total // 64, 16), 512), "iters": rng.choice([4, 5, 6, 8, 10]) if kind == "replan" else 1,
            "interp": interp, "degree": rng.choice([3, 3, 3, 2, 4, 5]) if interp == BSPLINE else 3,
            "replicas": replicas, "wor": wor, "dt": 0.0, "obstacles": rng.choice([20, 20, 8, 30])}


# ---------------------------------------------------------------- inputs

def _config(case, seed):
    common = dict(horizon=case["horizon"], n_layers=case["layers"], n_width=case["width"], n_tensor=case["tensor"],
                  n_gauss=case["gauss"], n_elites=case["elites"], n_iters=case["iters"], interp=case["interp"],
                  bspline_degree=case["degree"], seed=seed)
    if case["dynamics"] == POINT_MASS:
        cfg = W.point_mass_config(n_obstacles=case["obstacles"], **common)
    elif case["dynamics"] == CHAIN:
        cfg = W.chain_config(n_links=case["links"], **common)
    else:
        # short chains hang above a ground they can reach, as the contact tests have it
        ground = -4.0 if case["links"] > 7 else -0.5
        cfg = W.chain_contact_config(n_links=case["links"], n_replicas=case["replicas"], ground_y=ground, **common)
    if case["dt"] > 0.0:
        cfg = cfg.replace(dt=np.float32(case["dt"]))
    return cfg.replace(sample_wor=case["wor"])


def _instances(case, seed):
    """Instances of the uneven mix: sizes by the case, tasks and random streams by the seed."""
    out = []
    for i in range(case["instances"]):
        cfg = W.mix_instance(case["first"] + i)
        s = seed * 1009 + i
        task = W.point_mass_task(s) if cfg.dynamics == POINT_MASS else W.chain_task(s, cfg.n_links)
        out.append(cfg.replace(seed=s, task=task))
    return out


def _controls(case, cfg, seed):
    """Smooth random controls (T, n, B) within the control box, float32."""
    rng = np.random.default_rng([seed, 77])
    T, n, B = cfg.horizon, cfg.ctrl_dim, cfg.n_samples
    knots = rng.uniform(float(cfg.u_min), float(cfg.u_max), size=(6, n, B)).astype(np.float32)
    pos = np.arange(T) * (5.0 / T)
    i = pos.astype(np.int64)
    f = (pos - i).astype(np.float32)[:, None, None]
    return knots[i] * (np.float32(1) - f) + knots[i + 1] * f


def prepare(case, seed):
    dev = torch.device("cuda:0")
    if case["kind"] in ("replan", "rollout"):
        cfg = _config(case, seed)
        plan = mtp.Plan(cfg, device=dev)
        x0 = torch.tensor(W.initial_state(cfg, seed), device=dev)
        state = {"kind": case["kind"], "plan": plan, "x0": x0, "bufs": plan.buffers()}
        if case["kind"] == "rollout":
            state["bufs"]["U"].copy_(torch.from_numpy(_controls(case, cfg, seed)))
            plan.set_x0(x0)
        return state
    cfgs = _instances(case, seed)
    x0s = [W.initial_state(c, seed + i) for i, c in enumerate(cfgs)]
    if case["kind"] == "batch":
        b = mtp.Batch(cfgs, device=dev)
        return {"kind": "batch", "batch": b, "x0": b.pack_x0(x0s), "bufs": [b.buffers(i) for i in range(len(cfgs))]}
    budget = sum(mtp.resident_bytes(c) + mtp.transient_bytes(c) + (1 << 16) for c in cfgs)
    srv = mtp.Server(budget, len(cfgs), device=dev, robots=cfgs)
    return {"kind": "serve", "server": srv, "x0": x0s}


# ---------------------------------------------------------------- one pass

def run(state):
    if state["kind"] == "replan":
        state["plan"].replan(state["x0"], shift=1)
        b = state["bufs"]
        return {"action": b["action"], "mu": b["mu"], "sigma": b["sigma"], "cost": b["cost"]}
    if state["kind"] == "rollout":
        state["plan"].run_stage(mtp.STAGE_ROLLOUT, 0, 0)
        return {"cost": state["bufs"]["cost"]}
    if state["kind"] == "batch":
        state["batch"].replan(state["x0"], shift=1)
        bufs = state["bufs"]
        return {"action": torch.cat([b["action"] for b in bufs]),
                "mu": torch.cat([b["mu"].reshape(-1) for b in bufs]),
                "sigma": torch.cat([b["sigma"].reshape(-1) for b in bufs])}
    srv = state["server"]
    for robot, x in enumerate(state["x0"]):
        srv.submit(robot, x, shift=1)
    done = {}
    while len(done) < len(state["x0"]):
        srv.pump(50)
        for c in srv.poll():
            done[c["robot"]] = c["u"]
    return {"action": np.concatenate([done[i] for i in range(len(done))])}


# ---------------------------------------------------------------- necessary work

def _flops_per_step(dynamics, links, obstacles):
    """Floating-point operations of one step of one candidate: dynamics and cost (multiply-add counts two)."""
    if dynamics == POINT_MASS:
        return 8 + 6 + 8 * obstacles + 6
    return 186 * links - 108 + (96 * links if dynamics == CONTACT else 0)


def _replan_work(dynamics, links, obstacles, B, T, n, d, K, R, E):
    flops = float(B) * R * T * K * _flops_per_step(dynamics, links, obstacles)
    # start state, mean and spread read and written, task table, randomised models, costs, action
    table = R * B * (n + 1) if dynamics == CONTACT else 5 + 2 * n + 3 * obstacles
    return {"bytes": 4.0 * (d + 4 * T * n + table + B + n), "flops": flops}


def work(case):
    if case["kind"] in ("replan", "rollout"):
        dyn, links = case["dynamics"], case["links"]
        n, d = (2, 4) if dyn == POINT_MASS else (links, 2 * links)
        B, T, R = case["tensor"] + case["gauss"], case["horizon"], case["replicas"]
        if case["kind"] == "rollout":
            return {"bytes": 4.0 * (B * T * n + B + d),
                    "flops": float(B) * R * T * _flops_per_step(dyn, links, case["obstacles"])}
        return _replan_work(dyn, links, case["obstacles"], B, T, n, d, case["iters"], R, case["elites"])
    total = {"bytes": 0.0, "flops": 0.0}
    for i in range(case["instances"]):
        c = W.mix_instance(case["first"] + i)
        w = _replan_work(c.dynamics, c.n_links, 20, c.n_samples, c.horizon, c.ctrl_dim, c.state_dim, c.n_iters, 1,
                         c.n_elites)
        total = {k: total[k] + w[k] for k in total}
    return total


# ---------------------------------------------------------------- 64-bit values

def _exact_point_mass(cfg, x0, U):
    t = cfg.task
    T, _, B = U.shape
    p = np.repeat(x0[:2, None], B, 1)
    v = np.repeat(x0[2:, None], B, 1)
    dt, cost = float(cfg.dt), np.zeros(B)
    goal = t.goal.astype(np.float64)[:, None]
    obs = t.obstacles.astype(np.float64)
    for k in range(T):
        v = v + dt * U[k]
        p = p + dt * v
        hit = (p[0] - obs[:, 0:1]) ** 2 + (p[1] - obs[:, 1:2]) ** 2 < obs[:, 2:3] ** 2
        cost += float(t.goal_weight) * ((p - goal) ** 2).sum(0) + float(t.obstacle_penalty) * hit.sum(0)
        cost += float(t.ctrl_weight) * (U[k] ** 2).sum(0)
    return cost


def _exact_chain(cfg, x0, U):
    """Planar chain of point masses, absolute angles from the downward vertical: M(phi) phi'' = Q - h - g, RK4."""
    t, n = cfg.task, cfg.n_links
    T, _, B = U.shape
    ln = t.lengths.astype(np.float64)
    tail = np.cumsum(t.masses.astype(np.float64)[::-1])[::-1]
    idx = np.arange(n)
    coef = tail[np.maximum(idx[:, None], idx[None, :])] * ln[:, None] * ln[None, :]
    grav = float(t.gravity) * tail * ln
    dt = float(cfg.dt)
    ph, om, cost = np.repeat(x0[None, :n], B, 0), np.repeat(x0[None, n:], B, 0), np.zeros(B)

    def acc(phi, w, q):
        dif = phi[:, :, None] - phi[:, None, :]
        rhs = q - np.einsum("bij,bj->bi", coef * np.sin(dif), w * w) - grav * np.sin(phi)
        return np.linalg.solve(coef * np.cos(dif), rhs[:, :, None])[:, :, 0]

    for k in range(T):
        u = U[k].T
        q = u - np.concatenate([u[:, 1:], np.zeros((B, 1))], 1)
        a1 = acc(ph, om, q)
        w2 = om + 0.5 * dt * a1
        a2 = acc(ph + 0.5 * dt * om, w2, q)
        w3 = om + 0.5 * dt * a2
        a3 = acc(ph + 0.5 * dt * w2, w3, q)
        w4 = om + dt * a3
        a4 = acc(ph + dt * w3, w4, q)
        ph = ph + dt / 6.0 * (om + 2 * w2 + 2 * w3 + w4)
        om = om + dt / 6.0 * (a1 + 2 * a2 + 2 * a3 + a4)
        ex, ey = (ln * np.sin(ph)).sum(1), -(ln * np.cos(ph)).sum(1)
        cost += float(t.goal_weight) * ((ex - float(t.target[0])) ** 2 + (ey - float(t.target[1])) ** 2)
        cost += float(t.ctrl_weight) * (u * u).sum(1)
    return cost


def exact(case, seed):
    """Costs of the rollout cases in float64; a whole replan has none (its softmax parts any two roundings)."""
    if case["kind"] != "rollout":
        return None
    cfg = _config(case, seed)
    x0 = W.initial_state(cfg, seed).astype(np.float64)
    U = _controls(case, cfg, seed).astype(np.float64)
    return {"cost": (_exact_point_mass if case["dynamics"] == POINT_MASS else _exact_chain)(cfg, x0, U)}
