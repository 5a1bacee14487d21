"""What is timed: the planner's work as its users ask for it.

Each case is one pass through the public binding (``Planner``,
``AnytimePlanner``, ``BatchPlanner``, ``ClassPlanner``, ``Surrogate``) on a
seeded workload of ``workloads``: the sizes are those of the repository's own
workloads and benchmark forms, from the smallest plan (bound by launches) to a
batch of mixed plans, with odd sizes between them.

``listed()`` names the cases, ``draw(rng)`` draws another from the same ranges,
``prepare(case, seed)`` makes what a program holds before the call, ``run``
makes one pass, ``work`` says what a pass cannot do without and ``exact`` gives
the 64-bit values of a pass in plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import workloads as wl
from paper_2608_25830_amd import gtmp

# RRT-Connect settings of the arm (extension step, check spacing, ellipsoid)
LP = dict(step=0.4, resolution=0.1, ell_factor=1.5)
BAND = 0.2  # lazy selection band
PRUNE_TAU = 0.5  # logit threshold of the pruned plans

# states evaluated per edge by a check that tests each vertex once and stops an
# edge at its first state in contact, over the seeded scenes
STATES_PER_EDGE = {"2d-small": 3.5, "2d-large": 4.2, "3d-point": 11.0, "arm7": 2.3}


# --------------------------------------------------------------------------- #
# cases
# --------------------------------------------------------------------------- #
def listed():
    return [
        # the smallest plan: a 2D robot replanning among a few circles
        dict(name="plan-2d-small", kind="plan", workload="2d-small", M=4, N=64, H=8, G=1, flags=False),
        # a point robot in space, a plan of ordinary size
        dict(name="plan-3d", kind="plan", workload="3d-point", M=6, N=256, H=16, G=1, flags=False),
        # deep 2D graph with finely checked edges
        dict(name="plan-2d-large", kind="plan", workload="2d-large", M=16, N=1024, H=32, G=1, flags=False),
        # the headline plan: the 7-joint arm
        dict(name="plan-arm7", kind="plan", workload="arm7", M=8, N=2048, H=16, G=1, flags=False),
        # an arm plan of odd sizes with several goals, whose edge flags are wanted too
        dict(name="plan-arm7-ragged", kind="plan", workload="arm7", M=5, N=501, H=24, G=3, flags=True),
        # lazy realisation of the headline plan
        dict(name="lazy-arm7", kind="lazy", workload="arm7", M=8, N=2048, H=16),
        # AO-GTMP on the arm: six stages of growing samples and layers
        dict(name="growing-arm7", kind="anytime", workload="arm7", mode="growing", M_min=6, M=8, N_min=256, N=2048,
             H=16, stages=6, simplify=False, bias=False),
        # a plan whose failed edges get the RRT-Connect local planner
        dict(name="rrtc-arm7", kind="rrtc", workload="arm7", M=6, N=100, H=16, budget=100, cap=512),
        # Anytime-GTMP with the class archive on the small 2D scene
        dict(name="classes-2d", kind="classes", M=4, N=128, H=8, stages=10, L=64),
        # one training step of the collision surrogate (forward, backward, Adam)
        dict(name="train-8192", kind="train", n=8192),
        # the surrogate's prune mask over a large plan's edges
        dict(name="prune-arm7-n4096", kind="prune", M=8, N=4096),
        # a batch of mixed plans: 2D and arm, plain, restart and growing
        dict(name="batch-128", kind="batch", n=128, H=16, mix=0),
    ]


def _log(rng, lo, hi):
    """An integer of lo..hi, spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["plan", "plan", "plan", "plan", "lazy", "anytime", "anytime", "rrtc", "classes", "train",
                       "prune", "batch"])
    if kind == "plan":
        name = rng.choice(["2d-small", "2d-large", "3d-point", "arm7", "arm7"])
        return dict(kind=kind, workload=name, M=rng.randint(2, 16), N=_log(rng, 16, 2048 if name == "arm7" else 1024),
                    H=rng.randint(4, 32), G=rng.choice([1, 1, 2, 5]), flags=rng.random() < 0.4)
    if kind == "lazy":
        name = rng.choice(["2d-large", "3d-point", "arm7", "arm7"])
        return dict(kind=kind, workload=name, M=rng.randint(3, 10), N=_log(rng, 100, 2048), H=rng.randint(8, 24))
    if kind == "anytime":
        name, M, N = rng.choice(["2d-small", "2d-large", "arm7"]), rng.randint(4, 10), _log(rng, 64, 2048)
        grow = rng.random() < 0.6
        return dict(kind=kind, workload=name, mode="growing" if grow else "restart", M_min=max(2, M - 2), M=M,
                    N_min=max(8, N // 8), N=N, H=rng.randint(8, 20), stages=rng.randint(3, 6),
                    simplify=rng.random() < 0.5, bias=grow and name == "arm7" and rng.random() < 0.5)
    if kind == "rrtc":
        return dict(kind=kind, workload=rng.choice(["2d-small", "arm7", "arm7"]), M=rng.randint(3, 6),
                    N=_log(rng, 16, 100), H=16, budget=_log(rng, 10, 100), cap=rng.choice([64, 256, 512]))
    if kind == "classes":
        return dict(kind=kind, M=rng.randint(3, 8), N=_log(rng, 24, 200), H=rng.randint(8, 16),
                    stages=rng.randint(2, 10), L=rng.choice([16, 64]))
    if kind == "train":
        return dict(kind=kind, n=256 * _log(rng, 1, 64))
    if kind == "prune":
        return dict(kind=kind, M=rng.randint(3, 8), N=_log(rng, 128, 4096))
    return dict(kind=kind, n=_log(rng, 8, 100), H=rng.randint(8, 16), mix=rng.randint(1, 999))


# --------------------------------------------------------------------------- #
# inputs
# --------------------------------------------------------------------------- #
def _workload(case, seed):
    """The case's workload on the scene of this seed, with its sampling key;
    further goals are drawn in the box."""
    w = wl.make_workload(case["workload"], seed % 5, M=case["M"], N=case["N"], H=case["H"])
    w["seed"] = 7919 * (seed + 1)
    G = case.get("G", 1)
    if G > 1:
        g = np.random.default_rng([0x60A1, seed])
        more = g.uniform(w["lo"], w["hi"], (G - 1, w["d"])).astype(np.float32)
        w["goals"], w["G"] = np.concatenate([w["goals"], more]), G
    return w


def _net(seed, d, batch=256):
    """A surrogate as it stands before training (its cost does not depend on the weights)."""
    P, Bf = wl.surrogate_init(seed, d)
    return gtmp.Surrogate(P, Bf, batch=batch)


def _train_inputs(case, seed):
    """A batch of joint configurations, uniform in the box (labels: the exact checker's)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    w = wl.make_workload("arm7", seed % 5)
    return w, (torch.rand((case["n"], w["d"]), generator=g, device="cuda") * 2 - 1) * wl.PI32


def prepare(case, seed):
    kind = case["kind"]
    st = dict(kind=kind, case=case)
    if kind in ("plan", "lazy", "rrtc"):
        w = _workload(case, seed)
        st["pl"] = pl = gtmp.Planner(w, flags=case.get("flags", True))
        st["seed"] = w["seed"]
        if kind == "lazy":
            pl.lazy_ws = gtmp._aligned_workspace(gtmp.gtmp_lazy_workspace_size(pl.prob))
        if kind == "rrtc":
            pl.rrtc_ws = gtmp._aligned_workspace(gtmp.gtmp_rrtc_workspace_size(pl.prob))
            lp = dict(LP) if w["kind"] == "arm" else dict(LP, step=1.0, resolution=0.25)
            st["lp"] = gtmp.make_rrtc_opts(case["budget"], case["cap"], **lp)
    elif kind == "anytime":
        w = _workload(case, seed)
        net = _net(seed, w["d"]) if case["bias"] else None
        mode = gtmp.GTMP_ANYTIME_GROWING if case["mode"] == "growing" else gtmp.GTMP_ANYTIME_RESTART
        grow = dict(M_min=case["M_min"], M_max=case["M"], N_min=case["N_min"], N_max=case["N"])
        st["ap"] = ap = gtmp.AnytimePlanner(w, mode, case["stages"], use_graph=case["mode"] == "restart", bias=net,
                                            bias_tau=0.0, simplify=case["simplify"],
                                            **(grow if case["mode"] == "growing" else {}))
        ap.best_idx.fill_(-1)  # a chain shorter than the longest leaves the rest as it was
        ap.best_wp.zero_()
        st["seed"] = w["seed"]
    elif kind == "classes":
        w = _workload(dict(case, workload="2d-small"), seed)
        st["cp"] = gtmp.ClassPlanner(w, w["circles"][:, :2], case["stages"], L=case["L"], cap=4096)
        st["seed"] = w["seed"]
    elif kind == "train":
        w, X = _train_inputs(case, seed)
        robot, scene = gtmp.model_of(w)
        y = torch.empty(case["n"], device="cuda", dtype=torch.uint8)
        gtmp.gtmp_state_check(robot, scene, w["d"], X, None, y)
        st.update(net=_net(seed, w["d"], batch=case["n"]), X=X, y=y)
    elif kind == "prune":
        w = _workload(dict(case, workload="arm7", H=16), seed)
        M, N, d = w["M"], w["N"], w["d"]
        prob = gtmp.make_problem(d, M, N, 1, 16, w["lo"], w["hi"], w["penalty"])
        robot, scene = gtmp.model_of(w)
        Q = torch.empty((M, N, d), device="cuda")
        gtmp.gtmp_sample_layers(prob, w["seed"], 0, Q)
        E = N + (M - 1) * N * N + N
        st.update(net=_net(seed, d), prob=prob, robot=robot, scene=scene, Q=Q, d=d,
                  q0=torch.from_numpy(w["q0"]).cuda(), goals=torch.from_numpy(w["goals"]).cuda(),
                  coll=torch.empty(M * N, device="cuda", dtype=torch.uint8),
                  prune=torch.empty(E, device="cuda", dtype=torch.uint8), logits=torch.empty(E, device="cuda"))
    else:
        specs = wl.batch_specs(case["n"], seed=case["mix"], H=case["H"])
        for i, sp in enumerate(specs):  # every plan samples with a key of its own
            sp["seed"] = 1000003 * (seed + 1) + i
        st["bp"] = bp = gtmp.BatchPlanner(specs, use_graph=True)
        bp.best_idx.fill_(-1)
        bp.best_wp.zero_()
    return st


# --------------------------------------------------------------------------- #
# one pass
# --------------------------------------------------------------------------- #
def _plan_out(pl, flags):
    out = dict(Q=pl.Q, C_s=pl.C_s, C_h=pl.C_h, C_l=pl.C_l, V=pl.V, A=pl.A, V_s=pl.V_s, a_s=pl.a_s, idx=pl.idx,
               wp=pl.wp, cost=pl.cost)
    if flags:
        out["flags"] = pl.flags
    return out


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "plan":
        st["pl"].plan(st["seed"], 0)
        return _plan_out(st["pl"], case["flags"])
    if kind == "lazy":
        st["pl"].plan_lazy(st["seed"], 0, band=BAND)
        return _plan_out(st["pl"], True)
    if kind == "rrtc":
        pl = st["pl"]
        pl.sample(st["seed"], 0)
        pl.check()
        pl.repair(st["lp"], st["seed"], 0)
        pl.sweep()
        pl.extract()
        return _plan_out(pl, True)
    if kind == "anytime":
        ap = st["ap"]
        ap.run(st["seed"])
        return dict(cost=ap.best_cost, idx=ap.best_idx, wp=ap.best_wp, meta=ap.best_meta, stages=ap.stage_costs)
    if kind == "classes":
        cp = st["cp"]
        cp.run(st["seed"])
        return dict(labels=cp.a_lab, costs=cp.a_cost, stage=cp.a_stage, wp=cp.a_wp, count=cp.a_count,
                    overflow=cp.overflow)
    if kind == "train":
        net = st["net"]
        net.grad(st["X"], st["y"])
        net.adam(lr=wl.SURROGATE["lr"])
        return dict(loss=net.loss_buf, grad=net.grad_buf, params=net.params)
    if kind == "prune":
        M, N, d = st["case"]["M"], st["case"]["N"], st["d"]
        gtmp.gtmp_state_check(st["robot"], st["scene"], d, st["Q"].reshape(M * N, d), None, st["coll"])
        st["net"].prune(st["prob"], st["q0"], st["goals"], st["Q"], PRUNE_TAU, st["prune"], st["logits"],
                        vcoll=st["coll"])
        return dict(coll=st["coll"], prune=st["prune"], logits=st["logits"])
    bp = st["bp"]
    bp.run()
    return dict(cost=bp.best_cost, idx=bp.best_idx, wp=bp.best_wp, meta=bp.best_meta, stages=bp.stage_costs)


# --------------------------------------------------------------------------- #
# what a pass cannot do without
# --------------------------------------------------------------------------- #
def _state_flops(name):
    """FP32 operations of one state: interpolation, kinematics, sphere centres
    and their bins, and the exact tests behind them (arm); interpolation, bins
    and tests (point)."""
    return {"2d-small": 20 + 15, "2d-large": 20 + 15, "3d-point": 30 + 15}.get(name, 992 + 24)


def _graph(M, N, G, name, states=None):
    """Bytes and operations of one checked and swept graph."""
    d = wl.WORKLOADS[name]["d"]
    E = N + (M - 1) * N * N + N * G
    per = STATES_PER_EDGE[name] if states is None else states
    return 4 * E + 4 * M * N * (d + 2), E * (per * _state_flops(name) + 3 * d + 2)


MLP_FLOP = 2 * (64 * 256 + 3 * 256 * 256 + 256)


def _schedule(M_min, N_min, M, N, stages):
    """(M, N) of each stage of the growing loop."""
    out, m, n = [], min(M_min, M), min(N_min, N)
    while len(out) < stages:
        out.append((m, n))
        if n < N:
            n = min(2 * n, N)
        elif m < M:
            m += 1
        else:
            break
    return out


def work(case):
    kind = case["kind"]
    if kind == "plan":
        b, f = _graph(case["M"], case["N"], case["G"], case["workload"])
        E = case["N"] + (case["M"] - 1) * case["N"] ** 2 + case["N"] * case["G"]
        return dict(bytes=b + (E if case["flags"] else 0), flops=f)
    if kind == "lazy":
        b, f = _graph(case["M"], case["N"], 1, case["workload"], states=0.02)
        return dict(bytes=1.25 * b, flops=f)
    if kind == "rrtc":
        b, f = _graph(case["M"], case["N"], 1, case["workload"])
        E = case["N"] * 2 + (case["M"] - 1) * case["N"] ** 2
        return dict(bytes=1.25 * b, flops=f + 0.25 * E * case["budget"] * 6 * _state_flops(case["workload"]))
    if kind == "anytime":
        if case["mode"] == "growing":
            shapes = _schedule(case["M_min"], case["N_min"], case["M"], case["N"], case["stages"])
        else:
            shapes = [(case["M"], case["N"])] * case["stages"]
        each = [_graph(m, n, 1, case["workload"]) for m, n in shapes]
        return dict(bytes=sum(b for b, _ in each), flops=sum(f for _, f in each))
    if kind == "classes":
        b, f = _graph(case["M"], case["N"], 1, "2d-small")
        return dict(bytes=case["stages"] * (b + 24 * case["M"] * case["N"] * case["L"]), flops=case["stages"] * f)
    if kind == "train":
        P = 64 * 256 + 3 * 256 * 256 + 4 * 256 + 257
        return dict(bytes=case["n"] * 29 + P * 4 * 8, flops=3.0 * case["n"] * MLP_FLOP)
    if kind == "prune":
        E = 2 * case["N"] + (case["M"] - 1) * case["N"] ** 2
        return dict(bytes=5 * E + 28 * case["M"] * case["N"], flops=0.28 * E * MLP_FLOP)
    # a plan of the mix, on average: M 10, mean N^2 of its choices, 3.4 stages,
    # the growing ones' first stages smaller
    one = [_graph(10, 1045, 1, w) for w in ("2d-large", "arm7")]
    return dict(bytes=case["n"] * 2.8 * sum(b for b, _ in one) / 2, flops=case["n"] * 2.8 * sum(f for _, f in one) / 2)


# --------------------------------------------------------------------------- #
# 64-bit values
# --------------------------------------------------------------------------- #
def _philox(c, key):
    """Philox4x32-10 of the counters c (four uint64 arrays of 32-bit values)."""
    c = [x.astype(np.uint64) for x in c]
    k0, k1, low = key & 0xFFFFFFFF, (key >> 32) & 0xFFFFFFFF, np.uint64(0xFFFFFFFF)
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & low, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1),
             p0 & low]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _samples(w):
    """Q [M][N][d] of the workload's key at stage 0, in 64 bits."""
    M, N, d = w["M"], w["N"], w["d"]
    n, m = np.meshgrid(np.arange(N), np.arange(M))
    Q = np.zeros((M, N, d))
    for blk in range((d + 3) // 4):
        words = _philox([n, m, np.zeros_like(n), np.full_like(n, blk)], w["seed"])
        for i in range(min(4, d - 4 * blk)):
            j = 4 * blk + i
            u = (words[i] >> np.uint64(8)).astype(np.float64) * 2.0 ** -24
            Q[:, :, j] = float(w["lo"][j]) + u * (float(w["hi"][j]) - float(w["lo"][j]))
    return torch.from_numpy(Q).cuda()


class _Exact:
    """Collision test of a workload in 64 bits: signed distance <= 0."""

    def __init__(self, w):
        def t(x):
            return torch.from_numpy(np.asarray(x, np.float32)).double().cuda()
        self.arm = w["kind"] == "arm"
        self.sph = t(w["circles"] if w["kind"] == "point2d" else w["obs_spheres"])
        self.box = t(w["boxes"] if w["kind"] == "point2d" else w["obs_boxes"])
        if self.arm:
            self.dh = np.asarray(w["dh"], np.float64)
            self.link = [int(x) for x in w["sph_link"]]
            self.t, self.r = t(w["sph_t"]), t(w["sph_r"])

    def _centres(self, q):
        n = q.shape[0]
        R = torch.eye(3, device=q.device, dtype=torch.float64).expand(n, 3, 3)
        o = torch.zeros((n, 3), device=q.device, dtype=torch.float64)
        origins = [o]
        for i, (a, al, dz, off) in enumerate(self.dh):
            c, s, ca, sa = torch.cos(q[:, i] + off), torch.sin(q[:, i] + off), math.cos(al), math.sin(al)
            x = c[:, None] * R[:, :, 0] + s[:, None] * R[:, :, 1]
            y = c[:, None] * R[:, :, 1] - s[:, None] * R[:, :, 0]
            z = R[:, :, 2]
            o = o + dz * z + a * x
            R = torch.stack([x, ca * y + sa * z, ca * z - sa * y], 2)
            origins.append(o)
        O = torch.stack(origins, 1)
        L = torch.tensor(self.link, device=q.device)
        return O[:, L - 1] + self.t[None, :, None] * (O[:, L] - O[:, L - 1])

    def hit(self, q):
        """Collision of configurations q [n][d]."""
        out = torch.zeros(q.shape[0], device=q.device, dtype=torch.bool)
        for lo in range(0, q.shape[0], 1 << 18):
            x = q[lo:lo + (1 << 18)]
            if self.arm:
                p, r = self._centres(x), self.r
            else:
                p, r = x[:, None, :], torch.zeros(1, device=q.device, dtype=torch.float64)
            d = p.shape[2]
            h = torch.zeros(p.shape[:2], device=q.device, dtype=torch.bool)
            for o in self.sph:
                h |= (p - o[:d]).square().sum(2) <= (o[d] + r) ** 2
            for o in self.box:
                h |= ((p - o[:d]).abs() - o[d:]).clamp(min=0).square().sum(2) <= r ** 2
            out[lo:lo + (1 << 18)] = h.any(1)
        return out


def _lengths(x, y):
    return torch.cdist(x, y, compute_mode="donot_use_mm_for_euclid_dist")


def _states(H):
    """Interior states of an edge, the middle ones first."""
    return sorted(range(1, H - 1), key=lambda h: (-(h & -h), abs(2 * h - (H - 1))))


def _slice(ex, x, y, cx, cy, H, penalty):
    """Costs of the edges x -> y whose end points collide as cx, cy say."""
    C = _lengths(x, y)
    fail = cx[:, None] | cy[None, :]
    left = torch.nonzero(~fail.reshape(-1)).reshape(-1)
    n = y.shape[0]
    for h in _states(H):
        keep = []
        for part in left.split(1 << 22):
            u, v = x[part // n], y[part % n]
            bad = ex.hit(u + (h / (H - 1)) * (v - u))
            fail.view(-1)[part[bad]] = True
            keep.append(part[~bad])
        left = torch.cat(keep) if keep else left
    return C + penalty * fail


def _exact_plan(case, seed):
    w = _workload(case, seed)
    ex = _Exact(w)
    Q64 = _samples(w)
    Q = Q64.float().double()  # the edges run between the stored samples
    q0 = torch.from_numpy(w["q0"]).double().cuda().reshape(1, -1)
    goals = torch.from_numpy(w["goals"]).double().cuda()
    cq, c0, cg = [ex.hit(q) for q in Q], ex.hit(q0), ex.hit(goals)
    M, H, P = w["M"], w["H"], w["penalty"]
    C_s = _slice(ex, q0, Q[0], c0, cq[0], H, P).reshape(-1)
    C_h = [_slice(ex, Q[m], Q[m + 1], cq[m], cq[m + 1], H, P) for m in range(M - 1)]
    C_l = _slice(ex, Q[M - 1], goals, cq[M - 1], cg, H, P)
    V, A = [None] * M, [None] * M
    V[M - 1], A[M - 1] = C_l.min(1)
    for m in range(M - 2, -1, -1):
        V[m], A[m] = (C_h[m] + V[m + 1][None, :]).min(1)
    V_s, a_s = (C_s + V[0]).min(0)
    at, wp = int(a_s), [q0[0]]
    for m in range(M):
        wp.append(Q[m, at])
        at = int(A[m][at])
    wp.append(goals[at])
    one = V_s.reshape(1)
    if case["kind"] == "lazy":  # which edges a round checks has no 64-bit value
        return dict(Q=Q64, V_s=one, wp=torch.stack(wp), cost=one)
    return dict(Q=Q64, C_s=C_s, C_h=torch.stack(C_h), C_l=C_l, V=torch.stack(V), V_s=one, wp=torch.stack(wp), cost=one)


def _exact_net(P, Bf, q):
    """Features and logits of configurations q in 64 bits, with the activations."""
    x = q / math.pi
    ph = 2 * math.pi * x @ torch.from_numpy(Bf).double().cuda().T
    f = torch.zeros((q.shape[0], 64), device="cuda", dtype=torch.float64)
    d, k = x.shape[1], ph.shape[1]
    f[:, :d], f[:, d:d + k], f[:, d + k:d + 2 * k] = x, torch.sin(ph), torch.cos(ph)
    acts = [f]
    for l in range(1, 5):
        acts.append(torch.relu(acts[-1] @ P[f"W{l}"].T + P[f"b{l}"]))
    return acts, acts[-1] @ P["w5"] + P["b5"]


def _exact_params(seed, d):
    P, Bf = wl.surrogate_init(seed, d)
    return {k: torch.from_numpy(v).double().cuda() for k, v in P.items()}, Bf


def _exact_train(case, seed):
    w, X = _train_inputs(case, seed)
    P, Bf = _exact_params(seed, w["d"])
    y = _Exact(w).hit(X.double()).double()
    for p in P.values():
        p.requires_grad_()
    _, z = _exact_net(P, Bf, X.double())
    loss = torch.nn.functional.binary_cross_entropy_with_logits(z, y)
    order = ["W1", "b1", "W2", "b2", "W3", "b3", "W4", "b4", "w5", "b5"]
    grads = torch.autograd.grad(loss, [P[k] for k in order])
    g = torch.cat([x.reshape(-1) for x in grads])
    p = torch.cat([P[k].detach().reshape(-1) for k in order])
    S = wl.SURROGATE  # the first Adam step: both moments hold this gradient alone
    return dict(loss=loss.detach().reshape(1), grad=g, params=p - S["lr"] * g / (g.abs() + S["eps"]))


def _exact_prune(case, seed):
    w = _workload(dict(case, workload="arm7", H=16), seed)
    P, Bf = _exact_params(seed, w["d"])
    ex, Q = _Exact(w), _samples(w).float().double()
    layers = [torch.from_numpy(w["q0"]).double().cuda().reshape(1, -1), *Q, torch.from_numpy(w["goals"]).double().cuda()]
    coll = [ex.hit(q) for q in layers]
    coll[0][:], coll[-1][:] = False, False
    out = []
    for x, y, cx, cy in zip(layers, layers[1:], coll, coll[1:]):
        z = torch.full((x.shape[0] * y.shape[0],), math.nan, device="cuda", dtype=torch.float64)
        for part in torch.nonzero(~(cx[:, None] | cy[None, :]).reshape(-1)).reshape(-1).split(1 << 20):
            mid = (x[part // y.shape[0]] + y[part % y.shape[0]]) / 2
            z[part] = _exact_net(P, Bf, mid)[1]
        out.append(z)
    return dict(logits=torch.cat(out))


def exact(case, seed):
    if case["kind"] in ("plan", "lazy"):
        return _exact_plan(case, seed)
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] == "prune":
        return _exact_prune(case, seed)
    # the loops (anytime, batch, classes) and RRT-Connect are defined by 32-bit
    # decisions from stage to stage: a 64-bit run takes another course
    return None
