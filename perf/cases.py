"""Measured cases of the PI^2-RH library: the calls its users make, over the
range of sizes they make them in.

Every case is a plain dict; ``listed()`` gives the fixed ones, ``draw(rng)``
one more of the same ranges, ``prepare(case, seed)`` the problem, the model
and whatever a program keeps between calls, ``run(state)`` one pass through
the public entry points, ``work(case)`` the bytes and operations the pass
cannot do without, and ``exact(case, seed)`` the same results in plain torch
float64 (the random stream's counters and uniforms are exact in every
precision, so it draws the same noise).

Kinds of case
  step     one receding-horizon control step (rollouts, updates, plant step)
           of a controller that receives its measured state before each step
  iterate  one path-integral iteration without a graph: rollouts and update
  rollout  the sampled rollouts alone
  update   the control update alone, from given costs
  predict  the LWPR mixture at a set of inputs
  adjoint  expected cost and its gradients through torch.autograd
  batch    one control step of several uneven controllers in one launch

Float32 rollouts use the smooth obstacle cost of the flight experiments: with
the indicator a state within rounding of an obstacle's surface changes its
cost by the whole penalty.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1503_00330_amd as pi
from paper_1503_00330_amd.autograd import PI2RHAdjoint
from paper_1503_00330_amd.rh import RHController

# dynamics -> code, states, controls, outputs, LWPR inputs
_DYN = {"pointmass": (pi.PI_DYN_POINTMASS2D, 4, 2, 2, 6),
        "quad": (pi.PI_DYN_QUAD12, 12, 4, 6, 16),
        "hybrid": (pi.PI_DYN_QUAD_HYBRID, 9, 4, 3, 4)}
_VARIANT = {"auto": pi.PI_VARIANT_AUTO, "f16x2": pi.PI_VARIANT_MFMA_F16X2, "bf16x3": pi.PI_VARIANT_MFMA_BF16X3}
_NP = {"f32": np.float32, "f64": np.float64}
_TORCH = {"f32": torch.float32, "f64": torch.float64}
_DT = float(np.float32(0.02))     # a step that float32 and float64 hold alike
_RATE_GAIN = 25.0                 # attitude-rate response of the hybrid quadrotor
_LAMBDA = 1.0


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest controller: a planar point mass in float64, the precision
        # a user checks a task in; launches and the serial chain count
        dict(name="step_pointmass_f64", kind="step", dyn="pointmass", dtype="f64", variant="auto",
             K=256, T=20, M=1, L="16-16", R=2, n_obs=3, iterations=1),
        # the paper's own model at its timing shape, mean prediction only: an
        # eager iteration, where every host call is paid
        dict(name="iterate_paper_mean", kind="iterate", dyn="hybrid", dtype="f32", variant="auto",
             K=1000, T=50, M=0, L="15-15-24", R=2, n_obs=3),
        # the paper's largest sub-rollout count: one 50 Hz control step
        dict(name="step_paper_sub32", kind="step", dyn="hybrid", dtype="f32", variant="auto",
             K=950, T=50, M=32, L="15-15-24", R=2, n_obs=3, iterations=1),
        # the 12-state quadrotor at an ordinary rollout count, fp16 pieces
        dict(name="rollout_quad_2048", kind="rollout", dyn="quad", dtype="f32", variant="f16x2",
             K=2048, T=100, M=1, L="x256", R=4, n_obs=20, folded=True),
        # what the library picks by itself for a ragged problem: odd counts,
        # uneven outputs, sub-rollouts, a model that changes between calls
        dict(name="rollout_quad_ragged", kind="rollout", dyn="quad", dtype="f32", variant="auto",
             K=777, T=61, M=3, L="131-96-250-33-177-301", R=4, n_obs=13, folded=False),
        # more rollouts than tiles for every compute unit, library's choice
        dict(name="rollout_quad_16384", kind="rollout", dyn="quad", dtype="f32", variant="auto",
             K=16384, T=100, M=1, L="x256", R=4, n_obs=20, folded=True),
        # the largest single problem: the headline workload's rollouts
        dict(name="rollout_quad_65536", kind="rollout", dyn="quad", dtype="f32", variant="f16x2",
             K=65536, T=200, M=1, L="x1024", R=4, n_obs=20, folded=True),
        # the update of that workload by itself
        dict(name="update_65536", kind="update", dyn="quad", dtype="f32", K=65536, T=200, weighting=0),
        # a few queries of a model that has just been refitted (no fold kept)
        dict(name="predict_small", kind="predict", d=6, n_out=2, dtype="f32", N=33, L="16-16", R=2, folded=False),
        # validation of a learned model over a log of flights
        dict(name="predict_log", kind="predict", d=16, n_out=6, dtype="f32", N=100003, L="x256", R=4, folded=True),
        # gradient of the expected cost (controls, centres, metrics)
        dict(name="adjoint_quad_8192", kind="adjoint", dyn="quad", dtype="f32", variant="auto",
             K=8192, T=100, M=1, L="x256", R=4, n_obs=20, ckpt=20),
        # a fleet of uneven controllers in one launch
        dict(name="batch_16", kind="batch", dyn="quad", dtype="f32", variant="f16x2", B=16, K_lo=512, K_hi=16384,
             T_lo=50, T_hi=120, L_lo=64, L_hi=1024, R=4, sizes=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "iterate", "rollout", "rollout", "rollout", "update", "predict", "adjoint", "batch"])
    if kind in ("step", "iterate"):
        dyn = rng.choice(["pointmass", "hybrid"])
        c = dict(kind=kind, dyn=dyn, dtype=rng.choice(["f32", "f64"]), variant="auto", K=_log(rng, 200, 3000),
                 T=_log(rng, 10, 60), M=rng.choice([0, 1, 1, 4, 8, 16]), R=2, n_obs=rng.randint(0, 6),
                 L="-".join(str(rng.randint(9, 40)) for _ in range(_DYN[dyn][3])))
        if kind == "step":
            c["iterations"] = rng.choice([1, 2])
        return c
    if kind == "rollout":
        return dict(kind=kind, dyn="quad", dtype="f32", variant=rng.choice(["auto", "f16x2", "f16x2", "bf16x3"]),
                    K=_log(rng, 300, 40000), T=_log(rng, 20, 110), M=rng.choice([0, 1, 1, 1, 2]),
                    L="-".join(str(_log(rng, 60, 600)) for _ in range(6)), R=4, n_obs=rng.randint(3, 40),
                    folded=rng.random() < 0.7)
    if kind == "update":
        dyn = rng.choice(["pointmass", "hybrid", "quad"])
        return dict(kind=kind, dyn=dyn, dtype=rng.choice(["f32", "f32", "f64"]), K=_log(rng, 200, 65536),
                    T=_log(rng, 10, 200), weighting=rng.choice([0, 0, 1]))
    if kind == "predict":
        d = rng.choice([4, 6, 16, 16])
        n_out = {4: 3, 6: 2, 16: 6}[d]
        return dict(kind=kind, d=d, n_out=n_out, dtype=rng.choice(["f32", "f32", "f64"]), N=_log(rng, 1, 60000),
                    L="-".join(str(_log(rng, 9, 400)) for _ in range(n_out)), R=4, folded=rng.random() < 0.5)
    if kind == "adjoint":
        return dict(kind=kind, dyn="quad", dtype="f32", variant=rng.choice(["auto", "auto", "f16x2"]),
                    K=_log(rng, 200, 8192), T=_log(rng, 15, 100), M=1, R=4, n_obs=rng.randint(3, 30),
                    L="-".join(str(_log(rng, 60, 300)) for _ in range(6)), ckpt=rng.choice([0, 10, 20]))
    return dict(kind="batch", dyn="quad", dtype="f32", variant=rng.choice(["auto", "f16x2"]), B=rng.randint(2, 12),
                K_lo=300, K_hi=_log(rng, 2000, 8000), T_lo=20, T_hi=rng.randint(30, 100), L_lo=60, L_hi=500, R=4,
                sizes=rng.randint(0, 1 << 20))


def _models(case):
    """Local models of every output."""
    n_out = case["n_out"] if "n_out" in case else _DYN[case["dyn"]][3]
    return [int(case["L"][1:])] * n_out if case["L"].startswith("x") else [int(v) for v in case["L"].split("-")]


def _batch_cases(case):
    """The single problems of a batch."""
    r = np.random.Generator(np.random.PCG64(case["sizes"]))
    out = []
    for b in range(case["B"]):
        K, T = int(r.integers(case["K_lo"], case["K_hi"] + 1)), int(r.integers(case["T_lo"], case["T_hi"] + 1))
        L, n_obs = int(r.integers(case["L_lo"], case["L_hi"] + 1)), int(r.integers(10, 41))
        out.append(dict(dyn=case["dyn"], dtype=case["dtype"], variant=case["variant"], K=K, T=T, M=1, L="x%d" % L,
                        R=case["R"], n_obs=n_obs))
    return out


# ---------------------------------------------------------------- inputs
def _model(rng, d, Ls, R, dtype):
    """LWPR mixtures: centres over the unit box, metrics A A^T + I/2, random
    projection directions, unit-variance regression coefficients."""
    Lt = sum(Ls)
    centre = rng.uniform(-1.0, 1.0, (Lt, d))
    A = rng.normal(0.0, 0.3, (Lt, d, d))
    metric = A @ np.transpose(A, (0, 2, 1)) + 0.5 * np.eye(d)
    metric = 0.5 * (metric + np.transpose(metric, (0, 2, 1)))
    u = rng.standard_normal((Lt, R, d))
    u /= np.linalg.norm(u, axis=-1, keepdims=True)
    t = _NP[dtype]
    return SimpleNamespace(d=d, n_out=len(Ls), R=R, L_off=np.concatenate([[0], np.cumsum(Ls)]), centre=centre.astype(t),
                           metric=metric.astype(t), proj_u=u.astype(t), proj_p=None,
                           beta=rng.standard_normal((Lt, R + 1)).astype(t),
                           sigma2=(rng.uniform(0.01, 0.1, Lt) ** 2).astype(t))


def _problem(rng, case, problem_id=0):
    code, n_x, n_u, _, _ = _DYN[case["dyn"]]
    t, npos = _NP[case["dtype"]], 2 if case["dyn"] == "pointmass" else 3
    f = lambda v: v.astype(np.float32).astype(np.float64)     # values that both precisions hold
    x0, goal = np.zeros(n_x), np.zeros(3)
    x0[:npos] = rng.uniform(-1.0, 1.0, npos)
    goal[:npos] = rng.uniform(-1.0, 1.0, npos)
    obs = np.full((case.get("n_obs", 0), 3), 0.2)
    obs[:, :2] = rng.uniform(-1.0, 1.0, (obs.shape[0], 2))
    quad = case["dyn"] != "pointmass"
    return SimpleNamespace(
        dyn=code, K=case["K"], T=case["T"], M=case.get("M", 1), dt=_DT, lam=_LAMBDA, noise_std=np.full(n_u, 0.5),
        goal=f(goal), w_pos=np.array([1.0, 1.0, 10.0 if quad else 0.0]), w_ang=float(np.float32(0.2)) * quad,
        w_vel=float(np.float32(0.1)) * quad, obs_kind=pi.PI_OBS_SMOOTH, obs=f(obs), obs_penalty=100.0, obs_decay=10.0,
        weighting=case.get("weighting", pi.PI_W_COST_TO_GO), seed=int(rng.integers(1 << 62)), problem_id=problem_id,
        x0=x0.astype(t), u_nom=rng.normal(0.0, 0.2, (case["T"], n_u)).astype(t), ctrl_cost=0,
        iter=int(rng.integers(1000)))


def _host(case, seed, b=0):
    rng = np.random.Generator(np.random.PCG64([seed, b]))
    prob = _problem(rng, case, b)
    model = _model(rng, _DYN[case["dyn"]][4], _models(case), case["R"], case["dtype"]) if "L" in case else None
    return prob, model


def _device(prob, model, case):
    dp = pi.DeviceProblem(prob, variant=_VARIANT[case.get("variant", "auto")])
    dp.iter.fill_(prob.iter)
    return dp, pi.DeviceModel(model) if model is not None else None


def _predict_host(case, seed):
    rng = np.random.Generator(np.random.PCG64([seed, 0]))
    model = _model(rng, case["d"], _models(case), case["R"], case["dtype"])
    return model, rng.uniform(-1.0, 1.0, (case["N"], case["d"])).astype(_NP[case["dtype"]])


def _update_costs(case, prob, seed):
    """Step costs of K rollouts: a slow drift of every rollout about a common
    level, non-negative, with the spread of total costs a controller sees."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    kw = dict(generator=g, device="cuda", dtype=torch.float64)
    K, T = case["K"], case["T"]
    drift = torch.cumsum(torch.randn((K, T), **kw), dim=1) / math.sqrt(T)
    return (_DT * (2.0 + drift + 0.3 * torch.randn((K, T), **kw)).abs()).to(_TORCH[case["dtype"]])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "predict":
        model, Z = _predict_host(case, seed)
        dm = pi.DeviceModel(model)
        return dict(kind=kind, dm=dm.fold() if case["folded"] else dm, Z=torch.as_tensor(Z, device="cuda"))
    if kind == "batch":
        ps, ms = zip(*(_device(*_host(c, seed, b), c) for b, c in enumerate(_batch_cases(case))))
        for p in ps:
            p.tile_waves = 8 if case["variant"] == "f16x2" else 0     # the launch tuned for such a fleet
        for m in ms:
            m.fold()
        return dict(kind=kind, br=pi.BatchedRollout(ps, ms), x0=[p.x0 for p in ps],
                    measured=[p.x0.clone() for p in ps], u_nom=[p.u_nom for p in ps])
    prob, model = _host(case, seed)
    dp, dm = _device(prob, model, case)
    if kind == "update":
        return dict(kind=kind, dp=dp, cost=_update_costs(case, prob, seed))
    if kind == "step":
        ctl = RHController(dp, dm, iterations=case["iterations"], graph=True)
        ctl.capture()
        return dict(kind=kind, ctl=ctl, dp=dp, measured=dp.x0.clone())
    if kind == "adjoint":
        leaf = lambda t: t.clone().requires_grad_(True)
        return dict(kind=kind, dp=dp, dm=dm, ckpt=case["ckpt"], leaves=(leaf(dp.u_nom), leaf(dm.centre), leaf(dm.metric)))
    if case.get("folded", True):
        dm.fold()
    return dict(kind=kind, dp=dp, dm=dm, cost=torch.empty((dp.K, dp.T), dtype=dp.dtype, device="cuda"))


def run(state):
    kind = state["kind"]
    if kind == "rollout":
        return pi.rollout_cost(state["dp"], state["dm"], out=state["cost"])
    if kind == "predict":
        return pi.lwpr_predict(state["dm"], state["Z"])
    if kind == "update":
        return pi.update(state["dp"], state["cost"])[0]
    if kind == "iterate":
        pi.iteration(state["dp"], state["dm"], state["cost"])
        return state["cost"], state["dp"].u_nom
    if kind == "step":
        state["dp"].x0.copy_(state["measured"])
        state["ctl"].step()
        return state["ctl"].cost, state["dp"].u_nom, state["dp"].x0
    if kind == "adjoint":
        J = PI2RHAdjoint.apply(*state["leaves"], state["dp"], state["dm"], state["ckpt"])
        # J is summed in double from float32 costs: its precision is float32's
        return (J.detach().float(),) + torch.autograd.grad(J, state["leaves"])
    torch._foreach_copy_(state["x0"], state["measured"])
    state["br"].control_step()
    return state["br"].costs, state["u_nom"], state["x0"]


# ---------------------------------------------------------------- work
def _item(case):
    return 4 if case["dtype"] == "f32" else 8


def _model_bytes(case, d):
    return sum(_models(case)) * (d + d * d + case["R"] * d + case["R"] + 2) * _item(case)


def work(case):
    kind = case["kind"]
    if kind == "predict":
        d, N = case["d"], case["N"]
        return {"bytes": N * (d + 2 * case["n_out"]) * _item(case) + _model_bytes(case, d),
                "flops": N * sum(_models(case)) * (d * d + 5 * d + 8)}
    if kind == "batch":
        ws = [work(dict(c, kind="step", iterations=1)) for c in _batch_cases(case)]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    _, n_x, n_u, n_out, d = _DYN[case["dyn"]]
    K, T = case["K"], case["T"]
    plan = (n_x + 2 * T * n_u) * _item(case)
    # per rollout and step of the update: the running sum, the weight, n_u weighted sums
    upd = {"bytes": K * T * _item(case) + plan, "flops": K * T * (5 + 2 * n_u)}
    if kind == "update":
        return upd
    evals = K * max(case["M"], 1) * T
    roll = {"bytes": K * T * _item(case) + _model_bytes(case, d) + plan,
            "flops": evals * sum(_models(case)) * (d * d + 5 * d + 8)}
    if kind == "adjoint":
        # per evaluation, output and model, beyond the forward: the state's
        # gradient ((D + D^T) dl and b, scaled) and the parameters' (dl dl^T, dl)
        back = evals * sum(_models(case)) * (2 * d * d + 8 * d + 10)
        return {"bytes": 2 * _model_bytes(case, d) + plan, "flops": roll["flops"] + back}
    n = case.get("iterations", 1) if kind != "rollout" else 1
    if kind == "rollout":
        return roll
    return {"bytes": n * (roll["bytes"] + upd["bytes"]), "flops": n * (roll["flops"] + upd["flops"])}


# ---------------------------------------------------------------- float64
_M32 = 0xFFFFFFFF


def _mulhilo(m, c):
    """High and low words of the 64-bit product of 32-bit m and tensor c."""
    mh, ml, ch, cl = m >> 16, m & 0xFFFF, c >> 16, c & 0xFFFF
    low = ml * cl
    mid = mh * cl + (low >> 16)
    mid2 = ml * ch + (mid & 0xFFFF)
    return (mh * ch + (mid >> 16) + (mid2 >> 16)) & _M32, ((mid2 << 16) | (low & 0xFFFF)) & _M32


def _normals(seed, tag, pid, it, k, m, t, n):
    """n standard normals of draw (tag, k, m, t), float64: Philox4x32-10, exact
    23-bit uniforms, Box-Muller pairs.  k, m, t broadcast (int64 tensors)."""
    out = []
    shape = torch.broadcast_shapes(k.shape, m.shape, t.shape)
    for blk in range((n + 3) // 4):
        c = [t.expand(shape), k.expand(shape), (m.expand(shape) << 4) | blk,
             torch.full(shape, (tag << 30) | ((pid & 0x3FF) << 20) | (it & 0xFFFFF), dtype=torch.int64, device="cuda")]
        k0, k1 = seed & _M32, (seed >> 32) & _M32
        for _ in range(10):
            h0, l0 = _mulhilo(0xD2511F53, c[0])
            h1, l1 = _mulhilo(0xCD9E8D57, c[2])
            c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
            k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
        u = [((v >> 9).double() + 0.5) / 8388608.0 for v in c]
        for a, b in ((0, 1), (2, 3)):
            rad = torch.sqrt(-2.0 * torch.log(u[a]))
            out += [rad * torch.cos(2 * math.pi * u[b]), rad * torch.sin(2 * math.pi * u[b])]
    return torch.stack(out[:n], dim=-1)


class _Mixture:
    """Eq. (1) in float64: means and variances of every output at inputs z."""

    def __init__(self, model, centre=None, metric=None):
        dd = lambda a: torch.as_tensor(np.asarray(a), device="cuda").double()
        c = dd(model.centre) if centre is None else centre
        D = dd(model.metric) if metric is None else metric
        U, beta = dd(model.proj_u), dd(model.beta)
        b = torch.zeros_like(U[:, 0])
        for r in range(model.R - 1, -1, -1):      # p = u
            b = b + (beta[:, r + 1] - (U[:, r] * b).sum(1))[:, None] * U[:, r]
        d = model.d
        self.ia, self.ib = torch.triu_indices(d, d, device="cuda")
        S = D + D.transpose(1, 2)
        th = S[:, self.ia, self.ib] * torch.where(self.ia == self.ib, 0.5, 1.0)
        h = (S @ c[:, :, None])[:, :, 0]
        self.Wq = torch.cat([th, -h, 0.5 * (h * c).sum(1, keepdim=True)], 1) * -0.5
        self.Wy = torch.cat([b, (beta[:, 0] - (b * c).sum(1))[:, None]], 1)
        self.s2, self.off = dd(model.sigma2), [int(v) for v in model.L_off]

    def __call__(self, z):
        one = torch.ones_like(z[:, :1])
        fq, fy = torch.cat([z[:, self.ia] * z[:, self.ib], z, one], 1), torch.cat([z, one], 1)
        mu, var = [], []
        for lo, hi in zip(self.off[:-1], self.off[1:]):
            w = torch.softmax(fq @ self.Wq[lo:hi].t(), dim=1)
            y = fy @ self.Wy[lo:hi].t()
            m = (w * y).sum(1, keepdim=True)
            mu.append(m[:, 0])
            var.append((w * ((y - m) ** 2 + self.s2[lo:hi])).sum(1))
        return torch.stack(mu, 1), torch.stack(var, 1)


def _euler(dyn, x, acc, u):
    if dyn == "pointmass":
        return torch.cat([x[:, :2] + _DT * x[:, 2:], x[:, 2:] + _DT * acc], 1)
    p, v = x[:, :3] + _DT * x[:, 3:6], x[:, 3:6] + _DT * acc[:, :3]
    if dyn == "hybrid":
        return torch.cat([p, v, x[:, 6:9] + _DT * (_RATE_GAIN * (u[:, :3] - x[:, 6:9]))], 1)
    return torch.cat([p, v, x[:, 6:9] + _DT * x[:, 9:12], x[:, 9:12] + _DT * acc[:, 3:]], 1)


def _step_cost(dyn, prob, x):
    n = 2 if dyn == "pointmass" else 3
    dd = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float64), device="cuda")
    c = ((x[:, :n] - dd(prob.goal)[:n]) ** 2 * dd(prob.w_pos)[:n]).sum(1) + prob.w_vel * (x[:, n:2 * n] ** 2).sum(1)
    if dyn != "pointmass":
        c = c + prob.w_ang * (x[:, 6:9] ** 2).sum(1)
    for ox, oy, _ in prob.obs:
        c = c + prob.obs_penalty * torch.exp(-prob.obs_decay * ((x[:, 0] - ox) ** 2 + (x[:, 1] - oy) ** 2))
    return _DT * c


def _z(dyn, x, u):
    return torch.cat([x[:, 6:9], u[:, 3:]], 1) if dyn == "hybrid" else torch.cat([x, u], 1)


def _exact_costs(case, prob, mix, x0, u_nom, it, ks=None):
    """cbar [len(ks)][T] of the sampled rollouts ks (default all)."""
    dyn, Ms = case["dyn"], max(prob.M, 1)
    _, n_x, n_u, n_out, _ = _DYN[dyn]
    ks = torch.arange(prob.K, device="cuda") if ks is None else ks
    k, m = ks.repeat_interleave(Ms), torch.arange(Ms, device="cuda").repeat(len(ks))
    x, cost = x0.expand(len(k), n_x), []
    for t in range(prob.T):
        tt = torch.tensor([t], device="cuda")
        eps = 0.5 * _normals(prob.seed, 0, prob.problem_id, it, k, torch.zeros_like(m), tt, n_u)
        u = u_nom[t] + eps
        acc, var = mix(_z(dyn, x, u))
        if prob.M > 0:
            acc = acc + torch.sqrt(var) * _normals(prob.seed, 1, prob.problem_id, it, k, m, tt, n_out)
        x = _euler(dyn, x, acc, u)
        cost.append(_step_cost(dyn, prob, x).reshape(len(ks), Ms).mean(1))
    return torch.stack(cost, 1)


def _exact_update(case, prob, cost, u_nom, it):
    S = cost.flip(1).cumsum(1).flip(1) if prob.weighting == pi.PI_W_COST_TO_GO else \
        cost.sum(1, keepdim=True).expand(cost.shape)
    P = torch.softmax(-S / _LAMBDA, dim=0)
    n_u, du = _DYN[case["dyn"]][2], []
    k, zero = torch.arange(prob.K, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
    for t in range(prob.T):
        eps = 0.5 * _normals(prob.seed, 0, prob.problem_id, it, k, zero, zero + t, n_u)
        du.append((P[:, t:t + 1] * eps).sum(0))
    return u_nom + torch.stack(du)


def _exact_step(case, prob, mix, iterations, shift):
    dyn = case["dyn"]
    x0, u = (torch.as_tensor(a, device="cuda").double() for a in (prob.x0, prob.u_nom))
    it = prob.iter
    for _ in range(iterations):
        cost = _exact_costs(case, prob, mix, x0, u, it)
        u = _exact_update(case, prob, cost, u, it)
        it += 1
    if not shift:
        return cost, u
    zero = torch.zeros(1, dtype=torch.int64, device="cuda")
    mu, var = mix(_z(dyn, x0[None], u[:1]))
    xi = _normals(prob.seed, 2, prob.problem_id, it, zero, zero, zero, mu.shape[1])
    x = _euler(dyn, x0[None], mu + torch.sqrt(var) * xi, u[:1])[0]
    return cost, torch.cat([u[1:], u[-1:]]), x


def _exact_adjoint(case, prob, model):
    dd = lambda a: torch.as_tensor(a, device="cuda").double().requires_grad_(True)
    leaves = u, c, D = dd(prob.u_nom), dd(model.centre), dd(model.metric)
    x0 = torch.as_tensor(prob.x0, device="cuda").double()
    J, step = torch.zeros((), dtype=torch.float64, device="cuda"), 1024
    for k0 in range(0, prob.K, step):
        ks = torch.arange(k0, min(prob.K, k0 + step), device="cuda")
        part = _exact_costs(case, prob, _Mixture(model, c, D), x0, u, prob.iter, ks).sum() / prob.K
        part.backward()
        J = J + part.detach()
    return (J,) + tuple(v.grad for v in leaves)


def exact(case, seed):
    kind = case["kind"]
    if kind == "predict":
        model, Z = _predict_host(case, seed)
        mix, Z = _Mixture(model), torch.as_tensor(Z, device="cuda").double()
        parts = [mix(z) for z in Z.split(32768)]
        return tuple(torch.cat(p) for p in zip(*parts))
    if kind == "batch":
        costs, us, xs = [], [], []
        for b, c in enumerate(_batch_cases(case)):
            prob, model = _host(c, seed, b)
            cost, u, x = _exact_step(c, prob, _Mixture(model), 1, True)
            costs.append(cost), us.append(u), xs.append(x)
        return costs, us, xs
    prob, model = _host(case, seed)
    if kind == "update":
        u = torch.as_tensor(prob.u_nom, device="cuda").double()
        return _exact_update(case, prob, _update_costs(case, prob, seed).double(), u, prob.iter)
    if kind == "adjoint":
        return _exact_adjoint(case, prob, model)
    mix = _Mixture(model)
    if kind == "rollout":
        x0, u = (torch.as_tensor(a, device="cuda").double() for a in (prob.x0, prob.u_nom))
        return _exact_costs(case, prob, mix, x0, u, prob.iter)
    return _exact_step(case, prob, mix, case.get("iterations", 1), kind == "step")
