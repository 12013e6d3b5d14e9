"""Performance cases of the framework: what its users run, through its public entry points.

    listed()             the named cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  the inputs, handles and weights a program holds before the call
    run(state)           one pass
    work(case)           bytes and operations that one pass cannot do without
    tolerance(case)      how far two correct implementations may be apart
    exact(case, seed)    the pass in 64-bit torch arithmetic (bf16 rounding where the interface
                         in include/auv.h defines it), without the framework's code

Kinds of case: `step` (one control step per call), `rollout` (many steps per launch, the
caller keeps rewards and batch statistics), `collect` (sampled rollout with value head, every
record kept, then advantages: one PPO data collection), `gae`, `forward` (a network alone),
`ppo` (one update of policy and value net), `shac` (one window's actor gradient and step, and
with `critic` the value regression on it) and `critic` (that regression alone).
"""
import math

import numpy as np
import torch

import workloads as W
from paper_2512_13359_amd import AuvEnv, PpoLearner, ShacLearner, upload_mlp
from paper_2512_13359_amd import _abi as A

DEV = "cuda" if torch.cuda.is_available() else "cpu"
EXTERNAL, RANDOM, MEAN, SAMPLE = 0, 1, 2, 3
GAMMA, LAM = 0.99, 0.95


def listed():
    return [
        # a controller in the loop of another program: one policy step of a handful of vehicles
        dict(name="step_policy_64", kind="step", n=64, mode=MEAN, substeps=4, lissajous=True, stats=False),
        # an outside learner stepping the batch with its own actions, gym style
        dict(name="step_external_4096", kind="step", n=4096, mode=EXTERNAL, substeps=1, lissajous=False, stats=True),
        # open-loop exploration at the c2 workload's size, an odd batch
        dict(name="rollout_random_4001", kind="rollout", n=4001, T=200, mode=RANDOM, substeps=1, lissajous=False),
        # the headline rollout (c4): one 64-environment workgroup per CU, four RK4 substeps
        dict(name="rollout_policy_16384", kind="rollout", n=16384, T=24, mode=MEAN, substeps=4, lissajous=True),
        # PPO data collection at the c5 workload's width
        dict(name="collect_65536", kind="collect", n=65536, T=16, substeps=1, paper=False),
        # PPO data collection on the paper's task at its training width
        dict(name="collect_paper_4096", kind="collect", n=4096, T=24, substeps=2, paper=True),
        # advantages over whole long episodes (the c3 workload's length)
        dict(name="gae_4096x1000", kind="gae", n=4096, T=1000),
        # values of a ragged batch of observations
        dict(name="forward_value_20011", kind="forward", n=20011, n_out=1),
        # an update on a small ragged minibatch of the paper task (six actions)
        dict(name="ppo_3000", kind="ppo", B=3000, M=65536, n_act=6),
        # the update of the c5 buffer's sixteenth
        dict(name="ppo_262144", kind="ppo", B=262144, M=4194304, n_act=8),
        # SHAC at the paper's main scale: the actor's window and step
        dict(name="shac_window_4096x32", kind="shac", n=4096, h=32, mode=SAMPLE, substeps=2, box=False, critic=False),
        # and the critic's regression on such a window
        dict(name="shac_critic_4096x32", kind="critic", n=4096, h=32, iterations=16, batches=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Control steps of a closed-loop case, by substeps.  A bf16 rounding that falls the other way moves the trajectory
# that follows, so over a long horizon two correct runs part; this many steps are about 1.2 seconds of motion.
LOOP_STEPS = {1: 64, 2: 24, 4: 24}


def draw(rng):
    kind = rng.choice(["step", "rollout", "rollout", "collect", "gae", "forward", "ppo", "ppo", "shac", "critic"])
    if kind == "step":
        return dict(kind=kind, n=_log(rng, 1, 32768), mode=rng.choice([EXTERNAL, RANDOM, MEAN, SAMPLE]),
                    substeps=rng.choice([1, 2, 4]), lissajous=rng.random() < 0.5, stats=rng.random() < 0.5)
    if kind == "rollout":
        n, mode, sub = _log(rng, 16, 65536), rng.choice([RANDOM, MEAN, MEAN, SAMPLE]), rng.choice([1, 2, 4])
        most = 400 if mode == RANDOM else LOOP_STEPS[sub]
        return dict(kind=kind, n=n, T=_log(rng, 8, max(9, min(most, 1638400 // n))), mode=mode, substeps=sub,
                    lissajous=rng.random() < 0.5)
    if kind == "collect":
        n, sub = _log(rng, 256, 65536), rng.choice([1, 2, 4])
        return dict(kind=kind, n=n, T=_log(rng, 8, max(9, min(LOOP_STEPS[sub], 1048576 // n))), substeps=sub,
                    paper=rng.random() < 0.5)
    if kind == "gae":
        n = _log(rng, 16, 65536)
        return dict(kind=kind, n=n, T=_log(rng, 4, max(5, min(4000, 8388608 // n))))
    if kind == "forward":
        return dict(kind=kind, n=_log(rng, 16, 1 << 20), n_out=rng.choice([1, 8]))
    if kind == "ppo":
        B = _log(rng, 64, 262144)
        return dict(kind=kind, B=B, M=_log(rng, B + 16, min(4194304, 32 * B)), n_act=rng.choice([6, 8]))
    if kind == "shac":
        return dict(kind=kind, n=_log(rng, 16, 4096), h=_log(rng, 4, 32), mode=rng.choice([MEAN, SAMPLE, SAMPLE]),
                    substeps=rng.choice([1, 2, 4]), box=rng.random() < 0.3, critic=rng.random() < 0.7)
    return dict(kind=kind, n=_log(rng, 64, 4096), h=_log(rng, 4, 32), iterations=_log(rng, 1, 8), batches=rng.choice([1, 2, 4, 8]))


# ---------------------------------------------------------------------------- inputs ----
def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 16 + salt)
    return g


def _uniform(g, lo, hi, *shape):
    return torch.rand(*shape, generator=g, device=DEV) * (hi - lo) + lo


def _cfg(case, seed):
    flags = W.FLAG_DR | W.FLAG_CURRENT
    if case["kind"] in ("shac", "critic") or case.get("paper"):
        flags = 0
    if case["kind"] == "collect":
        flags |= W.FLAG_STAGGER
    if case.get("lissajous"):
        flags |= W.FLAG_LISSAJOUS
    H = 16 * case["h"] if "h" in case else (512 if case.get("paper") else W.EPISODE_LEN)
    s = case.get("substeps", 2)
    return dict(n_envs=case["n"], substeps=s, episode_len=H, dt_control={1: 0.02, 2: 0.05, 4: 0.04}[s], seed=seed, flags=flags)


def _env(case, seed):
    e = AuvEnv(_cfg(case, seed), W.VEHICLE, W.ALLOC)
    if case["kind"] in ("shac", "critic") or case.get("paper"):
        e.set_task(W.PAPER_TASK_BOX if case.get("box") else W.PAPER_TASK)
    e.reset()
    return e


def _nets(case, seed):
    paper = case.get("paper") or case["kind"] in ("shac", "critic") or case.get("n_act") == 6
    n_in = 12 if paper else 23
    pol, val = W.mlp_weights(6 if paper else 8, 2 * seed + 1, n_in=n_in), W.mlp_weights(1, 2 * seed + 2, n_in=n_in)
    if paper:   # a policy some iterations into training, which no longer saturates its wrench: outputs scaled by 1/4
        w3 = torch.from_numpy(pol["W3"].view(np.int16)).view(torch.bfloat16) * 0.25
        pol["W3"] = w3.view(torch.int16).numpy().view(np.uint16).copy()
    return pol, val


def _observations(g, n, paper):
    """Observations in the ranges of the environment's rows (position error, rotation, velocities, last action)."""
    if paper:
        hi = [3.0] * 3 + [1.5] * 3 + [1.0] * 3 + [1.5] * 3 + [0.0] * 11
    else:
        hi = [3.0] * 3 + [1.0] * 6 + [1.0] * 3 + [1.5] * 3 + [1.0] * 8
    hi = torch.tensor(hi, device=DEV)[:, None]
    return _uniform(g, -1.0, 1.0, 23, n) * hi


def _gae_inputs(g, T, n):
    return dict(reward=-_uniform(g, 0.0, 3.0, T, n), value=torch.randn(T, n, generator=g, device=DEV) - 20.0,
                done=(torch.rand(T, n, generator=g, device=DEV) < 0.004).float(),
                last_value=torch.randn(n, generator=g, device=DEV) - 20.0)


def _ppo_inputs(case, seed):
    """A rollout buffer of M samples whose actions came from a nearby policy: probability ratios in [0.6, 1.4], none
    within 0.03 of the clipping bounds; the minibatch is whole 16-sample blocks, cut to B."""
    g, M, B, k = _gen(seed), case["M"], case["B"], case["n_act"]
    pol, val = _nets(case, seed)
    obs = _observations(g, M, k == 6)
    n = _Net(pol, torch.float32)
    act = torch.zeros(8, M, device=DEV)
    logp = torch.empty(M, device=DEV)
    for a in range(0, M, 1 << 18):
        s = slice(a, min(M, a + (1 << 18)))
        mu = n.forward(obs[:, s])[:k]
        eps = torch.randn(k, mu.shape[1], generator=g, device=DEV)
        ratio = _uniform(g, 0.6, 1.4, mu.shape[1])
        near = ((ratio - 0.8).abs() < 0.03) | ((ratio - 1.2).abs() < 0.03)
        ratio = torch.where(near, 1.0 + 0.5 * (ratio - 1.0), ratio)
        ls = n.log_std[:k, None]
        act[:k, s] = mu + ls.exp() * eps
        logp[s] = (-0.5 * eps * eps - ls - 0.5 * math.log(2 * math.pi)).sum(0) - ratio.log()
    adv = 2.0 * torch.randn(M, generator=g, device=DEV) + 0.3
    ret = torch.randn(M, generator=g, device=DEV)
    blocks = torch.randperm(M // 16, generator=g, device=DEV)[: (B + 15) // 16]
    idx = (blocks[:, None] * 16 + torch.arange(16, device=DEV)).reshape(-1)[:B].to(torch.int32)
    if idx.numel() < B:   # fewer whole blocks than entries: the first samples again
        idx = torch.cat([idx, torch.arange(B - idx.numel(), device=DEV, dtype=torch.int32)])
    return pol, val, (obs, act, logp, adv, ret), idx.contiguous()


def _critic_inputs(case, seed):
    g, n, h = _gen(seed), case["n"], case["h"]
    return dict(obs=_observations(g, h * n, True).view(23, h, n), reward=-_uniform(g, 0.0, 3.0, h, n),
                value_last=torch.randn(n, generator=g, device=DEV) - 5.0)


# --------------------------------------------------------------------- prepare and run ----
def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, kind=kind)
    if kind in ("step", "rollout", "collect"):
        s["env"] = e = _env(case, seed)
        pol, val = _nets(case, seed)
        mode = case.get("mode", SAMPLE)
        s["mode"] = mode
        s["policy"] = upload_mlp(pol) if mode in (MEAN, SAMPLE) else None
        if kind == "step":
            s["actions"] = _uniform(_gen(seed), -1.2, 1.2, 8, case["n"]) if mode == EXTERNAL else None
        elif kind == "rollout":
            s["bufs"] = e.rollout_buffers(case["T"], record=("reward", "stats"))
        else:
            s["value"] = upload_mlp(val)
            s["bufs"] = e.rollout_buffers(case["T"], record=("obs", "act", "logp", "value", "reward", "done", "last_value"))
            s["bufs"]["act"].zero_()   # the paper task's rollout leaves rows 6 and 7 as they are
            s["adv"], s["ret"] = (torch.empty(case["T"], case["n"], device=DEV) for _ in range(2))
    elif kind == "gae":
        s.update(_gae_inputs(_gen(seed), case["T"], case["n"]))
        s["adv"], s["ret"] = (torch.empty(case["T"], case["n"], device=DEV) for _ in range(2))
    elif kind == "forward":
        s["net"] = upload_mlp(_forward_net(case, seed))
        s["obs"] = _observations(_gen(seed), case["n"], False)
        s["out"] = torch.empty(case["n_out"], case["n"], device=DEV)
    elif kind == "ppo":
        pol, val, buf, s["idx"] = _ppo_inputs(case, seed)
        s["learner"] = L = PpoLearner(pol, val)
        s["buf"], s["batch"] = buf, L.batch(*buf)
        L.work(case["B"])
    else:
        s["env"] = e = _env(case, seed)
        pol, val = _nets(case, seed)
        s["learner"] = L = ShacLearner(e, pol, val, h=case["h"], gamma=GAMMA)
        if kind == "shac":
            x = _moving_start(case, seed)
            e.state.copy_(x["state"])
            e.obs[12:18].copy_(x["abar"])
        else:
            rec = _critic_inputs(case, seed)
            own = {k: torch.empty_like(v) for k, v in rec.items()}
            L.window(MEAN, out=own, grad=False)   # the window whose records are regressed on ...
            for k, v in rec.items():              # ... holding values that the seed alone gives
                own[k].copy_(v)
    return s


def _forward_net(case, seed):
    return W.mlp_weights(case["n_out"], 2 * seed + 1)


def _moving_start(case, seed):
    """Vehicles under way: poses, velocities and action averages as in the middle of an episode."""
    g, n = _gen(seed, 1), case["n"]
    q = torch.randn(4, n, generator=g, device=DEV)
    q = torch.cat([2.0 + q[:1].abs(), q[1:]])   # within about 120 degrees of level
    q = q / q.norm(dim=0, keepdim=True)
    state = torch.cat([_uniform(g, -1.5, 1.5, 3, n), q, _uniform(g, -0.6, 0.6, 6, n)])
    return dict(state=state, abar=_uniform(g, -0.5, 0.5, 6, n))


def run(s):
    kind = s["kind"]
    if kind == "step":
        reward, done, stats = s["env"].step(s["mode"], s["actions"], s["case"]["stats"], s["policy"])
        out = dict(reward=reward, done=done, obs=s["env"].obs, state=s["env"].state)
        if stats is not None:
            out["stats"] = stats
        return out
    if kind == "rollout":
        b = s["env"].rollout(s["case"]["T"], s["mode"], policy=s["policy"], bufs=s["bufs"])
        return dict(reward=b["reward"], stats=b["stats"], state=s["env"].state, obs=s["env"].obs)
    if kind == "collect":
        b = s["env"].rollout(s["case"]["T"], s["mode"], policy=s["policy"], value=s["value"], bufs=s["bufs"])
        A.auv_gae(s["case"]["T"], s["case"]["n"], b["reward"], b["value"], b["done"], b["last_value"], GAMMA, LAM, s["adv"], s["ret"])
        return dict(b, adv=s["adv"], ret=s["ret"])
    if kind == "gae":
        A.auv_gae(s["case"]["T"], s["case"]["n"], s["reward"], s["value"], s["done"], s["last_value"], GAMMA, LAM, s["adv"], s["ret"])
        return dict(adv=s["adv"], ret=s["ret"])
    if kind == "forward":
        A.auv_mlp_forward(s["net"]["struct"], s["case"]["n"], s["obs"], s["out"])
        return s["out"]
    L = s["learner"]
    if kind == "ppo":
        L.update(s["batch"], s["idx"])
        return dict(grad_policy=L.pol.grad, grad_value=L.val.grad, stats=L.stats, policy=L.pol.theta, value=L.val.theta)
    if kind == "shac":
        L.window(s["case"]["mode"])
        L.step()
        out = dict(grad=L.grad, stats=L.stats, policy=L.pol.theta, state=s["env"].state, reward=L.rec["reward"])
        if s["case"]["critic"]:
            L.critic_update(iterations=16, batches=4, seed=1)
            out.update(values=L.values, ret=L.ret, value=L.val.theta)
        return out
    L.critic_update(iterations=s["case"]["iterations"], batches=s["case"]["batches"], seed=1)
    return dict(values=L.values, ret=L.ret, value=L.val.theta, stats=L.critic_stats)


# ---------------------------------------------------------------------- work, tolerance ----
F_NET = 2 * (23 * 256 + 256 * 256)   # one forward without the output layer
F_STAGE, F_STEP = 280, 335           # fp32 operations of a right-hand side, of the rest of a control step


def _physics(case, steps):
    return steps * (case.get("substeps", 2) * 4 * F_STAGE + F_STEP)


def work(case):
    kind, n = case["kind"], case.get("n", 0)
    weights = 2 * (23 * 256 + 256 * 256 + 8 * 256)
    io = n * 4 * (2 * (13 + 23 + 2) + 24)   # state, observation and counters in and out, parameters in
    if kind in ("step", "rollout", "collect"):
        T = case.get("T", 1)
        pol = case.get("mode", SAMPLE) in (MEAN, SAMPLE)
        flops = _physics(case, n * T) + (n * T * (F_NET + 2 * 256 * 8) if pol else 0)
        b = io + (weights if pol else 0)
        if kind == "step":
            b += n * (5 + (32 if case["mode"] == EXTERNAL else 0))
        elif kind == "rollout":
            b += 4 * n * T + 12 * T
        else:
            flops += n * (T + 1) * (F_NET + 512)
            b += weights + 4 * n * T * (23 + 8 + 1 + 1 + 1 + 1 + 2) + 4 * n
        return dict(bytes=b, flops=flops)
    if kind == "gae":
        return dict(bytes=4 * (5 * case["T"] * n + n), flops=8 * case["T"] * n)
    if kind == "forward":
        return dict(bytes=4 * n * (23 + case["n_out"]) + weights, flops=n * (F_NET + 512 * case["n_out"]))
    if kind == "ppo":
        B = case["B"]
        per = lambda k: 3 * F_NET - 2 * 23 * 256 + 6 * 256 * k   # forward, dW, dX (no input gradient)
        return dict(bytes=B * 4 * (23 + 8 + 4) + 4 * 2 * 72000 * 8, flops=B * (per(8) + per(1)))
    M = n * case["h"]
    fit = lambda its: M * its * (3 * F_NET - 2 * 23 * 256 + 6 * 256)
    if kind == "critic":
        return dict(bytes=M * 4 * (23 + 3 + case["iterations"] * 24), flops=fit(case["iterations"]) + M * (F_NET + 512))
    flops = M * (3 * (F_NET - 2 * 11 * 256) + 6 * 256 * 6) + 3 * _physics(case, M)
    b = io + 4 * M * (23 + 3) + 8 * weights
    if case["critic"]:
        flops += fit(16) + M * (F_NET + 512)
        b += M * 4 * (23 + 3 + 16 * 24)
    return dict(bytes=b, flops=flops)


def tolerance(case):
    """About four times the distance to exact(), measured over the ranges of draw()."""
    kind = case["kind"]
    if kind == "gae":
        return dict(rel=2e-6, max=1e-4)
    if kind == "forward":   # bf16 roundings of hidden values that fall the other way
        return dict(rel=4e-4, max=2e-2)
    if kind in ("step", "rollout") and case["mode"] in (EXTERNAL, RANDOM):
        return dict(rel=5e-6, max=1e-3)
    if kind == "step":
        return dict(rel=1e-3, max=2e-2, differ=1e-3)
    if kind in ("rollout", "collect"):   # such a rounding moves the trajectory that follows
        return dict(rel=8e-3, max=0.5)
    if kind == "ppo":
        return dict(rel=2e-3, max=0.3)
    return dict(rel=4e-3, max=0.5)


# ------------------------------------------------------------------ 64-bit reference ----
def _q(x):
    """Rounded to bf16 (nearest even), kept in the wide type."""
    return x.float().bfloat16().to(x.dtype)


class _Net:
    """An MLP with bf16 layer inputs; forward and the backward of the PPO update."""

    def __init__(self, net, dtype=torch.float64):
        def bits(x, rows, cols):
            t = torch.from_numpy(np.asarray(x, np.uint16).view(np.int16).copy()).view(torch.bfloat16).to(DEV).to(dtype)
            return torch.nn.functional.pad(t, (0, cols - t.shape[1], 0, rows - t.shape[0]))

        def f32(x, k):
            t = torch.from_numpy(np.asarray(x, np.float32)[:k].copy()).to(DEV).to(dtype)
            return torch.nn.functional.pad(t, (0, k - t.numel()))

        k = net["W3"].shape[0]
        self.n_out = 8 if k > 1 else 1
        self.W1, self.W2, self.W3 = bits(net["W1"], 256, 23), bits(net["W2"], 256, 256), bits(net["W3"], self.n_out, 256)
        self.b1, self.b2, self.b3 = f32(net["b1"], 256), f32(net["b2"], 256), f32(net["b3"], self.n_out)
        ls = torch.zeros(8, device=DEV, dtype=dtype)
        ls[:k] = torch.from_numpy(np.asarray(net["log_std"], np.float32)).to(DEV).to(dtype)[:k]
        self.log_std = ls

    def layers(self, x):
        x = _q(x)
        h1 = torch.tanh(self.W1 @ x + self.b1[:, None])
        h2 = torch.tanh(self.W2 @ _q(h1) + self.b2[:, None])
        return x, h1, h2, self.W3 @ _q(h2) + self.b3[:, None]

    def forward(self, x):
        return self.layers(x)[3]

    def backward(self, saved, gy, rounded_bias=False):
        """Gradients of the six parameter arrays and of the input."""
        x, h1, h2 = saved
        gq = _q(gy)
        d2 = (self.W3.t() @ gq) * (1 - h2 * h2)
        q2 = _q(d2)
        d1 = (self.W2.t() @ q2) * (1 - h1 * h1)
        q1 = _q(d1)
        rb = (lambda a, b: b) if rounded_bias else (lambda a, b: a)
        g = [q1 @ x.t(), q2 @ _q(h1).t(), gq @ _q(h2).t(), rb(d1, q1).sum(1), rb(d2, q2).sum(1), rb(gy, gq).sum(1)]
        return g, self.W1.t() @ q1

    def theta(self):
        t = [self.W1, self.W2, self.W3, self.b1, self.b2, self.b3] + ([self.log_std] if self.n_out == 8 else [])
        return torch.cat([x.reshape(-1) for x in t])

    def load(self, theta):
        """Parameters from the packed master vector: weights rounded to bf16."""
        o = 0
        for k in ("W1", "W2", "W3", "b1", "b2", "b3"):
            p = getattr(self, k)
            v = theta[o:o + p.numel()].view(p.shape)
            setattr(self, k, _q(v) if k[0] == "W" else v)
            o += p.numel()


def _adam(theta, g, m, v, t, lr, b1, b2, eps=1e-8):
    m = b1 * m + (1 - b1) * g
    v = b2 * v + (1 - b2) * g * g
    return theta - lr * (m / (1 - b1 ** t)) / ((v / (1 - b2 ** t)).sqrt() + eps), m, v


def _philox(c, key):
    """Philox4x32-10 (Salmon et al. 2011) on int64 tensors holding 32-bit words."""
    m32 = 0xFFFFFFFF

    def mul(a, b):
        p0, p1 = a * (b & 0xFFFF), a * (b >> 16)
        s = p1 + (p0 >> 16)
        return s >> 16, ((s << 16) | (p0 & 0xFFFF)) & m32

    x, y, z, w = c
    k0, k1 = key
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
        h0, l0 = mul(0xD2511F53, x)
        h1, l1 = mul(0xCD9E8D57, z)
        x, y, z, w = h1 ^ y ^ k0, l1, h0 ^ w ^ k1, l0
    return [x, y, z, w]


def _f32(x):
    return float(np.float32(x))


class _Sim:
    """The environments of include/auv.h in 64-bit torch arithmetic."""

    def __init__(self, case, seed, fluid_box=False):
        c = self.c = _cfg(case, seed)
        self.paper = case["kind"] in ("shac", "critic") or bool(case.get("paper"))
        self.n, self.key = case["n"], (seed & 0xFFFFFFFF, seed >> 32)
        self.gid = torch.arange(self.n, device=DEV, dtype=torch.int64)
        self.h = _f32(c["dt_control"]) / c["substeps"]
        self.t = 0
        V = W.VEHICLE
        d = lambda x: torch.tensor(np.asarray(x, np.float64), device=DEV)
        self.V = {k: d(v) for k, v in V.items()}
        if fluid_box:
            m, I = float(V["m"]), [float(x) for x in V["inertia"]]
            s = [math.sqrt(6 * (I[(i + 1) % 3] + I[(i + 2) % 3] - I[i]) / m) for i in range(3)]
            rho, mu, dm = 1000.0, _f32(1e-3), sum(s) / 3
            o = [(s[(i + 1) % 3], s[(i + 2) % 3]) for i in range(3)]
            self.V["added_mass"] = d([0.0] * 6)
            self.V["lin_damp"] = d([3 * math.pi * mu * dm] * 3 + [math.pi * mu * dm ** 3] * 3)
            self.V["quad_damp"] = d([0.5 * rho * a * b for a, b in o] + [rho * s[i] * (o[i][0] ** 4 + o[i][1] ** 4) / 64 for i in range(3)])
        self.alloc = d(W.ALLOC) * self.V["f_max"]
        self.ep = (self.gid % c["episode_len"]) if c["flags"] & W.FLAG_STAGGER else torch.zeros_like(self.gid)
        self.episode = torch.zeros_like(self.gid)
        self._reset(torch.ones(self.n, dtype=torch.bool, device=DEV), first=True)

    def words(self, a, b, blocks):
        out = []
        for k in range(blocks):
            z = torch.zeros_like(self.gid)
            out += _philox([self.gid, z + a, z + b, z + k], self.key)
        return out

    @staticmethod
    def u01(w):
        return (w >> 8).double() * 2.0 ** -24

    def _reset(self, who, first=False):
        wd = self.words(self.episode, 0, 8)
        af = lambda lo, span, k: _f32(lo) + _f32(span) * self.u01(wd[k])
        st = lambda lo, span, k0: torch.stack([af(lo, span, k0 + i) for i in range(3)])
        one, zero = torch.ones(3, self.n, device=DEV, dtype=torch.float64), torch.zeros(3, self.n, device=DEV, dtype=torch.float64)
        new = dict(pg=st(-2, 4, 12), v=zero, w=zero, s=one, cw=zero, gfac=one[0], u=torch.zeros(8, self.n, device=DEV, dtype=torch.float64))
        if self.paper:
            e = _f32(math.pi / 3)
            hf = 0.5 * torch.stack([af(-e, 2 * e, 15 + i) for i in range(3)])
            (sr, sp, sy), (cr, cp, cy) = hf.sin(), hf.cos()
            new["qg"] = torch.stack([cy * cp * cr + sy * sp * sr, cy * cp * sr - sy * sp * cr, cy * sp * cr + sy * cp * sr, sy * cp * cr - cy * sp * sr])
            new["gfac"] = af(0.95, 0.1, 0)
            new["p"] = zero
            new["q"] = torch.cat([one[:1], zero])
        else:
            def shoemake(k):
                u1, u2, u3 = (self.u01(wd[k + i]) for i in range(3))
                r1, r2, a, b = (1 - u1).sqrt(), u1.sqrt(), 2 * math.pi * u2, 2 * math.pi * u3
                return torch.stack([r2 * b.cos(), r1 * a.sin(), r1 * a.cos(), r2 * b.sin()])
            if self.c["flags"] & W.FLAG_DR:
                new["s"] = st(0.8, 0.4, 0)
            if self.c["flags"] & W.FLAG_CURRENT:
                new["cw"] = st(-0.3, 0.6, 3)
            new.update(p=st(-2, 4, 6), q=shoemake(9), qg=shoemake(15), amp=st(0.5, 1.5, 18), freq=st(0.02, 0.08, 21),
                       phase=st(0, 6.28318548, 24), yr=af(-0.1, 0.2, 27), y0=af(-3.14159274, 6.28318548, 28))
        for k, v in new.items():
            setattr(self, k, v if first else torch.where(who, v, getattr(self, k)))

    @staticmethod
    def rot(q):
        w, x, y, z = q
        return torch.stack([torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)]),
                            torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)]),
                            torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])])

    def rhs(self, tau, q, v, w):
        V, s, col = self.V, self.s, lambda x: x[:, None]
        cr = lambda a, b: torch.linalg.cross(a, b, dim=0)
        A1 = s[1] * col(V["added_mass"][:3])
        Ml, Ma = s[0] * V["m"] + A1, s[0] * col(V["inertia"]) + s[1] * col(V["added_mass"][3:])
        DL, DQ = s[2] * col(V["lin_damp"]), s[2] * col(V["quad_damp"])
        R = self.rot(q)
        cb, k = (R * self.cw[:, None]).sum(0), R[2]
        vr = v - cb
        F = tau[:3] - cr(w, Ml * vr) - (DL[:3] + DQ[:3] * vr.abs()) * vr - (V["B"] - self.gfac * V["W"]) * k
        G = tau[3:] - cr(w, Ma * w) - cr(vr, A1 * vr) - (DL[3:] + DQ[3:] * w.abs()) * w
        if not self.paper:
            G = G - cr((V["B"] * col(V["r_b"])).expand(3, self.n), k)
        e = q[1:]
        dq = 0.5 * torch.cat([-(e * w).sum(0)[None], q[0] * w + cr(e, w)])
        return (R * v[None]).sum(1), dq, F / Ml + cr(cb, w), G / Ma

    def integrate(self, tau):
        p, q, v, w = self.p, self.q, self.v, self.w
        for _ in range(self.c["substeps"]):
            k1 = self.rhs(tau, q, v, w)
            k2 = self.rhs(tau, *[x + 0.5 * self.h * k for x, k in zip((q, v, w), k1[1:])])
            k3 = self.rhs(tau, *[x + 0.5 * self.h * k for x, k in zip((q, v, w), k2[1:])])
            k4 = self.rhs(tau, *[x + self.h * k for x, k in zip((q, v, w), k3[1:])])
            p, q, v, w = (x + self.h / 6 * (a + 2 * b + 2 * c + d) for x, a, b, c, d in zip((p, q, v, w), k1, k2, k3, k4))
            q = q / q.norm(dim=0, keepdim=True)
        self.p, self.q, self.v, self.w = p, q, v, w

    def reference(self):
        if self.c["flags"] & W.FLAG_LISSAJOUS:
            t = self.ep.double() * _f32(self.c["dt_control"])
            psi = 0.5 * (self.y0 + self.yr * t)
            z = torch.zeros_like(psi)
            return self.pg + self.amp * (2 * math.pi * self.freq * t + self.phase).sin(), torch.stack([psi.cos(), z, z, psi.sin()])
        return self.pg, self.qg

    def observe(self):
        """Observation [23][N], distance, attitude angle (or rotation vector) of the current state."""
        pr, qr = self.reference()
        R = self.rot(self.q)
        rt = lambda x: (R * x[:, None]).sum(0)
        d = rt(pr - self.p)
        q = self.q
        ew = (q * qr).sum(0)
        ev = q[0] * qr[1:] - qr[0] * q[1:] - torch.linalg.cross(q[1:], qr[1:], dim=0)
        n = (ev * ev).sum(0).sqrt()
        theta = 2 * torch.atan2(n, ew.abs())
        if self.paper:
            rv = torch.where(ew < 0, -1.0, 1.0) * theta / n * ev
            return torch.cat([d, rv, self.v, self.w, torch.zeros(11, self.n, device=DEV, dtype=torch.float64)]), d.norm(dim=0), theta
        Rr = self.rot(qr)
        return torch.cat([d, rt(Rr[:, 0]), rt(Rr[:, 1]), self.v, self.w, self.u]), d.norm(dim=0), theta

    def noise(self, step):
        """Standard normals of the sampled actions, [8][N] (rows 6, 7 zero on the paper task)."""
        wd = self.words(step, 2, 2)
        eps = torch.zeros(8, self.n, device=DEV, dtype=torch.float64)
        for k in range(3 if self.paper else 4):
            rad = (-2 * ((wd[2 * k] >> 8).double() + 1).mul(2.0 ** -24).log()).sqrt()
            a = 2 * math.pi * self.u01(wd[2 * k + 1])
            i, j = (k, 3 + k) if self.paper else (2 * k, 2 * k + 1)
            eps[i], eps[j] = rad * a.cos(), rad * a.sin()
        return eps

    def random(self, step):
        wd = self.words(step, 1, 2)
        return torch.stack([2 * self.u01(w) - 1 for w in wd])

    def advance(self, a):
        """One control step without the reset: post-step observation, reward, distance."""
        u = a.clamp(-1, 1)
        if self.paper:
            T = W.PAPER_TASK
            self.integrate(torch.cat([T["f_max"] * u[:3], T["tau_max"] * u[3:6]]))
            ab, u = self.u[:6], u[:6]
            o, dist, _ = self.observe()
            D = torch.tensor(T["d_pos"], device=DEV, dtype=torch.float64)[:, None]
            sq = lambda x: (x * x).sum(0)
            r = (-_f32(T["w_pos"]) * sq(D * o[:3]) - _f32(T["w_att"]) * sq(o[3:6]) - _f32(T["w_act"]) * sq(u[3:])
                 - _f32(T["w_vel"]) * sq(o[9:12]) - _f32(T["w_mavg"]) * sq(u - ab))
            be = _f32(T["beta"])
            self.u = torch.cat([be * ab + (1 - be) * u, torch.zeros(2, self.n, device=DEV, dtype=torch.float64)])
            self.ep = self.ep + 1
            return o, r, dist
        self.integrate(self.alloc @ u)
        self.u = u
        self.ep = self.ep + 1
        o, dist, theta = self.observe()
        return o, -dist - 0.5 * theta - 0.01 * (u * u).sum(0), dist

    def end_step(self, o):
        """Resets finished episodes; returns the done flags and the next observation."""
        done = self.ep == self.c["episode_len"]
        if bool(done.any()):
            self.episode = self.episode + done.long()
            self._reset(done)
            self.ep = torch.where(done, torch.zeros_like(self.ep), self.ep)
            o = self.observe()[0]
        self.t += 1
        return done, o

    def state(self):
        return torch.cat([self.p, self.q, self.v, self.w])

    def env_obs(self, o):
        return torch.cat([o[:12], self.u[:6], o[18:]]) if self.paper else o


def _exact_gae(reward, value, done, last, T):
    adv = torch.empty_like(reward)
    a, v = torch.zeros_like(last), last
    for t in range(T - 1, -1, -1):
        nd = 1 - done[t]
        a = reward[t] + _f32(GAMMA) * nd * v - value[t] + _f32(GAMMA) * _f32(LAM) * nd * a
        adv[t], v = a, value[t]
    return adv, adv + value


def _packed(g, extra=None):
    return torch.cat([x.reshape(-1) for x in g] + ([extra] if extra is not None else []))


def _exact_rollout(case, seed):
    pol, val = _nets(case, seed)
    sim, T, n = _Sim(case, seed), case.get("T", 1), case["n"]
    mode = case.get("mode", SAMPLE)
    net = _Net(pol)
    ext = _uniform(_gen(seed), -1.2, 1.2, 8, n).double() if mode == EXTERNAL else None
    o = sim.observe()[0]
    k = 6 if sim.paper else 8
    keep = case["kind"] == "collect"
    f = dict(device=DEV, dtype=torch.float64)
    rec = dict(reward=torch.empty(T, n, **f), stats=torch.empty(3, T, **f), done=torch.empty(T, n, **f))
    if keep:
        rec.update(obs=torch.empty(23, T, n, **f), act=torch.zeros(8, T, n, **f), logp=torch.empty(T, n, **f), value=torch.empty(T, n, **f))
    for t in range(T):
        if mode == EXTERNAL:
            a = ext
        elif mode == RANDOM:
            a = sim.random(t)
        else:
            a = net.forward(o)
            if mode == SAMPLE:
                eps = sim.noise(t)
                a = a + net.log_std.exp()[:, None] * eps
                if keep:
                    rec["logp"][t] = (-0.5 * eps[:k] ** 2 - net.log_std[:k, None] - 0.5 * math.log(2 * math.pi)).sum(0)
        if keep:
            rec["obs"][:, t], rec["act"][:k, t] = o, a[:k]
        o, r, dist = sim.advance(a)
        done, o = sim.end_step(o)
        rec["reward"][t], rec["done"][t] = r, done.double()
        # the distance of a finished episode's statistics is the new episode's first
        dist = torch.where(done, o[:3].norm(dim=0), dist)
        rec["stats"][:, t] = torch.stack([r.sum(), done.double().sum(), dist.sum()])
    if keep:
        v = _Net(val)
        rec["value"] = v.forward(rec["obs"].reshape(23, -1)).view(T, n)
        rec["last_value"] = v.forward(o)[0]
        del rec["stats"]
        rec["adv"], rec["ret"] = _exact_gae(rec["reward"], rec["value"], rec["done"], rec["last_value"], T)
        return rec
    if case["kind"] == "step":
        out = dict(reward=rec["reward"][0], done=None, obs=sim.env_obs(o), state=sim.state())
        if case["stats"]:
            out["stats"] = rec["stats"][:, 0]
        return out
    return dict(reward=rec["reward"], stats=rec["stats"], state=sim.state(), obs=sim.env_obs(o))


def _exact_ppo(case, seed):
    pol, val, buf, idx = _ppo_inputs(case, seed)
    obs, act, logp, adv, ret = (x[..., idx.long()].double() for x in buf)
    B, k = case["B"], case["n_act"]
    P, V = _Net(pol), _Net(val)
    x, h1, h2, mu = P.layers(obs)
    iv = (-2 * P.log_std).exp()[:k, None]
    d = act[:k] - mu[:k]
    zz = d * d * iv
    lp = (-0.5 * zz - P.log_std[:k, None]).sum(0) - 0.5 * k * math.log(2 * math.pi)
    rho = (lp - logp).exp()
    ah = (adv - adv.mean()) / (adv.std(correction=0) + 1e-8)
    unc, clp = rho * ah, rho.clamp(1 - _f32(0.2), 1 + _f32(0.2)) * ah
    on = (unc <= clp).double()
    coef = -ah * rho * on / B
    gy = torch.zeros(8, B, device=DEV, dtype=torch.float64)
    gy[:k] = coef * d * iv
    gls = torch.zeros(8, device=DEV, dtype=torch.float64)
    gls[:k] = (coef * (zz - 1)).sum(1)
    gp = _packed(P.backward((x, h1, h2), gy)[0], gls)
    xv, v1, v2, y = V.layers(obs)
    e = y[0] - ret
    gv = _packed(V.backward((xv, v1, v2), (0.5 / B * e)[None])[0])
    sp, sv = (gp * gp).sum(), (gv * gv).sum()
    clip = (0.5 / ((sp + sv).sqrt() + 1e-6)).clamp(max=1.0)
    ent = (P.log_std[:k] + 0.5 * (1 + math.log(2 * math.pi))).sum()
    stats = torch.stack([-torch.minimum(unc, clp).mean(), 0.25 * (e * e).mean(), ent, (logp - lp).mean(), 1 - on.mean(), sp, sv, clip])
    th = lambda n, g: _adam(n.theta(), g * clip, 0 * g, 0 * g, 1, _f32(3e-4), _f32(0.9), _f32(0.999))[0]
    return dict(grad_policy=gp, grad_value=gv, stats=stats, policy=th(P, gp), value=th(V, gv))


class _ShacNet(torch.autograd.Function):
    """A network whose backward rounds each pre-activation's cotangent to bf16; parameter gradients go to `grads`."""

    @staticmethod
    def forward(ctx, x, net, grads):
        xq, h1, h2, y = net.layers(x)
        ctx.net, ctx.grads = net, grads
        ctx.save_for_backward(xq, h1, h2)
        return y

    @staticmethod
    def backward(ctx, gy):
        g, dx = ctx.net.backward(ctx.saved_tensors, gy, rounded_bias=True)
        if ctx.grads is not None:
            ctx.grads += _packed(g)
        return dx, None, None


def _exact_critic(net, obs, values, ret, iterations, batches, seed, lr=2e-3):
    """The regression's parameters after `iterations` shuffled passes."""
    M = ret.numel()
    nb = M // 16
    B = 16 * (nb // batches)
    theta = net.theta()
    m, v, t = torch.zeros_like(theta), torch.zeros_like(theta), 0
    m64, s = (1 << 64) - 1, seed
    for _ in range(iterations):
        perm = list(range(nb))
        for i in range(nb - 1, 0, -1):   # Fisher-Yates driven by SplitMix64
            s = (s + 0x9E3779B97F4A7C15) & m64
            z = s
            z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m64
            z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m64
            j = (((z ^ (z >> 31)) >> 32) * (i + 1)) >> 32
            perm[i], perm[j] = perm[j], perm[i]
        order = (torch.tensor(perm, device=DEV)[:, None] * 16 + torch.arange(16, device=DEV)).reshape(-1)
        for b in range(batches):
            c = order[b * B:(b + 1) * B]
            net.load(theta)
            x, h1, h2, y = net.layers(obs[:, c])
            e = y[0] - ret[c]
            g = _packed(net.backward((x, h1, h2), (2.0 / B * e)[None])[0])
            t += 1
            theta, m, v = _adam(theta, g, m, v, t, _f32(lr), _f32(0.7), _f32(0.95))
    return theta


def _exact_targets(val, obs, reward, last, h, n):
    values = val.forward(obs.reshape(23, -1)).view(h, n)
    return values, _exact_gae(reward, values, torch.zeros_like(reward), last, h)[1]


def _exact_shac(case, seed):
    pol, val = _nets(case, seed)
    P, V = _Net(pol), _Net(val)
    sim, n, h = _Sim(case, seed, fluid_box=case["box"]), case["n"], case["h"]
    x = _moving_start(case, seed)
    st = x["state"].double()
    sim.p, sim.q, sim.v, sim.w = st[:3], st[3:7], st[7:10], st[10:]
    sim.u = torch.cat([x["abar"].double(), torch.zeros(2, n, device=DEV, dtype=torch.float64)])
    ls = P.log_std.clone().requires_grad_()
    grads = torch.zeros(A.ppo_nparam(8) - 8, device=DEV, dtype=torch.float64)
    J, rewards, obs = 0.0, [], []
    o = sim.observe()[0].requires_grad_()
    for t in range(h):
        obs.append(o.detach())
        a = _ShacNet.apply(o, P, grads)
        if case["mode"] == SAMPLE:
            a = a + ls.exp()[:, None] * sim.noise(t)
        o, r, _ = sim.advance(a)
        rewards.append(r.detach())
        J = J + _f32(GAMMA) ** t * r
    vl = _ShacNet.apply(o, V, None)[0]
    Jv = J + _f32(GAMMA) ** h * vl
    loss = -Jv.sum() / (n * h)
    loss.backward()
    gls = ls.grad if ls.grad is not None else torch.zeros_like(ls)
    g = torch.cat([grads, gls])
    ss = (g * g).sum()
    clip = (1.0 / (ss.sqrt() + 1e-6)).clamp(max=1.0)
    z = torch.zeros((), device=DEV, dtype=torch.float64)
    stats = torch.stack([loss.detach(), J.detach().mean(), vl.detach().mean(), z, z, ss, z, clip])
    theta = _adam(P.theta(), g * clip, 0 * g, 0 * g, 1, _f32(2e-3), _f32(0.7), _f32(0.95))[0]
    out = dict(grad=g, stats=stats, policy=theta, state=sim.state().detach(), reward=torch.stack(rewards))
    if case["critic"]:
        O = torch.stack(obs, 1).reshape(23, -1)
        out["values"], out["ret"] = _exact_targets(V, O, out["reward"], vl.detach(), h, n)
        out["value"] = _exact_critic(V, O, out["values"], out["ret"].reshape(-1), 16, 4, 1)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "rollout", "collect"):
        if case.get("T", 1) * case["substeps"] > 800:
            return None
        return _exact_rollout(case, seed)
    if kind == "gae":
        x = {k: v.double() for k, v in _gae_inputs(_gen(seed), case["T"], case["n"]).items()}
        adv, ret = _exact_gae(x["reward"], x["value"], x["done"], x["last_value"], case["T"])
        return dict(adv=adv, ret=ret)
    if kind == "forward":
        return _Net(_forward_net(case, seed)).forward(_observations(_gen(seed), case["n"], False).double())[: case["n_out"]]
    if kind == "ppo":
        return _exact_ppo(case, seed)
    if kind == "shac":
        return _exact_shac(case, seed)
    x = {k: v.double() for k, v in _critic_inputs(case, seed).items()}
    V = _Net(_nets(case, seed)[1])
    values, ret = _exact_targets(V, x["obs"], x["reward"], x["value_last"], case["h"], case["n"])
    return dict(values=values, ret=ret, stats=None,
                value=_exact_critic(V, x["obs"].reshape(23, -1), values, ret.reshape(-1), case["iterations"], case["batches"], 1))
