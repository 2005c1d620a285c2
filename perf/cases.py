"""What a training program asks of this library, as cases that can be timed and checked.

The sizes are those of the repository's workloads (64, 4096 and 16 384 environments, 24 steps, observations 48 or 235
wide, 12 actions, networks [128, 128] and [512, 256, 128]) and irregular ones between them.  Each case is one call of
an entry point on what the program holds at that moment: roll-out, networks and optimiser moments in mid-training,
a workspace kept from call to call.  `exact` restates the same arithmetic in plain torch / numpy at 64 bits.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2509_10771_amd as rx

GAMMA, LAM = 0.99, 0.95
ADAM_STEP0 = 1000                    # optimiser steps behind the state that an update starts from
# The learning rate is that of the end of an annealed run.  It keeps the ratios off the clip range's edges: there one row
# more or less on the other side moves the whole trajectory, and two correct implementations would part for no fault
# of either.
PPO = dict(clip=0.2, value_coef=1.0, entropy_coef=0.01, max_grad_norm=1.0, lr=2e-6, beta1=0.9, beta2=0.999, adam_eps=1e-8)
NOISE_SEED, PERM_SEED = 7, 3


# ---- the cases ------------------------------------------------------------------------------------------------------
def listed():
    big, wide = "512,256,128", 235
    return [
        # a rollout step of a small run or of an evaluation: one launch, latency counts
        dict(name="act_64", kind="act", N=64, Da=48, A=12, hidden="128,128"),
        # the rollout step of the standard training run, 24 of them per iteration
        dict(name="act_4096", kind="act", N=4096, Da=48, A=12, hidden=big),
        # the same with a GRU memory per network
        dict(name="act_recurrent_4096", kind="act_recurrent", N=4096, Da=48, A=12, hidden=big, memory=256, cell="gru"),
        # the curiosity reward of one step at the largest environment count
        dict(name="rnd_16384", kind="rnd", N=16384, Da=48, hidden="256,256", K=64),
        # advantages of one iteration, with episodes cut by a time limit
        dict(name="gae_4096", kind="gae", N=4096, T=24, timeouts=True),
        # the update of a small run
        dict(name="update_tiny", kind="ppo", N=64, T=24, Da=48, A=12, hidden="128,128", epochs=5, minibatches=4, sym=False, rnd=False),
        # an update whose sizes fit no tile: 45 observations, a network of [400, 200, 100], an odd number of environments
        dict(name="update_ragged", kind="ppo", N=1501, T=24, Da=45, A=12, hidden="400,200,100", epochs=5, minibatches=4, sym=False,
             rnd=False),
        # the update of the standard training run
        dict(name="update_flat", kind="ppo", N=4096, T=24, Da=48, A=12, hidden=big, epochs=5, minibatches=4, sym=False, rnd=False),
        # height-scan observations, every minibatch doubled by its mirror image, mirror loss
        dict(name="update_rough", kind="ppo", N=4096, T=24, Da=wide, A=12, hidden=big, epochs=5, minibatches=4, sym=True, rnd=False),
        # the largest: 16 384 environments and the curiosity predictor trained on the same rows
        dict(name="update_curiosity", kind="ppo", N=16384, T=24, Da=48, A=12, hidden=big, epochs=5, minibatches=8, sym=False, rnd=True),
        # distillation: the student regresses on stored teacher actions
        dict(name="bc_distill", kind="bc", N=4096, T=24, Da=48, A=12, hidden="256,256,128", epochs=2, minibatches=4),
        # back-propagation through time over the rollout
        dict(name="update_recurrent", kind="ppo_recurrent", N=4096, T=24, Da=48, A=12, hidden=big, memory=256, cell="gru", epochs=5,
             minibatches=4),
    ]


def draw(rng):
    spread = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    kind = rng.choice(["act", "act_recurrent", "rnd", "gae", "ppo", "ppo", "bc", "ppo_recurrent"])
    hidden = rng.choice(["128,128", "256,128", "400,200,100", "256,256,128", "512,256,128"])
    Da, A = rng.choice([48, 235, rng.randint(20, 260)]), rng.choice([12, rng.randint(4, 24)])
    most = max(work(c)["flops"] for c in listed())
    while True:
        if kind == "act":
            c = dict(kind=kind, N=spread(1, 16384), Da=Da, A=A, hidden=hidden)
        elif kind == "act_recurrent":
            c = dict(kind=kind, N=spread(16, 4096), Da=Da, A=A, hidden=hidden, memory=rng.choice([128, 256]), cell=rng.choice(["gru", "lstm"]))
        elif kind == "rnd":
            c = dict(kind=kind, N=spread(64, 16384), Da=Da, hidden=rng.choice(["128,128", "256,256"]), K=rng.choice([32, 64]))
        elif kind == "gae":
            c = dict(kind=kind, N=spread(64, 65536), T=rng.randint(8, 48), timeouts=rng.random() < 0.5)
        elif kind == "ppo":
            sym = rng.random() < 0.25
            c = dict(kind=kind, N=spread(64, 16384), T=rng.choice([16, 24, 32]), Da=Da, A=A, hidden=hidden, epochs=5,
                     minibatches=rng.choice([4, 8]), sym=sym, rnd=not sym and rng.random() < 0.25)
        elif kind == "bc":
            c = dict(kind=kind, N=spread(64, 8192), T=24, Da=Da, A=A, hidden=hidden, epochs=2, minibatches=4)
        else:
            c = dict(kind=kind, N=4 * spread(16, 1024), T=24, Da=Da, A=A, hidden=hidden, memory=rng.choice([128, 256]),
                     cell=rng.choice(["gru", "lstm"]), epochs=5, minibatches=4)
        if work(c)["flops"] <= most:
            return c


# ---- sizes -----------------------------------------------------------------------------------------------------------
def _nets(case):
    """Layer widths (input, hidden..., output) of the networks that take part."""
    h = tuple(int(v) for v in case["hidden"].split(","))
    if case["kind"] == "rnd":
        return dict(predictor=(case["Da"],) + h + (case["K"],), target=(case["Da"],) + h + (case["K"],))
    if case["kind"] == "bc":
        return dict(student=(case["Da"],) + h + (case["A"],))
    d = case.get("memory", case["Da"])
    nets = dict(actor=(d,) + h + (case["A"],), critic=(d,) + h + (1,))
    if case.get("rnd"):
        nets.update(predictor=(case["Da"], 256, 256, 64), target=(case["Da"], 256, 256, 64))
    return nets


def _macs(dims):
    return sum(a * b for a, b in zip(dims[:-1], dims[1:]))


def _count(dims):
    return sum(a * b + b for a, b in zip(dims[:-1], dims[1:]))


def work(case):
    k, N = case["kind"], case["N"]
    if k == "gae":
        n = case["T"] * N
        return {"bytes": n * (8 + 1 + bool(case["timeouts"]) + 8) + 4 * N, "flops": 12 * n}
    nets, D, A = _nets(case), case["Da"], case.get("A", 0)
    params = sum(_count(d) for d in nets.values())
    cell = 0
    if "memory" in case:
        G, H = (4 if case["cell"] == "lstm" else 3), case["memory"]
        cell = 2 * G * H * (D + H)                                      # multiply-adds per row, both memories
        params += 2 * G * H * (D + H + 2)
    if k in ("act", "act_recurrent", "rnd"):
        out = 4 * N * (3 * A + 2) if k != "rnd" else 12 * N
        state = 2 * 2 * 4 * N * case["memory"] * (2 if case["cell"] == "lstm" else 1) if cell else 0
        return {"bytes": 4 * N * D + 4 * params + out + state, "flops": 2.0 * N * (cell + sum(_macs(d) for d in nets.values()))}
    rows = case["T"] * N
    sides = 2 if case.get("sym") else 1
    macs = 0                                                            # forward, weight gradient, input gradient
    for name, d in nets.items():
        first = 0 if cell else d[0] * d[1]                              # the network's own input needs no gradient
        macs += sides * ((_macs(d)) if name == "target" else 3 * _macs(d) - first)
    if cell:
        macs += 3 * cell - 2 * G * H * D
    per_row = D + (2 * A if k == "bc" else 3 * A + 4)
    return {"bytes": 4 * rows * per_row + 4 * 7 * params, "flops": 2.0 * case["epochs"] * rows * macs}


def tolerance(case):
    # fp32 throughout.  About four times the largest error against `exact` seen over a hundred seeds: single passes and
    # plain regression 6e-7 (elementwise 4e-6); the gradients of a PPO update are sums of terms that nearly cancel, and
    # the moments carry them over all steps of the call: 4e-5 (elementwise 1e-3)
    if case["kind"] in ("ppo", "ppo_recurrent"):
        return {"rel": 1.6e-4, "max": 4e-3}
    return {"rel": 2.4e-6, "max": 2e-5}


# ---- inputs ----------------------------------------------------------------------------------------------------------
def _data(case, seed):
    """All tensors of a case, drawn on the GPU from the seed."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)
    normal = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    uniform = lambda *s: torch.rand(*s, generator=g, device="cuda")  # noqa: E731
    k, N = case["kind"], case["N"]
    d = {}

    def observations(*lead):
        """Proprioception (normal, 5 % of the entries ten times as large), behind column 48 a height scan."""
        D = case["Da"]
        n = min(D, 48)
        x = normal(*lead, n)
        x = torch.where(uniform(*lead, n) < 0.05, x * 10.0, x)
        return torch.cat([x, uniform(*lead, D - n) * 2.0 - 1.0], -1).contiguous() if D > n else x

    def mlp(dims, log_std):
        parts = []
        for a, b in zip(dims[:-1], dims[1:]):
            parts += [(uniform(a * b) * 2.0 - 1.0) * math.sqrt(6.0 / (a + b)), normal(b) * 0.01]
        return torch.cat(parts + ([uniform(dims[-1]) * -0.5] if log_std else []))

    def moments(p):
        """Adam moments of a run in progress: a gradient norm near the clip, steps of about a tenth of the learning rate."""
        return 3e-4 * normal(p.numel()), 1e-5 * (0.5 + uniform(p.numel()))

    if k == "gae":
        T = case["T"]
        d.update(rewards=0.5 + 0.3 * normal(T, N), values=normal(T, N), last=normal(N))
        timeouts = (uniform(T, N) < 0.02).to(torch.uint8)
        d["dones"] = (uniform(T, N) < 0.01).to(torch.uint8)
        if case["timeouts"]:
            d.update(timeouts=timeouts, dones=d["dones"] | timeouts)
        return d
    nets = _nets(case)
    for name, dims in nets.items():
        d[name] = mlp(dims, name == "actor")
    if "memory" in case:
        G, H = (4 if case["cell"] == "lstm" else 3), case["memory"]
        S = 2 * H if case["cell"] == "lstm" else H
        for name in ("mem_actor", "mem_critic"):
            d[name] = (uniform(G * H * (case["Da"] + H + 2)) * 2.0 - 1.0) / math.sqrt(H)
        for name in ("h_actor", "h_critic"):
            d[name] = 0.5 * normal(N, S)
    if k in ("act", "act_recurrent", "rnd"):
        d["obs"] = observations(N)
        if k == "rnd":
            d.update(rewards=0.5 + 0.3 * normal(N), running=torch.tensor([0.4, 0.05, 1e5], device="cuda"))
        if k == "act_recurrent":
            d["reset"] = (uniform(N) < 0.01).to(torch.uint8)
        return d

    # an update: the rollout was collected by the networks as they are now
    T, A = case["T"], case["A"]
    d["obs"] = observations(T, N)
    for name in list(d):
        if name in ("actor", "critic", "student", "predictor", "mem_actor", "mem_critic"):
            d["m_" + name], d["v_" + name] = moments(d[name])
    if k == "bc":
        d["targets"] = 0.5 * normal(T, N, A)
        return d
    if "memory" in case:
        d["dones"] = (uniform(T, N) < 0.01).to(torch.uint8)
        xa = _sequence(d["mem_actor"], case, d["obs"], d["h_actor"], d["dones"])
        xc = _sequence(d["mem_critic"], case, d["obs"], d["h_critic"], d["dones"])
    else:
        xa = xc = d["obs"]
    mu = _forward(d["actor"], nets["actor"], xa)
    sigma = torch.exp(d["actor"][-A:]).expand(T, N, A).contiguous()
    eps = normal(T, N, A)
    d.update(mu=mu, sigma=sigma, actions=mu + sigma * eps, values=_forward(d["critic"], nets["critic"], xc)[..., 0].contiguous(),
             logp=(-0.5 * eps * eps - torch.log(sigma) - 0.5 * math.log(2 * math.pi)).sum(-1), adv=normal(T, N))
    d["returns"] = d["values"] + 0.5 * d["adv"] + 0.1 * normal(T, N)
    if case["kind"] == "ppo" and case["sym"]:
        h = np.random.default_rng(int(seed) + 5)
        for name, n in (("obs", case["Da"]), ("act", A)):               # mirror images: paired columns, signs
            perm, sign, order = np.arange(n), np.ones(n), h.permutation(n)
            for a, b in zip(order[: n // 2], order[n // 2:]):
                perm[a], perm[b] = b, a
                sign[a] = sign[b] = h.choice([-1.0, 1.0])
            d["perm_" + name] = torch.from_numpy(perm.astype(np.int32))
            d["sign_" + name] = torch.from_numpy(sign.astype(np.float32))
    return d


def prepare(case, seed):
    d, k, N = _data(case, seed), case["kind"], case["N"]
    s = dict(case=case, d=d, calls=0)
    new = lambda *sh: torch.empty(*sh, device="cuda")  # noqa: E731
    if k == "gae":
        T = case["T"]
        s.update(adv=new(T, N), ret=new(T, N), ws=rx.workspace(rx.rslx_gae_workspace_bytes(T, N)))
        return s
    nets = _nets(case)
    for name, dims in nets.items():
        trained = "m_" + name in d
        s[name] = rx.Mlp(dims, d[name], trainable=trained, has_log_std=name == "actor")
        if trained:
            s[name].adam_m, s[name].adam_v = d["m_" + name], d["v_" + name]
    if "memory" in case:
        cell = rx.CELL_LSTM if case["cell"] == "lstm" else rx.CELL_GRU
        for name in ("mem_actor", "mem_critic"):
            trained = "m_" + name in d
            s[name] = rx.Memory(cell, case["Da"], case["memory"], d[name], trainable=trained)
            if trained:
                s[name].adam_m, s[name].adam_v = d["m_" + name], d["v_" + name]
    if k in ("act", "act_recurrent"):
        A = case["A"]
        s.update(actions=new(N, A), logp=new(N), values=new(N), mu=new(N, A), sigma=new(N, A))
        s["ws"] = rx.workspace(rx.rslx_act_workspace_bytes(s["actor"], s["critic"], N) if k == "act" else
                               rx.rslx_act_recurrent_workspace_bytes(s["mem_actor"], s["actor"], s["mem_critic"], s["critic"], N))
        return s
    if k == "rnd":
        s.update(r_int=new(N), ws=rx.workspace(rx.rslx_rnd_workspace_bytes(s["target"], N)))
        return s
    T, E, M = case["T"], case["epochs"], case["minibatches"]
    s.update(stats=torch.zeros(E * M, rx.NSTATS, device="cuda"), step=ctypes.c_int64(ADAM_STEP0))
    if k == "bc":
        s["ws"] = rx.workspace(rx.rslx_bc_update_workspace_bytes(s["student"], None, T * N, _bc_cfg(case, 0)))
        return s
    s["rollout"] = rx.Rollout(T, N, d["obs"], d["obs"], d["actions"], d["logp"], d["values"], d["mu"], d["sigma"], d["adv"], d["returns"])
    if k == "ppo_recurrent":
        s["ws"] = rx.workspace(rx.rslx_ppo_update_recurrent_workspace_bytes(s["mem_actor"], s["actor"], s["mem_critic"], s["critic"],
                                                                            s["rollout"], _ppo_cfg(case, 0)))
        return s
    s["sym"] = rx.Sym(d["perm_obs"], d["sign_obs"], d["perm_obs"], d["sign_obs"], d["perm_act"], d["sign_act"]) if case["sym"] else None
    s["rnd"] = rx.RndTrain(s["target"], s["predictor"], lr=PPO["lr"], adam_step=ADAM_STEP0) if case["rnd"] else None
    s["ws"] = rx.workspace(rx.rslx_ppo_update_workspace_bytes(s["actor"], s["critic"], s["rollout"], _ppo_cfg(case, 0), s["sym"], s["rnd"]))
    return s


def _ppo_cfg(case, call):
    return rx.PpoCfg(epochs=case["epochs"], minibatches=case["minibatches"], seed=PERM_SEED, call_index=call, **PPO)


def _bc_cfg(case, call):
    return rx.BcCfg(lr=PPO["lr"], epochs=case["epochs"], minibatches=case["minibatches"], seed=PERM_SEED, call_index=call)


# ---- one pass --------------------------------------------------------------------------------------------------------
def run(s):
    case, d = s["case"], s["d"]
    k, N, call = case["kind"], case["N"], s["calls"]
    s["calls"] += 1
    if k == "act":
        rx.rslx_act(s["actor"], s["critic"], d["obs"], d["obs"], N, NOISE_SEED, call, None, s["actions"], s["logp"], s["values"], s["mu"],
                    s["sigma"], 0, s["ws"])
        return {n: s[n] for n in ("actions", "logp", "values", "mu", "sigma")}
    if k == "act_recurrent":
        rx.rslx_act_recurrent(s["mem_actor"], s["actor"], s["mem_critic"], s["critic"], d["obs"], d["obs"], N, d["h_actor"], d["h_critic"],
                              d["reset"], None, None, NOISE_SEED, call, None, s["actions"], s["logp"], s["values"], s["mu"], s["sigma"],
                              0, s["ws"])
        return dict({n: s[n] for n in ("actions", "logp", "values", "mu", "sigma")}, h_actor=d["h_actor"], h_critic=d["h_critic"])
    if k == "rnd":
        rx.rslx_rnd(s["target"], s["predictor"], d["obs"], N, case["Da"], None, case["Da"], d["running"], 0.5, True, s["r_int"],
                    d["rewards"], s["ws"])
        return dict(r_int=s["r_int"], rewards=d["rewards"], running=d["running"])
    if k == "gae":
        rx.rslx_gae(d["rewards"], d["values"], d["last"], d["dones"], d.get("timeouts"), case["T"], N, GAMMA, LAM, True, s["adv"], s["ret"],
                    s["ws"])
        return dict(advantages=s["adv"], returns=s["ret"])
    if k == "bc":
        rx.rslx_bc_update(s["student"], None, d["obs"], None, d["targets"], case["T"] * N, _bc_cfg(case, call), s["step"], s["stats"], s["ws"])
    elif k == "ppo":
        rx.rslx_ppo_update(s["actor"], s["critic"], s["rollout"], _ppo_cfg(case, call), s["sym"], s["rnd"], s["step"], s["stats"], s["ws"])
    else:
        rx.rslx_ppo_update_recurrent(s["mem_actor"], s["actor"], s["mem_critic"], s["critic"], s["rollout"], d["dones"], d["h_actor"],
                                     d["h_critic"], _ppo_cfg(case, call), s["step"], s["stats"], s["ws"])
    out = dict(stats=s["stats"])
    for name in ("actor", "critic", "student", "predictor", "mem_actor", "mem_critic"):
        if name in s:
            out[name] = dict(params=s[name].params, grads=s[name].grads, m=s[name].adam_m, v=s[name].adam_v)
    return out


# ---- the same at 64 bits, without the library -------------------------------------------------------------------------
def _layers(flat, dims):
    o = 0
    for a, b in zip(dims[:-1], dims[1:]):
        yield flat[o:o + a * b].view(a, b), flat[o + a * b:o + a * b + b]
        o += a * b + b


def _forward(flat, dims, x):
    last = len(dims) - 2
    for i, (w, b) in enumerate(_layers(flat, dims)):
        x = x @ w + b
        if i < last:
            x = torch.where(x > 0, x, torch.expm1(torch.clamp(x, max=0.0)))
    return x


def _cell_step(flat, case, x, s):
    """Packed new state of a GRU (gates r, z, n; state h) or an LSTM (gates i, f, g, o; state [h | c])."""
    H, D = case["memory"], case["Da"]
    G = 4 if case["cell"] == "lstm" else 3
    w_ih, b_ih = flat[:D * G * H].view(D, G * H), flat[D * G * H:(D + 1) * G * H]
    o = (D + 1) * G * H
    w_hh, b_hh = flat[o:o + H * G * H].view(H, G * H), flat[o + H * G * H:]
    gi, gh = x @ w_ih + b_ih, s[..., :H] @ w_hh + b_hh
    if G == 3:
        r, z = torch.sigmoid(gi[..., :H] + gh[..., :H]), torch.sigmoid(gi[..., H:2 * H] + gh[..., H:2 * H])
        n = torch.tanh(gi[..., 2 * H:] + r * gh[..., 2 * H:])
        return (1 - z) * n + z * s
    a = gi + gh
    i, f, g, q = torch.sigmoid(a[..., :H]), torch.sigmoid(a[..., H:2 * H]), torch.tanh(a[..., 2 * H:3 * H]), torch.sigmoid(a[..., 3 * H:])
    c = f * s[..., H:] + i * g
    return torch.cat([q * torch.tanh(c), c], -1)


def _sequence(flat, case, x, s, dones):
    """Hidden states of a whole rollout [T, N, H]; a state is zeroed after the step on which its episode ended."""
    out = []
    for t in range(x.shape[0]):
        if t:
            s = s * (1 - dones[t - 1].to(s.dtype))[:, None]
        s = _cell_step(flat, case, x[t], s)
        out.append(s[..., :case["memory"]])
    return torch.stack(out)


def _mix(x):
    """SplitMix64 output function on uint64 arrays."""
    with np.errstate(over="ignore"):
        x = np.asarray(x, np.uint64) + np.uint64(0x9E3779B97F4A7C15)
        x = (x ^ (x >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return x ^ (x >> np.uint64(31))


def _permutation(epoch, n):
    base = _mix(_mix(_mix(np.uint64(PERM_SEED)) ^ np.uint64(0)) ^ np.uint64(epoch))
    return torch.from_numpy(np.argsort(_mix(base ^ np.arange(n, dtype=np.uint64)), kind="stable")).cuda()


def _noise(N, A):
    base = _mix(_mix(np.uint64(NOISE_SEED ^ 0xAC7)) ^ np.uint64(0))
    h = _mix(base ^ np.arange(N * A, dtype=np.uint64))
    u1 = ((h >> np.uint64(40)).astype(np.float64) + 1) * 2.0 ** -24
    u2 = ((h >> np.uint64(8)) & np.uint64(0xFFFFFF)).astype(np.float64) * 2.0 ** -24
    return torch.from_numpy(np.sqrt(-2 * np.log(u1)) * np.cos(2 * np.pi * u2)).cuda().view(N, A)


def _log_density(a, mu, log_std):
    return (-0.5 * ((a - mu) / torch.exp(log_std)) ** 2 - log_std - 0.5 * math.log(2 * math.pi)).sum(-1)


class _Adam:
    """Parameters, moments and last gradient of one network at 64 bits."""

    def __init__(self, d, name):
        self.p, self.m, self.v = d[name].clone().requires_grad_(True), d["m_" + name].clone(), d["v_" + name].clone()

    def step(self, t, scale, lr):
        b1, b2, eps = (float(np.float32(PPO[n])) for n in ("beta1", "beta2", "adam_eps"))
        self.g, g = self.p.grad, self.p.grad * scale
        self.m, self.v = b1 * self.m + (1 - b1) * g, b2 * self.v + (1 - b2) * g * g
        step = lr * (self.m / (1 - b1 ** t)) / (torch.sqrt(self.v / (1 - b2 ** t)) + eps)
        self.p = (self.p.detach() - step).requires_grad_(True)

    def outputs(self):
        return dict(params=self.p.detach(), grads=self.g, m=self.m, v=self.v)


def exact(case, seed):
    d = {n: (t.double() if t.is_floating_point() else t) for n, t in _data(case, seed).items()}
    k, N = case["kind"], case["N"]
    f32 = lambda v: float(np.float32(v))  # noqa: E731   (the C structures carry 32-bit hyper-parameters)
    if k == "gae":
        r, v, nd = d["rewards"], d["values"], 1.0 - d["dones"].double()
        if case["timeouts"]:
            r = r + f32(GAMMA) * v * d["timeouts"].double()
        adv, a, nxt = torch.empty_like(r), torch.zeros_like(d["last"]), d["last"]
        for t in range(case["T"] - 1, -1, -1):
            a = r[t] + f32(GAMMA) * nd[t] * nxt - v[t] + f32(GAMMA) * f32(LAM) * nd[t] * a
            adv[t], nxt = a, v[t]
        return dict(advantages=(adv - adv.mean()) / (adv.std() + 1e-8), returns=adv + v)
    nets = _nets(case)
    if k == "rnd":
        raw = ((_forward(d["predictor"], nets["predictor"], d["obs"]) - _forward(d["target"], nets["target"], d["obs"])) ** 2).sum(-1)
        mean, var, count = (float(x) for x in d["running"])
        tot, delta = count + N, float(raw.mean()) - mean
        var = (var * count + float(raw.var(unbiased=False)) * N + delta * delta * count * N / tot) / tot
        r = raw / math.sqrt(var + 1e-8)
        return dict(r_int=r, rewards=d["rewards"] + 0.5 * r, running=torch.tensor([mean + delta * N / tot, var, tot], dtype=torch.float64))
    if k in ("act", "act_recurrent"):
        xa = xc = d["obs"]
        more = {}
        if k == "act_recurrent":
            keep = (1.0 - d["reset"].double())[:, None]
            for w in ("actor", "critic"):
                more["h_" + w] = _cell_step(d["mem_" + w], case, d["obs"], d["h_" + w] * keep)
            xa, xc = more["h_actor"][:, :case["memory"]], more["h_critic"][:, :case["memory"]]
        log_std = d["actor"][-case["A"]:]
        mu = _forward(d["actor"], nets["actor"], xa)
        sigma = torch.exp(log_std).expand_as(mu)
        a = mu + sigma * _noise(N, case["A"])
        return dict(actions=a, logp=_log_density(a, mu, log_std), values=_forward(d["critic"], nets["critic"], xc)[:, 0], mu=mu, sigma=sigma, **more)

    T, A, M, clip, t_adam = case["T"], case["A"], case["minibatches"], f32(PPO["clip"]), ADAM_STEP0
    names = [n for n in ("actor", "critic", "student", "mem_actor", "mem_critic") if n in d]
    opt = {n: _Adam(d, n) for n in names + (["predictor"] if case.get("rnd") else [])}
    columns = "memory" in case                                          # minibatches of whole environments
    flat = {n: d[n].reshape((T * N,) + d[n].shape[2:]) for n in ("obs", "actions", "logp", "values", "mu", "sigma", "adv", "returns", "targets") if n in d}
    stats = torch.zeros(case["epochs"] * M, 8, dtype=torch.float64)
    for e in range(case["epochs"]):
        perm = _permutation(e, N if columns else T * N)
        n = perm.numel() // M
        for b in range(M):
            row, i = stats[e * M + b], perm[b * n:(b + 1) * n]
            if columns:
                envs, i = i, (torch.arange(T, device="cuda")[:, None] * N + i).reshape(-1)
            t_adam += 1
            x = flat["obs"][i]
            if k == "bc":
                loss = ((_forward(opt["student"].p, nets["student"], x) - flat["targets"][i]) ** 2).mean()
                row[0] = loss.detach()
            else:
                rows = {m: v[i] for m, v in flat.items() if m != "obs"}
                xa = xc = x
                if columns:
                    seq = lambda w: _sequence(opt["mem_" + w].p, case, d["obs"][:, envs], d["h_" + w][envs], d["dones"][:, envs])  # noqa: E731
                    xa, xc = (seq(w).reshape(-1, case["memory"]) for w in ("actor", "critic"))
                act, mu_old, sg_old = rows["actions"], rows["mu"], rows["sigma"]
                if case.get("sym"):
                    mirror = lambda v, w: v[..., d["perm_" + w].long().cuda()] * d["sign_" + w].cuda()  # noqa: E731
                    xa = xc = torch.cat([x, mirror(x, "obs")])
                    act = torch.cat([act, mirror(act, "act")])
                    rows.update({m: torch.cat([rows[m]] * 2) for m in ("logp", "adv", "returns", "values")})
                mu, ls = _forward(opt["actor"].p, nets["actor"], xa), opt["actor"].p[-A:]
                v = _forward(opt["critic"].p, nets["critic"], xc)[:, 0]
                ratio = torch.exp(_log_density(act, mu, ls) - rows["logp"])
                pol = torch.maximum(-rows["adv"] * ratio, -rows["adv"] * torch.clamp(ratio, 1 - clip, 1 + clip)).mean()
                near = rows["values"] + torch.clamp(v - rows["values"], -clip, clip)
                val = torch.maximum((v - rows["returns"]) ** 2, (near - rows["returns"]) ** 2).mean()
                ent = ls.sum() + 0.5 * A * (1 + math.log(2 * math.pi))
                loss = pol + f32(PPO["value_coef"]) * val - f32(PPO["entropy_coef"]) * ent
                with torch.no_grad():
                    sg, mu0 = torch.exp(ls), mu[:mu_old.shape[0]]
                    kl = (torch.log(sg / sg_old) + (sg_old ** 2 + (mu_old - mu0) ** 2) / (2 * sg ** 2) - 0.5).sum(-1).mean()
                    for c, q in ((0, pol), (1, val), (2, ent), (3, kl), (5, ((ratio < 1 - clip) | (ratio > 1 + clip)).double().mean())):
                        row[c] = q
                if case.get("sym"):
                    h = mu_old.shape[0]
                    ml = ((mu[h:] - mirror(mu[:h], "act").detach()) ** 2).mean()
                    loss, row[6] = loss + ml, ml.detach()
            loss.backward()
            norm = math.sqrt(sum(float((opt[m].p.grad ** 2).sum()) for m in names))
            row[4] = norm
            most = 0.0 if k == "bc" else f32(PPO["max_grad_norm"])
            scale = min(1.0, most / (norm + 1e-6)) if most > 0 else 1.0
            for m in names:
                opt[m].step(t_adam, scale, f32(PPO["lr"]))
            if case.get("rnd"):
                pr = opt["predictor"]
                rl = ((_forward(pr.p, nets["predictor"], x) - _forward(d["target"], nets["target"], x)) ** 2).mean()
                rl.backward()
                row[7] = rl.detach()
                pr.step(t_adam, 1.0, f32(PPO["lr"]))
    return dict(stats=stats, **{m: o.outputs() for m, o in opt.items()})
