"""The work that users of this package have it do, as measurable cases.

Each case is one call pattern through the public entry points (cp_step,
cp_rollout, cp_policy) at one size: `prepare` makes what a program has in
hand before the call, `run` is one pass, `exact` the same pass in plain torch
at 64 bits.  The kinds:

step     one environment step with the caller's actions and every output --
         the inner call of an agent loop that chooses actions itself.
infer    one cp_policy followed by one such step on its actions: simulation
         and inference as separate kernels.
rollout  a whole rollout in registers (CP_RESIDENT), random actions, no
         trajectory, per-environment statistics and totals.
collect  the same with the full trajectory (obs, reward, done).
fused    a rollout of one launch per step (CP_FUSED with its workspace);
         from 2,097,152 environments with the trajectory it streams.
policy   a register-resident rollout whose actions come from the MLP policy;
         with the trajectory (what a learner collects) or with statistics only
         (policy evaluation).
"""
import math

import numpy as np
import torch

import paper_2301_13062_amd as cp
from paper_2301_13062_amd import synth

STEP_FLOPS = 31  # operations of one environment step's dynamics
POLICY_FLOPS = 2 * (4 * 64 + 64 * 64 + 64 * 2)
ELEM = {"f32": 4, "f64": 8, "f16": 2}


def listed():
    return [
        # an agent's loop over a few thousand environments, its own actions
        dict(name="step_4096", kind="step", n=4096),
        # simulation and inference as separate kernels, a ragged batch
        dict(name="infer_1000003", kind="infer", n=1000003),
        # the small rollout of the configurations
        dict(name="rollout_1024x200", kind="rollout", n=1024, T=200, prec="f32"),
        # the compute-bound rollout of the configurations, each precision
        dict(name="rollout_1048576x1000", kind="rollout", n=1 << 20, T=1000, prec="f32"),
        dict(name="rollout_f64_1048576x1000", kind="rollout", n=1 << 20, T=1000, prec="f64"),
        dict(name="rollout_f16_1048576x1000", kind="rollout", n=1 << 20, T=1000, prec="f16"),
        # experience collection: every step's outputs kept
        dict(name="collect_4194304x64", kind="collect", n=1 << 22, T=64, prec="f32"),
        dict(name="collect_f16_3000001x50", kind="collect", n=3000001, T=50, prec="f16"),
        # one launch per step: the launch-bound configuration, and the
        # streaming one with the full trajectory
        dict(name="fused_65536x1000", kind="fused", n=65536, T=1000, traj=False),
        dict(name="fused_16777216x32", kind="fused", n=1 << 24, T=32, traj=True),
        # MLP policy: a learner's collection over a ragged small batch, and the
        # large configuration
        dict(name="policy_10007x128", kind="policy", n=10007, T=128, traj=True),
        dict(name="policy_4194304x500", kind="policy", n=1 << 22, T=500, traj=False),
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]: ragged in two
    draws of three, else a multiple of 64."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 1 / 3:
        v = (v + 32) // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["step", "infer", "rollout", "rollout", "collect", "collect", "fused",
                       "fused", "policy", "policy"])
    if kind in ("step", "infer"):
        return dict(kind=kind, n=_log_int(rng, 1024, 1 << 22))
    if kind == "rollout":
        return dict(kind=kind, n=_log_int(rng, 1024, 1 << 20), T=_log_int(rng, 100, 1000),
                    prec=rng.choice(["f32", "f64", "f16"]))
    if kind == "collect":
        return dict(kind=kind, n=_log_int(rng, 4096, 1 << 22), T=_log_int(rng, 16, 64),
                    prec=rng.choice(["f32", "f32", "f64", "f16"]))
    if kind == "fused":
        if rng.random() < 0.5:
            return dict(kind=kind, n=_log_int(rng, 1 << 21, 1 << 24), T=_log_int(rng, 8, 32), traj=True)
        return dict(kind=kind, n=_log_int(rng, 4096, 1 << 20), T=_log_int(rng, 64, 1000), traj=False)
    if rng.random() < 0.5:
        return dict(kind=kind, n=_log_int(rng, 1024, 1 << 18), T=_log_int(rng, 16, 128), traj=True)
    return dict(kind=kind, n=_log_int(rng, 4096, 1 << 22), T=_log_int(rng, 100, 500), traj=False)


# ---------------------------------------------------------------- inputs
def _typical_states(n, seed):
    """[4, n] states inside the limits with moderate velocities, as an agent
    meets them in mid-episode (drawn on the GPU)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.rand((4, n), generator=g, device="cuda", dtype=torch.float32) * 2.0 - 1.0
    return u * torch.tensor([[2.4], [2.0], [0.2094], [2.0]], device="cuda")


def _actions(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    return torch.randint(0, 2, (n,), generator=g, device="cuda", dtype=torch.uint8)


def _weights(seed):
    return synth.policy_weights(seed)


def _weights_gpu(seed):
    return torch.from_numpy(_weights(seed).view(np.int16)).cuda()


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    st = {"kind": kind, "seed": seed}
    if kind in ("step", "infer"):
        s = cp.CartPoleStates(n, variant=cp.CP_FUSED, graphs=False)
        cp.cp_init(s, seed)
        for dst, src in zip((s.x, s.x_dot, s.theta, s.theta_dot), _typical_states(n, seed)):
            dst.copy_(src)
        st.update(s=s, obs=s.state(), reward=torch.empty(n, device="cuda"),
                  done=torch.empty(n, dtype=torch.uint8, device="cuda"))
        if kind == "step":
            st["actions"] = _actions(n, seed)
        else:
            st["w"] = _weights_gpu(seed)
            st["actions"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        return st
    traj = kind == "collect" or (kind in ("fused", "policy") and case["traj"])
    prec = case.get("prec", "f32")
    s = cp.CartPoleStates(n, variant=cp.CP_FUSED if kind == "fused" else cp.CP_RESIDENT,
                          precision=prec, policy_w=_weights_gpu(seed) if kind == "policy" else None)
    cp.cp_init(s, seed)
    tr = cp.Trajectory(n, case["T"], obs=traj, reward=traj, done=traj, dtype=s.dtype)
    st.update(s=s, tr=tr, T=case["T"])
    return st


def run(st):
    s = st["s"]
    if st["kind"] in ("step", "infer"):
        if st["kind"] == "infer":
            cp.cp_policy(st["obs"], st["w"], st["actions"])
        cp.cp_step(s, st["actions"], st["obs"], st["reward"], st["done"])
        return {"x": s.x, "x_dot": s.x_dot, "theta": s.theta, "theta_dot": s.theta_dot,
                "ep_index": s.ep_index, "ep_len": s.ep_len, "obs": st["obs"],
                "reward": st["reward"], "done": st["done"], "actions": st["actions"]}
    tr = st["tr"]
    cp.cp_rollout(s, st["T"], st["seed"], tr)
    return {"x": s.x, "x_dot": s.x_dot, "theta": s.theta, "theta_dot": s.theta_dot,
            "ep_index": s.ep_index, "ep_len": s.ep_len, "obs": tr.obs, "reward": tr.reward,
            "done": tr.done, "done_count": tr.done_count, "total_reward": tr.total_reward,
            "ret_sum": tr.ret_sum, "totals": tr.totals}


def work(case):
    kind, n = case["kind"], case["n"]
    if kind in ("step", "infer"):
        # state and counters read and written (48 B), the action read, obs,
        # reward and done written
        b, f = n * (48 + 1 + 21), n * STEP_FLOPS
        if kind == "infer":
            b, f = b + n * 16 + 8960, f + n * POLICY_FLOPS
        return {"bytes": b, "flops": f}
    e, T = ELEM[case.get("prec", "f32")], case["T"]
    traj = kind == "collect" or (kind in ("fused", "policy") and case["traj"])
    # state and counters in and out, the statistics, and every step's rows
    b = n * (2 * (4 * e + 8) + 12 + (T * (4 * e + 5) if traj else 0)) + 16
    f = n * T * STEP_FLOPS
    if kind == "policy":
        b, f = b + 8960, f + n * T * POLICY_FLOPS
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Random-action rollouts are defined bit for bit: every operation of a
    step rounded once in the state's precision, the same at every fusion
    level and launch shape; one rounding moved would end some episode a step
    earlier or later and change all that follows.  A single step with given
    actions: an ulp or two per value.

    With the MLP policy, binary32 sums in another order choose another action
    where two logits nearly tie, for about 1 environment-step in 4,000,000
    (measured).  Such an environment gets other velocities, or ends its episode
    at another step, and is another one from there on.  Allowed: four times
    that share, and one environment in a small batch."""
    if case["kind"] == "step":
        return {"rel": 1e-6, "max": 1e-5}
    if case["kind"] in ("infer", "policy"):
        share = 1e-6 * case.get("T", 1) + 1.5 / case["n"]
        return {"rel": 1.4 * math.sqrt(share), "max": 0.99, "differ": share}
    return "exact"


# ---------------------------------------------------------------- 64 bits
M32 = 0xFFFFFFFF


def _threefry(k0, k1, c0, c1):
    """Threefry-2x32-20 on int64 tensors holding 32-bit values."""
    ks = (k0, k1, k0 ^ k1 ^ 0x1BD11BDA)
    x0, x1 = (c0 + ks[0]) & M32, (c1 + ks[1]) & M32
    for r in range(20):
        rot = (13, 15, 26, 6, 17, 29, 16, 24)[r % 8]
        x0 = (x0 + x1) & M32
        x1 = (((x1 << rot) | (x1 >> (32 - rot))) & M32) ^ x0
        if r % 4 == 3:
            j = r // 4 + 1
            x0, x1 = (x0 + ks[j % 3]) & M32, (x1 + ks[(j + 1) % 3] + j) & M32
    return x0, x1


def _stream_key(seed, tag):
    a, b = _threefry(seed >> 32, seed & M32, torch.tensor([tag]), torch.tensor([0]))
    return int(a), int(b)


def _start_states(key, env, k, f64):
    """[4, m] start states of episodes k of environments env, as binary64:
    the binary32 draw, or at binary64 the same halves scaled in binary64."""
    a, b = _threefry(key[0], key[1], env, k)
    h = torch.stack([a & 0xFFFF, a >> 16, b & 0xFFFF, b >> 16]) - 32768
    if f64:
        return h.double() * (0.1 * 2.0 ** -16)
    scale = torch.tensor(0.1, dtype=torch.float32, device=h.device) * 2.0 ** -16
    return (h.float() * scale).double()


class _Sim:
    """The environments in binary64, constants rounded to the case's precision."""

    def __init__(self, n, seed, f64):
        c = float if f64 else (lambda v: float(np.float32(v)))
        self.f64, self.env = f64, torch.arange(n, device="cuda")
        self.key = _stream_key(seed, 2)
        self.g, self.tau, self.l, self.mp = c(9.8), c(0.02), 0.5, c(0.1)
        self.mass = c(self.mp + 1.0)
        self.pml, self.four3 = c(self.mp * 0.5), c(4.0 / 3.0)
        self.xl, self.tl = c(2.4), c(12 * 2 * math.pi / 360)
        self.k = torch.zeros(n, dtype=torch.int64, device="cuda")
        self.s = _start_states(self.key, self.env, self.k, f64)

    def step(self, right):
        x, xd, th, thd = self.s
        sn, co = torch.sin(th), torch.cos(th)
        force = torch.where(right, 10.0, -10.0).double()
        temp = (force + self.pml * thd * thd * sn) / self.mass
        acc = (self.g * sn - co * temp) / (self.l * (self.four3 - self.mp * co * co / self.mass))
        xacc = temp - self.pml * acc * co / self.mass
        s = torch.stack([x + self.tau * xd, xd + self.tau * xacc, th + self.tau * thd,
                         thd + self.tau * acc])
        done = (s[0].abs() > self.xl) | (s[2].abs() > self.tl)
        at = done.nonzero()[:, 0]
        self.k[at] += 1
        s[:, at] = _start_states(self.key, self.env[at], self.k[at], self.f64)
        self.s = s
        return done


def _bf16(v):
    return v.float().bfloat16().double()


def _mlp(w, s):
    """Which environments the policy pushes right: bf16 inputs and hidden
    activations as the network is defined, sums and tanh in binary64."""
    w = torch.from_numpy(w.astype(np.int32) << 16).view(torch.float32).double().cuda()
    w1, w2, w3 = w[:256].view(4, 64), w[256:4352].view(64, 64), w[4352:].view(64, 2)
    out = torch.empty(s.shape[1], dtype=torch.bool, device="cuda")
    for a in range(0, s.shape[1], 1 << 20):
        o = _bf16(s[:, a:a + (1 << 20)]).t().contiguous()
        h = _bf16(torch.tanh(_bf16(torch.tanh(o @ w1)) @ w2))
        z = h @ w3
        out[a:a + (1 << 20)] = z[:, 1] > z[:, 0]
    return out


def exact(case, seed):
    """run()'s floating outputs at 64 bits.  None for binary16, whose results
    are the roundings themselves, and for policy rollouts: where two
    logits nearly tie, both actions are correct."""
    kind, n = case["kind"], case["n"]
    if kind == "policy" or case.get("prec") == "f16":
        return None
    f64 = case.get("prec") == "f64"
    sim = _Sim(n, seed, f64)
    whole = dict.fromkeys(("ep_index", "ep_len", "done", "actions", "done_count", "ret_sum", "totals"))
    if kind in ("step", "infer"):
        sim.s = _typical_states(n, seed).double()
        right = _mlp(_weights(seed), sim.s) if kind == "infer" else _actions(n, seed) != 0
        sim.step(right)
        x, xd, th, thd = sim.s
        return {**whole, "x": x, "x_dot": xd, "theta": th, "theta_dot": thd, "obs": sim.s,
                "reward": torch.ones(n, device="cuda", dtype=torch.float64)}
    whole.pop("actions")
    T = case["T"]
    traj = kind == "collect" or (kind == "fused" and case["traj"])
    obs = torch.empty((T, 4, n), dtype=torch.float64, device="cuda") if traj else None
    key = _stream_key(seed, 1)
    blocks = torch.arange((n + 63) // 64, device="cuda")
    bit = torch.arange(32, device="cuda")
    for t in range(T):
        a, b = _threefry(key[0], key[1], blocks, torch.full_like(blocks, t))
        right = (torch.stack([a, b], 1)[:, :, None] >> bit & 1).view(-1)[:n] != 0
        sim.step(right)
        if traj:
            obs[t] = sim.s
    x, xd, th, thd = sim.s
    return {**whole, "x": x, "x_dot": xd, "theta": th, "theta_dot": thd, "obs": obs,
            "reward": torch.ones((T, n), dtype=torch.float64, device="cuda") if traj else None,
            "total_reward": torch.full((n,), float(T), dtype=torch.float64, device="cuda")}
