"""Launches of few steps -- a rollout in pieces of one to nine steps, whose
actions come from the generator's outputs by other code than a long launch's --
against the whole rollout in one launch; and batches with angles beyond 1/4,
infinities and NaN in waves that the batch fills in part, against launches of one
step each and the fused step."""
import math

import pytest
import torch

import paper_2301_13062_amd as cp

pytestmark = pytest.mark.gpu

STATE = ("x", "x_dot", "theta", "theta_dot", "ep_index", "ep_len")
OUT = ("obs", "reward", "done", "done_count", "total_reward", "ret_sum", "totals")


def rollout(variant, n, T, t0, prec, env_base, per_launch, traj, prepare):
    s = cp.CartPoleStates(n, variant=variant, precision=prec, env_base=env_base,
                          steps_per_launch=per_launch, graphs=False)
    cp.cp_init(s, 12)
    prepare(s)
    s.t = t0
    tr = cp.Trajectory(n, T, obs=traj, reward=traj, done=traj, dtype=s.dtype)
    cp.cp_rollout(s, T, 21, tr)
    torch.cuda.synchronize()
    return [getattr(s, f) for f in STATE] + [getattr(tr, f) for f in OUT]


def same(a, b, where):
    for f, u, v in zip(STATE + OUT, a, b):
        if u is not None:
            assert torch.equal(torch.nan_to_num(u.double(), nan=-1e300),
                               torch.nan_to_num(v.double(), nan=-1e300)), (where, f)


def kick(s):
    s.theta_dot[::2] += 12.0  # half of the episodes end at the first step


@pytest.mark.parametrize("prec", ["f32", "f64", "f16"])
@pytest.mark.parametrize("n,env_base,traj", [(1, 0, False), (100, 37, False), (321, 0, True),
                                             (130, 5, True), (300, 4294966996, False)])
def test_pieces(gpu, prec, n, env_base, traj):
    T, t0 = 75, 59  # across two multiples of 64
    whole = rollout(cp.CP_RESIDENT, n, T, t0, prec, env_base, 0, traj, kick)
    for per_launch in (1, 2, 3, 4, 5, 8, 9):
        print(prec, n, env_base, traj, per_launch, flush=True)
        same(whole, rollout(cp.CP_RESIDENT, n, T, t0, prec, env_base, per_launch, traj, kick),
             per_launch)


def unusual(s):
    n = s.n
    values = [0.3, -2.0, 100.0, math.inf, math.nan, 0.2, -math.inf, 0.25]
    for k, v in enumerate(values):
        s.theta[k::13] = v
    s.x[5::17] = math.nan
    s.x[6::17] = math.inf
    s.theta_dot[7::19] = -3.0  # back within the limit from beyond it
    assert n > 8


@pytest.mark.parametrize("prec", ["f32", "f64", "f16"])
@pytest.mark.parametrize("n,env_base", [(9, 0), (100, 0), (257, 64), (70, 3)])
def test_unusual_states(gpu, prec, n, env_base):
    whole = rollout(cp.CP_RESIDENT, n, 20, 0, prec, env_base, 0, True, unusual)
    print(prec, n, env_base, flush=True)
    same(whole, rollout(cp.CP_RESIDENT, n, 20, 0, prec, env_base, 1, True, unusual), "one step")
    if prec == "f32":
        same(whole, rollout(cp.CP_FUSED, n, 20, 0, prec, env_base, 0, True, unusual), "fused")
