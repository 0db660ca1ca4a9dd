"""The whole-rollout loop's actions held per lane (a wave's 64 steps transposed)
and its start states held ahead, over several blocks of 64 steps and many
terminations, against launches of one step each (whose actions and start states
are the first of each launch) and the fused step (which draws them by other
code), bit for bit."""
import pytest
import torch

import paper_2301_13062_amd as cp

pytestmark = pytest.mark.gpu

NAMES = ("x", "x_dot", "theta", "theta_dot", "ep_index", "ep_len")


def run(variant, n, T, t0, prec, env_base, per_launch, kick):
    s = cp.CartPoleStates(n, variant=variant, precision=prec, steps_per_launch=per_launch,
                          env_base=env_base, graphs=False)
    cp.cp_init(s, 8)
    s.theta_dot[::3] += kick  # a third of the episodes end at once
    s.t = t0
    tr = cp.Trajectory(n, T, obs=False, reward=False, done=False, dtype=s.dtype)
    cp.cp_rollout(s, T, 11, tr)
    torch.cuda.synchronize()
    return [getattr(s, f) for f in NAMES] + [tr.done_count, tr.ret_sum, tr.totals]


@pytest.mark.parametrize("prec", ["f32", "f64", "f16"])
@pytest.mark.parametrize("n,env_base", [(63, 0), (129, 1), (1030, 63), (700, 128), (300, 4294966996)])
def test_actions_and_start_states(gpu, prec, n, env_base):
    for t0, T, kick in [(0, 64, 0.0), (31, 34, 9.0), (32, 100, 0.0), (61, 523, 9.0)]:
        print(prec, n, env_base, t0, T, flush=True)
        whole = run(cp.CP_RESIDENT, n, T, t0, prec, env_base, 0, kick)
        others = [run(cp.CP_RESIDENT, n, T, t0, prec, env_base, 1, kick)]
        if prec == "f32":
            others.append(run(cp.CP_FUSED, n, T, t0, prec, env_base, 0, kick))
        for other in others:
            for k, (a, b) in enumerate(zip(whole, other)):
                assert torch.equal(a, b), (t0, T, k)
