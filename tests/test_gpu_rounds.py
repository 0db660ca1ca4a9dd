"""The whole-rollout loop's groups of steps -- the first step, single steps up
to a multiple of eight of the global step, rounds of eight, the rest -- and
its forms by outputs, against launches of one step each (which run the first
step's code alone), bit for bit."""
import pytest
import torch

import paper_2301_13062_amd as cp

pytestmark = pytest.mark.gpu


def bits(t):
    if t is None:
        return None
    return t.contiguous().view(torch.uint8).cpu()


def run(n, T, t0, prec, per_launch, env_base, outs):
    s = cp.CartPoleStates(n, variant=cp.CP_RESIDENT, precision=prec, steps_per_launch=per_launch,
                          env_base=env_base)
    cp.cp_init(s, 3)
    s.theta_dot += 0.5  # some episodes end early
    s.t = t0
    tr = cp.Trajectory(n, T, obs="o" in outs, reward="r" in outs, done="d" in outs, dtype=s.dtype)
    cp.cp_rollout(s, T, 5, tr)
    torch.cuda.synchronize()
    return [bits(t) for t in (s.x, s.x_dot, s.theta, s.theta_dot, s.ep_index, s.ep_len, tr.obs,
                              tr.reward, tr.done, tr.done_count, tr.total_reward, tr.ret_sum,
                              tr.totals)]


@pytest.mark.parametrize("prec", ["f32", "f64", "f16"])
@pytest.mark.parametrize("n,env_base,outs", [(1, 0, ""), (65, 0, "ord"), (321, 37, "ord"),
                                             (130, 64, "d"), (257, 1, "or")])
def test_groups_of_steps(gpu, prec, n, env_base, outs):
    for t0, T in [(0, 1), (0, 2), (0, 8), (0, 9), (7, 9), (5, 16), (63, 33), (1, 40), (8, 130)]:
        print(prec, n, env_base, outs, t0, T, flush=True)
        whole = run(n, T, t0, prec, 0, env_base, outs)
        ones = run(n, T, t0, prec, 1, env_base, outs)
        for k, (a, b) in enumerate(zip(whole, ones)):
            assert (a is None and b is None) or torch.equal(a, b), (t0, T, k)
