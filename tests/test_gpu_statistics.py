"""Per-environment statistics of the per-step levels, which write them at a
rollout's first and last steps only, against the whole-rollout kernel: the
shortest rollouts, direct launches and graph replays, both sides of the large
fused step's threshold, counters that wrap."""
import pytest
import torch

import paper_2301_13062_amd as cp

pytestmark = pytest.mark.gpu


def stats(variant, n, T, calls, graphs=False, some=("done_count", "total_reward", "ret_sum")):
    s = cp.CartPoleStates(n, variant=variant, graphs=graphs)
    cp.cp_init(s, 2)
    s.theta_dot += 0.7
    s.ep_index -= 1  # 2^32 - 1: wraps at the first termination
    s.ep_len -= 2
    tr = cp.Trajectory(n, T, obs=False, reward=False, done=False, totals=False)
    for f in ("done_count", "total_reward", "ret_sum"):
        getattr(tr, f).fill_(-7)  # what was there does not count
        if f not in some:
            setattr(tr, f, None)
    for _ in range(calls):
        cp.cp_rollout(s, T, 9, tr)
    torch.cuda.synchronize()
    return s, tr


@pytest.mark.parametrize("T,calls,graphs", [(1, 1, False), (2, 2, False), (3, 1, False),
                                            (16, 3, True), (129, 3, True)])
@pytest.mark.parametrize("n", [1, 321, (1 << 21) + 5])
def test_first_and_last_step(gpu, n, T, calls, graphs):
    variants = [cp.CP_FUSED] if graphs else [cp.CP_FUSED, cp.CP_CONCAT]
    ref, want = stats(cp.CP_RESIDENT, n, T, calls)
    for v in variants:
        for some in (("done_count", "total_reward", "ret_sum"), ("ret_sum",), ("done_count",)):
            print(n, T, v, some, flush=True)
            s, tr = stats(v, n, T, calls, graphs, some)
            for f in some:
                assert torch.equal(getattr(tr, f), getattr(want, f)), (v, f)
            assert torch.equal(s.ep_index, ref.ep_index) and torch.equal(s.ep_len, ref.ep_len)
