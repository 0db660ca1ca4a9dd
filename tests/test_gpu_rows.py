"""Trajectories whose rows do not start on 128-byte lines, stored by block in
whole rows: the whole-rollout kernel (blocks of 512 and 1,024) and the streaming
step, against the kernels that store by waves, bit for bit.  The rows path of
the whole-rollout kernel is chosen by the batch and the trajectory's bytes, so
the sizes sit just past that (or, by waves, just before; the CPU test of the
rule checks the kernel of each); the other side is the same rollout in launches
too short for it."""
import pytest
import torch

import paper_2301_13062_amd as cp

pytestmark = pytest.mark.gpu


def rollout(variant, n, T, prec, env_base=0, per_launch=0, shift=0):
    s = cp.CartPoleStates(n, variant=variant, precision=prec, steps_per_launch=per_launch,
                          env_base=env_base)
    cp.cp_init(s, 4)
    s.theta_dot += 0.4
    tr = cp.Trajectory(n, T, dtype=s.dtype)
    if shift:  # the arrays of an aligned n, started `shift` elements later
        tr.obs = torch.empty(T * 4 * n + shift, dtype=s.dtype, device="cuda")[shift:].view(T, 4, n)
        tr.reward = torch.empty(T * n + shift, device="cuda")[shift:].view(T, n)
        tr.done = torch.empty(T * n + shift, dtype=torch.uint8, device="cuda")[shift:].view(T, n)
    for t in (tr.obs, tr.reward):
        t.fill_(-3.0)
    tr.done.fill_(7)
    cp.cp_rollout(s, T, 6, tr)
    torch.cuda.synchronize()
    return s, tr


def same(a, b):
    (s, tr), (s2, tr2) = a, b
    for f in ("x", "x_dot", "theta", "theta_dot", "ep_index", "ep_len"):
        assert torch.equal(getattr(s, f), getattr(s2, f)), f
    for f in ("obs", "reward", "done", "done_count", "total_reward", "ret_sum", "totals"):
        assert torch.equal(getattr(tr, f), getattr(tr2, f)), f


# precision, environments, steps, env_base, elements that the arrays are
# shifted by, threads per block of the rows kernel (0: by waves)
CASES = [
    ("f32", 300007, 64, 0, 0, 512), ("f32", 400001, 49, 37, 0, 1024),
    ("f32", 524289, 40, 0, 0, 0), ("f32", 524287, 40, 0, 0, 1024),
    ("f32", 500016, 41, 64, 0, 1024), ("f32", 1048576, 20, 0, 5, 1024),
    ("f32", 2500009, 8, 0, 0, 1024),
    ("f64", 200003, 55, 0, 0, 512), ("f64", 409601, 29, 1, 0, 1024),
    # the least batches, and one environment less; a long rollout of a small one
    ("f32", 196097, 98, 0, 0, 512), ("f32", 196096, 98, 0, 5, 0),
    ("f32", 128001, 150, 0, 0, 512), ("f32", 127999, 150, 0, 0, 0),
    ("f64", 97793, 112, 0, 0, 512), ("f64", 97792, 112, 0, 1, 0),
    ("f32", 4097, 4700, 0, 0, 0), ("f64", 4097, 2700, 3, 0, 0), ("f16", 10001, 7300, 0, 0, 0),
    # binary16: a last block of a few environments, one short of full, rows off
    # the lines by the arrays' starts alone; by waves
    ("f16", 1000003, 73, 0, 0, 1024), ("f16", 1036287, 71, 64, 0, 1024),
    ("f16", 1048576, 70, 0, 3, 1024), ("f16", 1000003, 35, 0, 0, 0),
    ("f16", 700002, 50, 64, 0, 0), ("f16", 1048575, 31, 64, 0, 0),
    ("f16", 655360, 50, 0, 3, 0), ("f16", 1100001, 66, 0, 0, 0)]


@pytest.mark.parametrize("prec,n,T,env_base,shift,block", CASES)
def test_resident_rows(gpu, prec, n, T, env_base, shift, block):
    whole = rollout(cp.CP_RESIDENT, n, T, prec, env_base, 0, shift)
    same(whole, rollout(cp.CP_RESIDENT, n, T, prec, env_base, 7))


@pytest.mark.parametrize("n,T,shift", [(2097153, 3, 0), (2097152 + 511, 5, 0),
                                       (2097152 + 528, 2, 0), (2097152, 4, 1)])
def test_streaming_rows(gpu, n, T, shift):
    same(rollout(cp.CP_FUSED, n, T, "f32", 0, 0, shift), rollout(cp.CP_RESIDENT, n, T, "f32", 0, 1))
