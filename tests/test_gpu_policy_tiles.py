"""The MLP kernels' forms -- one, two or four tiles of 16 environments per
wave by the batch's size, activations with and without the clamp, weights
staged in wide or narrow loads -- give the same results, bit for bit: an
environment's result depends on itself alone."""
import numpy as np
import pytest
import torch

import paper_2301_13062_amd as cp
from paper_2301_13062_amd import synth

pytestmark = pytest.mark.gpu

SIZES = (1, 17, 16384 + 5, 49152, 49153, 131072, 131073)  # either side of each rule
T = 9


def weights(kind):
    w = (synth.policy_weights(4).astype(np.uint32) << 16).view(np.float32).copy()
    if kind == "wide":  # layer-2 sums past the clamp-free range
        w *= 8
    if kind == "infinite":
        w[3], w[300] = np.inf, -np.inf
    return torch.from_numpy((w.view(np.uint32) >> 16).astype(np.int16)).cuda()


def states(n):
    """Typical states; of every 32 environments one fast, one not a number
    (both need the clamps, for their whole wave)."""
    s = torch.from_numpy(synth.states(n, seed=6)).cuda()
    s[3, 7::32] = 40.0
    s[0, 21::64] = float("nan")
    return s


def rollout(w, st, n, traj):
    s = cp.CartPoleStates(n, variant=cp.CP_RESIDENT, policy_w=w)
    cp.cp_init(s, 1)
    for dst, src in zip((s.x, s.x_dot, s.theta, s.theta_dot), st):
        dst.copy_(src[:n])
    tr = cp.Trajectory(n, T, obs=traj, reward=traj, done=traj)
    cp.cp_rollout(s, T, 0, tr)
    torch.cuda.synchronize()
    return s, tr


def bits(t):
    return t.contiguous().view(torch.int32)


@pytest.mark.parametrize("kind", ["usual", "wide", "infinite"])
@pytest.mark.parametrize("traj", [False, True])
def test_sizes_agree(gpu, kind, traj):
    w = weights(kind)
    st = states(max(SIZES))
    ref, rtr = rollout(w, st, max(SIZES), traj)
    for n in SIZES[:-1]:
        print(kind, n, flush=True)
        s, tr = rollout(w, st, n, traj)
        assert torch.equal(bits(s.state()), bits(ref.state()[:, :n]))
        assert torch.equal(s.ep_index, ref.ep_index[:n]) and torch.equal(s.ep_len, ref.ep_len[:n])
        assert torch.equal(tr.ret_sum, rtr.ret_sum[:n])
        assert int(tr.totals[0]) == int(tr.done_count.sum())
        if traj:
            assert torch.equal(bits(tr.obs), bits(rtr.obs[:, :, :n]))
            assert torch.equal(tr.done, rtr.done[:, :n])


@pytest.mark.parametrize("n", [100, 50000, 140000])
def test_clamped_waves_leave_their_neighbours_alone(gpu, n):
    w = weights("usual")
    plain = torch.from_numpy(synth.states(n, seed=6)).cuda()
    a, _ = rollout(w, plain, n, False)
    mixed = plain.clone()
    mixed[0, 5::16] = float("nan")  # every wave takes the clamps
    b, _ = rollout(w, mixed, n, False)
    keep = torch.arange(n, device="cuda") % 16 != 5
    assert torch.equal(bits(a.state())[:, keep], bits(b.state())[:, keep])


@pytest.mark.parametrize("kind", ["usual", "wide"])
def test_policy_alone(gpu, kind):
    w = weights(kind)
    odd = torch.empty(w.numel() + 8, dtype=torch.int16, device="cuda")[1:1 + w.numel()]
    odd.copy_(w)  # 2-byte aligned only
    n = 1024 * 256 * 2 + 77  # three rounds of the blocks
    st = states(n).contiguous()
    ref = torch.empty(n, dtype=torch.uint8, device="cuda")
    cp.cp_policy(st, w, ref)
    act = torch.empty_like(ref)
    cp.cp_policy(st, odd, act)
    assert torch.equal(ref, act)
    for m in SIZES:
        print(kind, m, flush=True)
        part = torch.empty(m, dtype=torch.uint8, device="cuda")
        cp.cp_policy(st[:, :m].contiguous(), w, part)
        assert torch.equal(part, ref[:m])


@pytest.mark.parametrize("n", [8192, 8193, 16385, 40961])
@pytest.mark.parametrize("traj", [False, True])
def test_short_rollouts(gpu, n, traj):
    """Tiles by the launch's steps: a rollout in pieces on both sides of the
    rule (8,192 environments per step) against one launch."""
    w, st = weights("usual"), states(n)
    ref, rtr = rollout(w, st, n, traj)
    for per_launch in (1, 2, 4, 5):
        print(n, traj, per_launch, flush=True)
        s = cp.CartPoleStates(n, variant=cp.CP_RESIDENT, policy_w=w, steps_per_launch=per_launch)
        cp.cp_init(s, 1)
        for dst, src in zip((s.x, s.x_dot, s.theta, s.theta_dot), st):
            dst.copy_(src)
        tr = cp.Trajectory(n, T, obs=traj, reward=traj, done=traj)
        cp.cp_rollout(s, T, 0, tr)
        torch.cuda.synchronize()
        assert torch.equal(bits(s.state()), bits(ref.state()))
        assert torch.equal(s.ep_index, ref.ep_index) and torch.equal(tr.ret_sum, rtr.ret_sum)
        if traj:
            assert torch.equal(bits(tr.obs), bits(rtr.obs)) and torch.equal(tr.done, rtr.done)
