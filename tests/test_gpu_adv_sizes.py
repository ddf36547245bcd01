"""Advantage normalisation and sequence weights where the launches change: one workgroup
for a small batch, one or several blocks presetting the member ranges, unaligned arrays.
Bit-exact against the oracle, trajectories numbered at random."""
import numpy as np
import pytest
import torch

import oracle

from helpers import log

pytestmark = pytest.mark.gpu


def _batch(n_traj, n_group, n_task, T, seed):
    rng = np.random.default_rng([seed, n_traj, T])
    group = rng.integers(0, n_group, n_traj).astype(np.int32)
    task = (group * n_task // n_group).astype(np.int32)
    reward = np.where(task % 2 == 0, rng.random(n_traj) < 0.5, rng.normal(0, 1, n_traj)).astype(np.float32)
    cuts = np.sort(rng.integers(0, T + 1, n_traj - 1)) if n_traj > 1 else np.zeros(0, int)
    ids = np.repeat(rng.permutation(n_traj), np.diff(np.concatenate([[0], cuts, [T]]))).astype(np.int32)
    ids[rng.random(T) < 0.02] = -1
    return task, group, reward, ids, (rng.random(T) < 0.4).astype(np.uint8)


@pytest.mark.parametrize("n_traj,n_group,n_task,T,offset", [
    (1, 1, 1, 1, 0), (64, 3, 2, 1000, 1), (1024, 62, 2, 32768, 0), (1024, 62, 2, 32769, 0),
    (1024, 63, 2, 5003, 0), (1025, 60, 2, 4000, 3), (4096, 4000, 96, 60001, 0),
    (4097, 1000, 7, 60001, 0), (5000, 4500, 20, 9000, 5),
    # the most segments that one workgroup takes, and one more
    (256, 240, 16, 3000, 0), (256, 241, 16, 3000, 0), (1024, 80, 16, 32000, 1), (1024, 81, 16, 32000, 1),
    (3, 112, 74, 2000, 0), (3, 113, 74, 2000, 0), (3, 4000, 3000, 200, 0)])
@pytest.mark.parametrize("drop", [False, True])
def test_adv_norm_sizes(n_traj, n_group, n_task, T, offset, drop):
    import paper_2510_04206_amd as P
    task, group, reward, ids, mask = _batch(n_traj, n_group, n_task, T, 3)
    log(f"adv sizes n_traj={n_traj} groups={n_group} tasks={n_task} T={T} offset={offset} drop={drop}")

    def t(a):
        return torch.from_numpy(a).cuda()

    def at(a):           # the same values `offset` elements into an aligned array
        return torch.cat([torch.zeros(offset, dtype=t(a).dtype, device="cuda"), t(a)])[offset:]

    want = oracle.task_adv_norm(ids, mask, task, group, reward, n_task, n_group, drop_uniform=drop)
    for ranges in (True, False):
        got = P.task_adv_norm(at(ids), at(mask), t(task), t(group), t(reward), n_task, n_group,
                              opt=dict(drop_uniform_groups=int(drop)), member_ranges=ranges)
        assert P.agrl_get_device_error() == 0
        for k in ("act_count", "task_count", "task_mean", "task_std", "adv_traj", "adv_tok"):
            a, b = got[k].cpu().numpy(), np.asarray(want[k])
            if a.dtype == np.float32:
                a, b = a.view(np.uint32), b.view(np.uint32)
            np.testing.assert_array_equal(a, b, err_msg=f"{k} ranges={ranges}")


@pytest.mark.parametrize("n_traj,T,offset", [
    (1, 1, 0), (7, 100, 3), (4096, 65536, 0), (4096, 65535, 1), (4097, 3000, 0), (64, 65537, 0)])
def test_sequence_weight_sizes(n_traj, T, offset):
    import paper_2510_04206_amd as P
    _, _, _, ids, mask = _batch(n_traj, n_traj, 1, T + offset, 5)
    log(f"sequence weight sizes n_traj={n_traj} T={T} offset={offset}")
    count, w = P.sequence_mean_weights(torch.from_numpy(ids).cuda()[offset:],
                                       torch.from_numpy(mask).cuda()[offset:], n_traj)
    assert P.agrl_get_device_error() == 0
    want_count, want_w = oracle.sequence_mean_weights(ids[offset:], mask[offset:], n_traj)
    np.testing.assert_array_equal(count.cpu().numpy(), want_count)
    np.testing.assert_array_equal(w.cpu().numpy().view(np.uint32), want_w.view(np.uint32))


# a lane's 16 tokens with no, one (at each place) and several changes of trajectory, ids that
# are skipped among them; any nonzero mask byte is an action token
@pytest.mark.parametrize("T,n_traj", [(4096, 256), (70000, 5000)])
def test_count_trajectory_changes(T, n_traj):
    import paper_2510_04206_amd as P
    rng = np.random.default_rng(T)
    ids = np.repeat(rng.integers(-1, n_traj, T // 16 + 1), 16)[:T].astype(np.int32)
    for at in range(T // 16):
        if at % 3:
            ids[16 * at + at % 16:16 * at + 16] = rng.integers(-1, n_traj)
        if at % 7 == 0:
            ids[16 * at + 5:16 * at + 9] = rng.integers(0, n_traj)
    mask = np.where(rng.random(T) < 0.5, rng.integers(1, 256, T), 0).astype(np.uint8)
    log(f"trajectory changes T={T}")
    count, _ = P.sequence_mean_weights(torch.from_numpy(ids).cuda(), torch.from_numpy(mask).cuda(), n_traj)
    assert P.agrl_get_device_error() == 0
    want = np.bincount(ids[(mask != 0) & (ids >= 0)], minlength=n_traj)
    np.testing.assert_array_equal(count.cpu().numpy(), want)


# ids, mask and token outputs that start anywhere in their arrays, each by itself: runs of 16
# and of 4 tokens cut at both ends, one workgroup (1023 trajectories) and several launches
@pytest.mark.parametrize("n_traj", [1023, 5000])
@pytest.mark.parametrize("T", [1, 3, 15, 16, 17, 33, 4099, 66001])
@pytest.mark.parametrize("o_id,o_mask,o_out", [(0, 1, 0), (1, 0, 2), (1, 1, 1), (3, 15, 3), (0, 4, 1), (2, 17, 0)])
def test_arrays_that_start_anywhere(n_traj, T, o_id, o_mask, o_out):
    import paper_2510_04206_amd as P
    task, group, reward, ids, mask = _batch(n_traj, 40, 3, T, 7)
    mask = mask * np.random.default_rng(T).integers(1, 256, T).astype(np.uint8)
    log(f"arrays at {o_id}, {o_mask}, {o_out}: n_traj={n_traj} T={T}")

    def at(a, k):        # `a` from element k on of a larger array whose other elements would count
        t = torch.from_numpy(a).cuda()
        pad = torch.full((k + 16,), 1, dtype=t.dtype, device="cuda")
        return torch.cat([pad[:k], t, pad[k:]])[k:k + T]

    t_ids, t_mask = at(ids, o_id), at(mask, o_mask)
    dev = dict(device="cuda")
    outs = (torch.empty(n_traj, dtype=torch.int32, **dev), torch.empty(3, dtype=torch.int64, **dev),
            torch.empty(3, **dev), torch.empty(3, **dev), torch.empty(n_traj, **dev))
    whole = torch.full((2, T + o_out + 16), 7.0, **dev)
    tok, w = whole[0, o_out:o_out + T], whole[1, o_out:o_out + T]
    t = [torch.from_numpy(a).cuda() for a in (task, group, reward)]
    P.agrl_task_adv_norm(T, n_traj, 3, 40, t_ids, t_mask, *t, None, *outs, tok)
    count = torch.empty(n_traj, dtype=torch.int32, **dev)
    P.agrl_sequence_mean_weights(T, n_traj, t_ids, t_mask, count, w)
    assert P.agrl_get_device_error() == 0
    want = oracle.task_adv_norm(ids, mask, task, group, reward, 3, 40)
    want_count, want_w = oracle.sequence_mean_weights(ids, mask, n_traj)
    np.testing.assert_array_equal(outs[0].cpu().numpy(), want["act_count"])
    np.testing.assert_array_equal(outs[1].cpu().numpy(), want["task_count"])
    np.testing.assert_array_equal(count.cpu().numpy(), want_count)
    for a, b in ((outs[2], want["task_mean"]), (outs[3], want["task_std"]), (outs[4], want["adv_traj"]),
                 (tok, want["adv_tok"]), (w, want_w)):
        np.testing.assert_array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))
    assert (whole[:, :o_out] == 7).all() and (whole[:, o_out + T:] == 7).all()   # nothing beside them


# ids outside their ranges, in one workgroup's batch and in the launches': the error bit, and
# everything that the id does not touch as if its token were padding, or its trajectory apart
SIZES = [(64, 16, 4, 4096), (2000, 300, 20, 70000)]


def _call(ids, mask, task, group, reward, n_task, n_group, ranges=True):
    import paper_2510_04206_amd as P
    t = lambda a: torch.from_numpy(a).cuda()                         # noqa: E731
    out = P.task_adv_norm(t(ids), t(mask), t(task), t(group), t(reward), n_task, n_group, member_ranges=ranges)
    return {k: v.cpu().numpy() for k, v in out.items() if k != "member_ranges"}, P.agrl_get_device_error()


@pytest.mark.parametrize("n_traj,n_group,n_task,T", SIZES)
@pytest.mark.parametrize("run,place", [("first", 3), ("second", 9), ("whole", 0), ("third", 5)])
@pytest.mark.parametrize("action", [False, True])
def test_bad_trajectory_ids(n_traj, n_group, n_task, T, run, place, action):
    import paper_2510_04206_amd as P
    task, group, reward, ids, mask = _batch(n_traj, n_group, n_task, T, 11)
    ids = np.repeat(ids[::16], 16)[:T].copy()            # whole runs of 16 tokens
    at = 16 * (T // 40)
    bad = {"first": slice(at, at + place), "second": slice(at + place, at + 16), "whole": slice(at, at + 16),
           "third": slice(at + place, at + place + 4)}[run]
    ids[at:at + 16] = n_traj // 2
    if run == "third":
        ids[at + 12:at + 16] = 1
    ids[bad] = n_traj + (1 << 20)
    mask[bad] = action
    log(f"bad trajectory ids n_traj={n_traj} {run} action={action}")
    clean = np.where(ids >= n_traj, -1, ids).astype(np.int32)
    want = oracle.task_adv_norm(clean, mask, task, group, reward, n_task, n_group)
    got, err = _call(ids, mask, task, group, reward, n_task, n_group)
    assert err == 2
    for k in want:
        np.testing.assert_array_equal(np.asarray(got[k]).view(np.uint8), np.asarray(want[k]).view(np.uint8), err_msg=k)
    count, w = P.sequence_mean_weights(torch.from_numpy(ids).cuda(), torch.from_numpy(mask).cuda(), n_traj)
    assert P.agrl_get_device_error() == 2
    want_count, want_w = oracle.sequence_mean_weights(clean, mask, n_traj)
    np.testing.assert_array_equal(count.cpu().numpy(), want_count)
    np.testing.assert_array_equal(w.cpu().numpy().view(np.uint32), want_w.view(np.uint32))


@pytest.mark.parametrize("n_traj,n_group,n_task,T", SIZES)
@pytest.mark.parametrize("ranges", [True, False])
@pytest.mark.parametrize("what,value,bit", [("task", -1, 4), ("task", 1 << 20, 4), ("group", -5, 8), ("group", 1 << 20, 8)])
def test_bad_task_and_group_ids(n_traj, n_group, n_task, T, ranges, what, value, bit):
    task, group, reward, ids, mask = _batch(n_traj, n_group, n_task, T, 13)
    j = n_traj // 3
    good = (task.copy(), group.copy())
    good[what == "group"][j] = (n_task, n_group)[what == "group"]     # a task or group of its own
    touched = {"task": np.arange(n_traj) == j, "group": task == task[j]}[what]
    log(f"bad {what} id {value} n_traj={n_traj} ranges={ranges}")
    want = oracle.task_adv_norm(ids, mask, *good, reward, n_task + 1, n_group + 1)
    (task, group)[what == "group"][j] = value
    got, err = _call(ids, mask, task, group, reward, n_task, n_group, ranges)
    assert err == bit
    np.testing.assert_array_equal(got["act_count"], want["act_count"])
    np.testing.assert_array_equal(got["task_count"], want["task_count"][:n_task])
    np.testing.assert_array_equal(got["adv_traj"][~touched].view(np.uint32), want["adv_traj"][~touched].view(np.uint32))
    keep = np.ones(n_task, bool)
    if what == "group":
        keep[task[j]] = False
    for k in ("task_mean", "task_std"):
        np.testing.assert_array_equal(got[k][keep].view(np.uint32), want[k][:n_task][keep].view(np.uint32))
