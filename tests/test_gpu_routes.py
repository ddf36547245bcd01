"""A call is not much slower than its neighbour on the other side of a dispatch's line.  Each pair
does the same work or the second a little more; the bounds lie between what was measured (up to 1.0,
sequence weights and the loose bound 1.4) and what they guard against (1.6 to 200)."""
import pytest
import torch

from helpers import log

pytestmark = pytest.mark.gpu


def _us(call, n=20, repeats=9):
    """Microseconds a call among others: the fastest of several batches."""
    call()
    best = float("inf")
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(n):
            call()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) / n * 1e3)
    return best


def _not_slower(name, call, other, bound=1.4):
    a, b = _us(call), _us(other)
    a, b = min(a, _us(call)), min(b, _us(other))
    log(f"{name}: {a:.1f} us against {b:.1f}")
    assert a <= bound * b, (name, a, b)


# the compaction in one launch up to 2^16 tokens, in three beyond
@pytest.mark.parametrize("T", [1 << 16, 1 << 18])
def test_compaction_line(T):
    import paper_2510_04206_amd as P
    V, d, n_act = 300, 64, 64

    def call(T):
        g = torch.Generator(device="cuda").manual_seed(1)
        H = torch.randn((T, d), generator=g, device="cuda").bfloat16()
        W = torch.randn((V, d), generator=g, device="cuda").bfloat16()
        y = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
        mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
        mask[torch.randperm(T, generator=g, device="cuda")[:n_act]] = 1
        lp = P.TokenLogprob(T, d, V, H.dtype, max_act=n_act)
        return lambda: lp(H, W, y, mask)

    _not_slower(f"log-prob pass, T={T}", call(T), call(T + 256))


# a bound of every token of a long batch against the bound that its few action tokens need
def test_forward_with_a_loose_bound():
    import paper_2510_04206_amd as P
    T, V, d, n_act = 281575, 300, 64, 3
    g = torch.Generator(device="cuda").manual_seed(3)
    H = torch.randn((T, d), generator=g, device="cuda").bfloat16()
    W = torch.randn((V, d), generator=g, device="cuda").bfloat16()
    y = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    mask[torch.randperm(T, generator=g, device="cuda")[:n_act]] = 1
    adv, old = torch.randn(T, generator=g, device="cuda"), torch.full((T,), -6.0, device="cuda")
    pl = {m: P.PolicyLoss(T, d, V, H.dtype, max_act=m) for m in (0, n_act)}
    call = lambda m: lambda: pl[m].forward(H, W, y, mask, adv, old)      # noqa: E731
    _not_slower("forward, loose bound", call(0), call(n_act), bound=2.2)
    assert pl[0].loss.item() == pl[n_act].loss.item()


def _tokens(T, n_traj, offset):
    """Ids in runs and a mask that start `offset` elements into their arrays, and an output."""
    g = torch.Generator(device="cuda").manual_seed(2)
    ids = torch.randint(0, n_traj, (T + offset,), generator=g, device="cuda", dtype=torch.int32).sort()[0]
    mask = (torch.rand(T + offset, generator=g, device="cuda") < 0.4).to(torch.uint8)
    return ids[offset:], mask[offset:], torch.empty(T + offset, device="cuda")[offset:]


# arrays cut out of a longer token stream against aligned ones
@pytest.mark.parametrize("offset", [1, 4])
def test_sequence_weights_unaligned(offset):
    import paper_2510_04206_amd as P
    T, n_traj = 65536, 640
    count = torch.empty(n_traj, dtype=torch.int32, device="cuda")

    def call(offset):
        ids, mask, w = _tokens(T, n_traj, offset)
        return lambda: P.agrl_sequence_mean_weights(T, n_traj, ids, mask, count, w)

    _not_slower(f"sequence weights at offset {offset}", call(offset), call(0), bound=2.0)


def _adv_call(n_traj, n_group, n_task, T, offset=0):
    import paper_2510_04206_amd as P
    ids, mask, tok = _tokens(T, max(n_traj, 1), offset)
    dev = dict(device="cuda")
    task = torch.arange(n_traj, dtype=torch.int32, **dev) % n_task
    group = torch.arange(n_traj, dtype=torch.int32, **dev) % n_group if n_group else None
    reward = torch.rand(n_traj, **dev)
    outs = (torch.empty(n_traj, dtype=torch.int32, **dev), torch.empty(n_task, dtype=torch.int64, **dev),
            torch.empty(n_task, **dev), torch.empty(n_task, **dev), torch.empty(n_traj, **dev), tok)
    ranges = torch.empty(2 * (n_group + n_task), dtype=torch.int32, **dev)
    opt = P.agrl_options(adv_ranges=ranges.data_ptr())
    keep = (ranges,)
    return lambda: (P.agrl_task_adv_norm(T, n_traj, n_task, n_group, ids, mask, task, group, reward, opt,
                                         *outs), keep)


@pytest.mark.parametrize("offset", [1, 4])
def test_advantages_of_a_small_batch_unaligned(offset):
    _not_slower(f"advantages at offset {offset}", _adv_call(512, 64, 8, 32000, offset), _adv_call(512, 64, 8, 32000),
                bound=1.6)


# many segments and few trajectories, which one workgroup once took, against more trajectories
@pytest.mark.parametrize("n_traj,n_group,n_task", [(0, 0, 100000), (1, 0, 65535), (8, 8, 8000), (256, 250, 6)])
def test_advantages_of_many_segments(n_traj, n_group, n_task):
    T = 1000 if n_traj else 0
    _not_slower(f"advantages of {n_traj} trajectories, {n_group} groups, {n_task} tasks",
                _adv_call(n_traj, n_group, n_task, T), _adv_call(1025, n_group, n_task, 1000))
