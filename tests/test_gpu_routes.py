"""A call is not much slower than its neighbour on the other side of a dispatch's line.  Each pair
does the same work or the second a little more; the bound leaves 40% for noise, and what it
guards against was 1.6 to 12 times."""
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
