"""Logits that are NaN, +inf or -inf, in the forward and the log-prob pass: a token that has a
NaN or a +inf logit gets a non-finite lse and logp and the loss is not finite; -inf logits
carry no weight, also where a whole tile or half of one has no others.  Finite results
against log-sum-exp in 64 bits, with the tolerances of finite logits."""
import pytest
import torch

from helpers import LOGP_ATOL, LSE_ATOL, log

pytestmark = pytest.mark.gpu


# (rows of W, what is planted in their first column; H's first column is made positive)
PLANTS = {"nan row": (slice(130, 131), float("nan")), "inf row": (slice(130, 131), float("inf")),
          "nan in the ragged tile": (slice(699, 700), float("nan")),
          "-inf row": (slice(130, 131), float("-inf")), "-inf half tile": (slice(128, 256), float("-inf")),
          "-inf tile": (slice(256, 512), float("-inf")), "-inf ragged tile": (slice(512, 700), float("-inf"))}


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("plant", list(PLANTS))
@pytest.mark.parametrize("n_act", [40, 600])
def test_non_finite_logits(dtype, plant, n_act):
    import paper_2510_04206_amd as P
    T, V, d = n_act + 70, 700, 64
    rows, value = PLANTS[plant]
    log(f"non-finite logits {dtype} {plant} n_act={n_act}")
    g = torch.Generator().manual_seed(n_act)
    H = torch.randn((T, d), generator=g)
    H[:, 0] = H[:, 0].abs() + 0.1
    W = torch.randn((V, d), generator=g).mul_(0.2)
    W[rows, 0] = value
    H, W = H.to(dtype), W.to(dtype)
    y = torch.randint(0, 128, (T,), generator=g).to(torch.int32)     # never a planted row
    mask = torch.zeros(T, dtype=torch.uint8)
    mask[torch.randperm(T, generator=g)[:n_act]] = 1
    z = H.double() @ W.double().t()
    want_lse = z.logsumexp(1)
    want_logp = z.gather(1, y.long()[:, None])[:, 0] - want_lse
    finite = value == float("-inf")
    act = mask != 0
    assert bool(torch.isfinite(want_lse[act]).all()) == finite
    adv, old = torch.randn(T, generator=g), want_logp.float().nan_to_num(-5.0, -5.0, -5.0)
    c = lambda t: t.cuda()                                           # noqa: E731
    lp = P.TokenLogprob(T, d, V, dtype, max_act=n_act)
    pl = P.PolicyLoss(T, d, V, dtype, max_act=n_act)
    loss, *fwd, _ = pl.forward(c(H), c(W), c(y), c(mask), c(adv), c(old))
    for logp, lse in (lp(c(H), c(W), c(y), c(mask)), fwd):
        assert P.agrl_get_device_error() == 0
        logp, lse = logp.cpu().double(), lse.cpu().double()
        assert (logp[~act] == 0).all() and (lse[~act] == 0).all()
        if finite:
            assert (lse - want_lse)[act].abs().max() <= LSE_ATOL
            assert (logp - want_logp)[act].abs().max() <= LOGP_ATOL
        else:
            assert not torch.isfinite(lse[act]).any() and not torch.isfinite(logp[act]).any()
    assert bool(torch.isfinite(loss).all()) == finite


def test_nan_old_logp():
    import paper_2510_04206_amd as P
    T, V, d = 300, 500, 64
    log("NaN behaviour log-prob on one action token")
    g = torch.Generator(device="cuda").manual_seed(1)
    H = torch.randn((T, d), generator=g, device="cuda").bfloat16()
    W = torch.randn((V, d), generator=g, device="cuda").bfloat16()
    y = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    mask = (torch.arange(T, device="cuda") % 3 == 0).to(torch.uint8)
    adv, old = torch.randn(T, generator=g, device="cuda"), torch.full((T,), -6.0, device="cuda")
    pl = P.PolicyLoss(T, d, V, H.dtype)
    old[100] = float("nan")                      # not an action token: never read
    assert pl.forward(H, W, y, mask, adv, old)[0].isfinite().item()
    old[99] = float("nan")
    loss, logp, lse, _ = pl.forward(H, W, y, mask, adv, old)
    assert loss.isnan().item() and logp.isfinite().all() and lse.isfinite().all()
    dH, _ = pl.backward(H, W, y, mask, adv, old)
    assert dH[99].isnan().all() and dH[102].isfinite().all()
