"""The policy loss at the sizes where its kernels change tile, split or tail: every
output of forward and backward against the oracle.

dH and dW, relative Frobenius.  fp32: sums of up to 8192 products (random walk of
2^-24 roundings: 5e-6) of probabilities whose exponent carries up to 2^-24 * 16
absolute (1e-6): 1e-5.  bf16: G rounded to 2^-9 relative: 4e-3 (twice the bound, for
the few elements in which a sum is dominated by one product).
"""
import numpy as np
import pytest
import torch

import oracle

from helpers import compare_loss, log, run_gpu

pytestmark = pytest.mark.gpu


def _case(dtype, V, d, n_act, *, T=None, seed=1, opt=None, max_act=None, dW0=None):
    import paper_2510_04206_amd as P
    rng = np.random.default_rng([seed, V, d, n_act])
    T = T or n_act + n_act // 2 + 3
    mask = np.zeros(T, np.uint8)
    mask[np.sort(rng.permutation(T)[:n_act])] = 1
    g = torch.Generator().manual_seed(seed)
    H = torch.randn((T, d), generator=g).to(dtype)
    W = torch.randn((V, d), generator=g).mul_(0.1).to(dtype)
    y = rng.integers(0, V, T).astype(np.int32)
    y[:: 7] = V - 1                                  # the last vocabulary row's tile
    act = torch.from_numpy(np.nonzero(mask)[0])
    logp = torch.zeros(T)
    logp[act] = torch.log_softmax(H[act].float() @ W.float().t(), 1).gather(
        1, torch.from_numpy(y).long()[act][:, None])[:, 0]
    old = (logp.numpy() + 0.2 * rng.standard_normal(T)).astype(np.float32)
    adv = rng.standard_normal(T).astype(np.float32)
    log(f"shape {dtype} V={V} d={d} n_act={n_act} T={T} max_act={max_act} {opt}")
    pl = P.PolicyLoss(T, d, V, dtype, max_act=n_act if max_act is None else max_act, opt=opt)
    if dW0 is not None:
        pl.dW.fill_(dW0)
    t = lambda a: torch.from_numpy(a).cuda()                    # noqa: E731
    got = run_gpu(pl, dict(H=H.cuda(), W=W.cuda(), token_id=t(y), mask=t(mask), old_logp=t(old)), t(adv))
    assert P.agrl_get_device_error() == 0
    ref = oracle.policy_loss(H, W, y, mask, adv, old)
    if dW0 is not None:
        ref["dW"] = ref["dW"] + dW0
    errs = compare_loss(got, ref, mask, adv, old, 0.2, 0.2,
                        grad_rel=1e-5 if dtype == torch.float32 else 4e-3)
    log(f"  dH, dW: {errs}")


# fp32: logit tiles of 256 x 32 and 256 x 64 (the second from 512 tiles on), gradient
# tiles of 64 x 64, K stages of 32; dW split (few rows, many tokens), dH split (many
# rows, few tokens), neither; a hidden size above and below one tile
@pytest.mark.parametrize("V,d,n_act", [
    (1, 64, 1), (255, 64, 31), (257, 64, 33), (256, 128, 64), (300, 192, 65), (33, 64, 3000),
    (256, 64, 8192), (8191, 64, 129), (8193, 64, 1056), (4099, 320, 257), (2049, 1024, 100)])
def test_fp32_shapes(V, d, n_act):
    _case(torch.float32, V, d, n_act)


def test_fp32_chunks_accumulate_loose_bound():
    # chunks of 512 columns, the last of 3; dW added to; room for every token
    _case(torch.float32, 1027, 128, 300, T=1500, opt=dict(g_chunk_bytes=2 * 1536 * 4 * 512, dw_accumulate=1),
          max_act=0, dW0=0.25)


def _pad(n):
    return -(-n // 256) * 256


def _reads_w(T, max_act, V, d):
    """Whether a bf16 backward reads W as it lies for dH (EpiGrad) or builds W^T (EpiStore): the
    bound on the action tokens is at most 8192, and W^T's place holds one part of dH beside
    W's padded tail."""
    A = _pad(max_act or T)
    return A <= 8192 and (_pad(d) * _pad(V) * 2 - _pad(128 * d * 2)) // (A * d * 4) > 0


# bf16 with few action tokens (dH reads W as it lies): one, several and many parts of
# dH's K; W's last rows a whole stage pair or a remainder of 1, 63, 64, 127; a hidden
# size that leaves a partial 256-tile; one row of tokens more and less than a tile
@pytest.mark.parametrize("V,d,n_act", [
    (1, 64, 1), (127, 64, 255), (1025, 128, 256), (2048, 192, 257), (4100, 192, 261), (8191, 320, 100),
    (20031, 128, 300), (50240, 256, 70), (6079, 512, 2000)])
def test_bf16_few_tokens(V, d, n_act):
    assert _reads_w(0, n_act, V, d)
    _case(torch.bfloat16, V, d, n_act)


# bf16 with W^T: a vocabulary too small for a part of dH; more than 8192 action tokens; and a
# bound above that with few tokens.  The last: two chunks whose dW tiles fill two rounds of
# the queues, the last chunk ragged, d partial, dH added to over the chunks and dW added to.
@pytest.mark.parametrize("V,d,n_act,T,opt", [
    (129, 128, 256, None, {}), (33, 512, 2000, None, {}), (700, 192, 8300, None, {}), (1, 64, 1, 8200, {}),
    (257, 1088, 257, 8300, {}), (1027, 320, 600, 9000, dict(dw_accumulate=1)),
    (1665, 192, 300, 9000, dict(g_chunk_bytes=9216 * 2 * 512, dw_accumulate=1)),
    (131001, 320, 600, 9000, dict(g_chunk_bytes=9216 * 2 * 65536, dw_accumulate=1))])
def test_bf16_with_transposed_w(V, d, n_act, T, opt):
    import paper_2510_04206_amd as P
    max_act = 0 if T else n_act
    assert not _reads_w(T, max_act, V, d)
    if V > 100000:
        vc = P.PolicyLoss(T, d, V, torch.bfloat16, opt=opt).vocab_chunk
        tiles = [-(-c // 256) * -(-d // 256) for c in (vc, V - vc)]      # of dW, in each launch
        assert vc < V < 2 * vc and min(tiles) >= 2 * 256 and (V - vc) % 256 and d % 256
    _case(torch.bfloat16, V, d, n_act, T=T, opt=opt, max_act=max_act, dW0=0.25 if opt else None)


# the same launch without action tokens (dW written as zeros, or left as it is), with an id
# outside the vocabulary, and with more action tokens than the bound
def test_bf16_with_transposed_w_faults():
    import paper_2510_04206_amd as P
    T, V, d, n_act = 8300, 400, 192, 300
    log("W^T backward: no action tokens, bad id, over the bound")
    g = torch.Generator(device="cuda").manual_seed(5)
    H = torch.randn((T, d), generator=g, device="cuda").bfloat16()
    W = torch.randn((V, d), generator=g, device="cuda").mul_(0.1).bfloat16()
    y = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    adv, old = torch.randn(T, generator=g, device="cuda"), torch.full((T,), -6.0, device="cuda")
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    for acc in (0, 1):
        pl = P.PolicyLoss(T, d, V, H.dtype, opt=dict(dw_accumulate=acc))
        pl.dW.fill_(2.0)
        pl.dH.fill_(float("nan"))
        loss, *_ = pl.forward(H, W, y, mask, adv, old)
        dH, dW = pl.backward(H, W, y, mask, adv, old)
        assert loss.item() == 0 and (dH == 0).all() and not torch.signbit(dH).any()
        assert (dW == 2.0 * acc).all()
    mask[torch.randperm(T, generator=g, device="cuda")[:n_act]] = 1
    act = torch.nonzero(mask)[:, 0]
    bad = int(act[n_act // 2])
    y[bad] = V
    pl = P.PolicyLoss(T, d, V, H.dtype)
    loss, logp, lse, _ = pl.forward(H, W, y, mask, adv, old)
    dH, dW = pl.backward(H, W, y, mask, adv, old)
    assert P.agrl_get_device_error() == 1
    others = act[act != bad]
    assert loss.isnan().item() and logp[bad].isnan() and lse[bad].isnan()
    assert logp[others].isfinite().all() and dH[others].isfinite().all()
    assert dH[bad].isnan().all() and dW.isnan().all() and (dH[mask == 0] == 0).all()
    # over the bound, at the sizes of the one-launch and of the three-launch compaction
    for T2 in (T, 70000):
        H2, m2 = torch.zeros((T2, d), dtype=H.dtype, device="cuda"), torch.ones(T2, dtype=torch.uint8, device="cuda")
        z = torch.zeros(T2, device="cuda")
        pl = P.PolicyLoss(T2, d, V, H.dtype, max_act=T2 - 1)
        loss, *_ = pl.forward(H2, W, torch.zeros(T2, dtype=torch.int32, device="cuda"), m2, z, z)
        assert loss.isnan().item() and P.agrl_get_device_error() == 16
    assert P.agrl_get_device_error() == 0


def test_bf16_few_tokens_chunks_accumulate_loose_bound():
    # chunks of 4096 columns, the last of 1; dW added to; room for every token
    _case(torch.bfloat16, 8193, 320, 130, T=700, opt=dict(g_chunk_bytes=768 * 2 * 4096, dw_accumulate=1),
          max_act=0, dW0=0.25)


# compaction: tokens before, at and after a block of 256, a mask that starts off a 16-byte
# boundary, as many tokens as one launch handles (2^16) and more
@pytest.mark.parametrize("T,offset", [(1, 0), (255, 3), (256, 0), (257, 1), (4097, 16), (5000, 7),
                                      (1 << 16, 0), (1 << 16, 9), ((1 << 16) + 1, 0),
                                      ((1 << 18) + 333, 0), ((1 << 18) + 77, 5)])
def test_compaction(T, offset):
    import paper_2510_04206_amd as P
    rng = np.random.default_rng(T)
    d, V = 64, 300
    m = np.zeros(T + offset, np.uint8)
    m[offset:] = rng.random(T) < (0.4 if T < 10000 else 0.004)
    m[-1] = 1
    m[offset:] *= rng.integers(1, 256, T).astype(np.uint8)      # any nonzero byte is an action
    log(f"compaction T={T} offset={offset}")
    mask = torch.from_numpy(m).cuda()[offset:]
    g = torch.Generator(device="cuda").manual_seed(T)
    H = torch.randn((T, d), generator=g, device="cuda").bfloat16()
    W = torch.randn((V, d), generator=g, device="cuda").bfloat16()
    y = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    act = mask != 0
    lp = P.TokenLogprob(T, d, V, H.dtype, max_act=int(act.sum()))
    logp, lse = lp(H, W, y, mask)
    assert P.agrl_get_device_error() == 0
    z = H[act].double() @ W.double().t()
    want = torch.zeros(2, T, dtype=torch.float64, device="cuda")
    want[0, act] = torch.log_softmax(z, 1).gather(1, y[act].long()[:, None])[:, 0]
    want[1, act] = z.logsumexp(1)
    assert (logp.double() - want[0]).abs().max() < 5e-5 and (lse.double() - want[1]).abs().max() < 2e-5
    adv = torch.randn(T, generator=g, device="cuda")
    pl = P.PolicyLoss(T, d, V, H.dtype, max_act=int(act.sum()))
    pl.dH.fill_(float("nan"))
    pl.forward(H, W, y, mask, adv, want[0].float())
    dH, _ = pl.backward(H, W, y, mask, adv, want[0].float())
    assert (dH[~act] == 0).all() and not torch.signbit(dH[~act]).any()
    p = torch.softmax(z, 1)
    p.scatter_add_(1, y[act].long()[:, None], torch.full((int(act.sum()), 1), -1.0, device="cuda").double())
    ref = (adv[act].double() / act.sum())[:, None] * p @ W.double()
    assert ((dH[act].double() - ref).norm() / ref.norm()) < 4e-3


# bf16, a hidden size that is an odd number of 64-deep stages: one stage, three, five, seventeen
@pytest.mark.parametrize("V,d,n_act", [(700, 64, 300), (513, 192, 257), (900, 320, 300), (1000, 1088, 40)])
def test_bf16_odd_stages(V, d, n_act):
    _case(torch.bfloat16, V, d, n_act)


# fp32 with rows so long that a tile's last rows lie more than 2^32 bytes after its first,
# against fp64.  A logit is a sum of 2^22 terms of rms 2^-11 whose partial sums are of order 1,
# each rounded by up to 2^-24 of itself: a random walk of 2^11 * 2^-24 = 1.2e-4.
def test_fp32_rows_beyond_32_bit_offsets():
    import paper_2510_04206_amd as P
    T, V, d = 2, 256, 4210816                        # 255 * 4 d = 2^32 + 65024
    log(f"long fp32 rows V={V} d={d}")
    g = torch.Generator(device="cuda").manual_seed(3)
    H = torch.randn((T, d), generator=g, device="cuda")
    W = torch.randn((V, d), generator=g, device="cuda").mul_(d ** -0.5)
    y = torch.tensor([5, V - 1], dtype=torch.int32, device="cuda")
    mask = torch.tensor([0, 1], dtype=torch.uint8, device="cuda")
    lp = P.TokenLogprob(T, d, V, H.dtype, max_act=1)
    logp, lse = lp(H, W, y, mask)
    assert P.agrl_get_device_error() == 0
    z = torch.stack([torch.dot(H[1].double(), w.double()) for w in W])
    assert abs(lse[1].item() - z.logsumexp(0).item()) < 1e-3
    assert abs(logp[1].item() - torch.log_softmax(z, 0)[V - 1].item()) < 1e-3


# fp32 with more than 2^24 logit tiles of 64 tokens, 2^32 threads at 256 each: more than one
# launch holds.  Tokens spread over all tiles, the first and the last, against fp64.
def test_fp32_more_tiles_than_a_launch():
    import paper_2510_04206_amd as P
    T, V, d = 1 << 20, (1 << 18) + 5, 64
    log(f"fp32 logit tiles T={T} V={V} d={d}")
    g = torch.Generator(device="cuda").manual_seed(4)
    H = torch.randn((T, d), generator=g, device="cuda")
    W = torch.randn((V, d), generator=g, device="cuda").mul_(0.1)
    y = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    y[-1] = V - 1
    mask = torch.ones(T, dtype=torch.uint8, device="cuda")
    lp = P.TokenLogprob(T, d, V, H.dtype)
    logp, lse = lp(H, W, y, mask)
    assert P.agrl_get_device_error() == 0
    at = torch.cat([torch.arange(0, T, 4099, device="cuda"), torch.tensor([T - 64, T - 1], device="cuda")])
    for part in at.split(64):
        z = H[part].double() @ W.double().t()
        want_lse = z.logsumexp(1)
        want = z.gather(1, y[part].long()[:, None])[:, 0] - want_lse
        assert (lse[part].double() - want_lse).abs().max() < 2e-5
        assert (logp[part].double() - want).abs().max() < 5e-5
