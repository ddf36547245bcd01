"""The work that is timed: what a trainer has this library do, through its public entry points.

Four kinds of call, over the sizes that agentic RL training meets:

  adv      task advantage normalisation over a global batch of trajectories, once per step
           (``task_adv_norm``);
  seqw     the per-token weights of sequence-level aggregation, once per micro-batch
           (``sequence_mean_weights``);
  logprob  the forward-only log-prob pass that recomputes the behaviour policy's
           log-probs on the trainer (``TokenLogprob``, or the call without a workspace);
  loss     forward and backward of the fused LM-head and clipped policy loss over one
           packed micro-batch (``PolicyLoss``), with the options training uses: the KL
           penalty, sequence-level weights, gradient accumulation into dW, a temperature,
           decoupled clip bounds, a bound on the logit gradient's memory.

Inputs follow workloads/gen.py: multi-turn trajectories whose turns are an observation
(masked) and action tokens, H ~ N(0, 1), W ~ N(0, 0.02^2), target tokens sampled from the
softmax of the logits, behaviour log-probs near the policy's own so that some ratios reach
the clip bounds, one advantage per trajectory.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_04206_amd as P
from paper_2510_04206_amd import _binding as B

DEV = "cuda"
W_STD = 0.02


# ------------------------------------------------------------------ the cases
def listed():
    loss = dict(kind="loss", dtype="bf16", noise=0.1, eps_lo=0.2, eps_hi=0.2, kl=0.0, weighted=False,
                accumulate=False, temperature=0.0, chunk_bytes=0, bound=True)
    lp = dict(kind="logprob", dtype="bf16", temperature=0.0, noalloc=False)
    adv = dict(kind="adv", ddof=0, groups=True, drop=False)
    return [
        # a debugging or toy run's whole batch: 32 short trajectories of two tasks.  Nothing
        # but launches and latency.
        dict(adv, name="adv small", n_task=2, n_group=8, group_size=4, mean_len=120, scale=False),
        # the global batch of a step on twenty tasks (2560 trajectories of 8 turns), with
        # uniform-reward groups dropped as DAPO does.
        dict(adv, name="adv large", n_task=20, n_group=640, group_size=4, mean_len=3500,
             scale=True, drop=True),
        # sequence-level weights of one packed micro-batch out of a batch of 640 trajectories.
        dict(kind="seqw", name="sequence weights", T=65536, n_traj=640),
        # one turn scored on its own, by a loop that allocates nothing: a 7B model's head.
        dict(lp, name="logprob one turn", T=600, n_act=150, V=152064, d=3584, noalloc=True),
        # old log-probs of a packed batch, a 7B model's head.
        dict(lp, name="logprob packed", T=16384, n_act=5257, V=152064, d=3584),
        # the fp32 parity configuration: a tiny model on 16 trajectories per task.
        dict(loss, name="loss fp32 tiny", dtype="f32", T=3823, n_act=1519, V=4096, d=256, noise=0.05),
        # fp32 training of a small model, odd vocabulary, the KL penalty on.
        dict(loss, name="loss fp32 small", dtype="f32", T=4001, n_act=1333, V=16391, d=1024, kl=0.04),
        # one trajectory per micro-batch on a 7B model's head, accumulated over micro-batches,
        # the workspace laid out for any number of action tokens.
        dict(loss, name="loss one trajectory", T=2304, n_act=700, V=152064, d=3584, accumulate=True,
             bound=False),
        # a small model with a hidden size that is no multiple of 128, ragged everywhere,
        # temperature and decoupled clip bounds, the logit gradient held in several chunks.
        dict(loss, name="loss ragged", T=7013, n_act=2122, V=131001, d=1088, temperature=0.8,
             eps_hi=0.28, chunk_bytes=1 << 28),
        # a packed micro-batch of a 14B/32B model's head with the GRPO form's sequence weights.
        dict(loss, name="loss packed 8k", T=8192, n_act=2871, V=152064, d=5120, weighted=True, kl=0.01),
        # a packed micro-batch of a 7B model's head.
        dict(loss, name="loss 7B", T=32768, n_act=10515, V=152064, d=3584),
        # a packed micro-batch of a 32B model's head: the benchmark's sizes.
        dict(loss, name="loss 32B", T=65536, n_act=22793, V=152064, d=5120, noise=0.2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["adv", "seqw", "logprob", "logprob", "loss", "loss", "loss", "loss32"])
    if kind == "adv":
        groups = rng.random() < 0.8
        n_task = rng.randint(1, 20)
        return dict(kind="adv", n_task=n_task, n_group=_log_int(rng, max(8, n_task), 640),
                    group_size=rng.choice([2, 4, 5, 8]), mean_len=_log_int(rng, 60, 1750),
                    scale=rng.random() < 0.5, ddof=rng.randint(0, 1), groups=groups,
                    drop=groups and rng.random() < 0.5)
    if kind == "seqw":
        return dict(kind="seqw", T=_log_int(rng, 512, 131072), n_traj=_log_int(rng, 8, 2560))
    if kind == "loss32":
        d, V = 64 * _log_int(rng, 1, 16), _log_int(rng, 256, 16391)
        n_act = _log_int(rng, 64, min(8192, 25_000_000_000 // (V * d)))
    else:
        # any hidden size the kernels take; most models' are multiples of 128
        d = 64 * _log_int(rng, 2, 40) * rng.choice([1, 2, 2])
        d = min(d, 5120)
        V = _log_int(rng, 4096, 256000)
        if rng.random() < 0.5:
            V = -(-V // 64) * 64
        n_act = _log_int(rng, 64, min(22793, 17_000_000_000_000 // (V * d)))
    T = int(n_act * rng.uniform(1.2, 5.0)) + rng.randint(0, 63)
    temperature = rng.choice([0.0, 0.0, 0.8])
    if kind == "logprob":
        fits = -(-n_act // 256) * 256 * (2 * d + 8 * -(-V // 256) + 64) < B.AGRL_NOALLOC_SCRATCH_BYTES - (1 << 20)
        return dict(kind="logprob", dtype="bf16", T=T, n_act=n_act, V=V, d=d, temperature=temperature,
                    noalloc=fits and rng.random() < 0.5)
    return dict(kind="loss", dtype="f32" if kind == "loss32" else "bf16", T=T, n_act=n_act, V=V, d=d,
                noise=rng.choice([0.05, 0.1, 0.2]), eps_lo=0.2, eps_hi=rng.choice([0.2, 0.28]),
                kl=rng.choice([0.0, 0.0, 0.04]), weighted=rng.random() < 0.3,
                accumulate=rng.random() < 0.3, temperature=temperature,
                chunk_bytes=rng.choice([0, 0, 0, 1 << 28]), bound=rng.random() < 0.7)


# ------------------------------------------------------------------ inputs
def _turns(rng, T, n_act):
    """uint8[T]: n_act action tokens in runs of about 100, observations between them."""
    k = max(1, min(n_act, T - n_act, n_act // 100))

    def parts(n):
        cuts = np.sort(rng.choice(np.arange(1, n), k - 1, replace=False)) if k > 1 else np.array([], int)
        return np.diff(np.concatenate([[0], cuts, [n]]))

    m = np.zeros(T, np.uint8)
    at = 0
    for o, a in zip(parts(T - n_act), parts(n_act)):
        m[at + o:at + o + a] = 1
        at += o + a
    return m


def _trajectories(rng, n, lengths):
    """int32 ids of n trajectories in a random order, one after the other, and their mask."""
    order = rng.permutation(n)
    ids = np.repeat(order.astype(np.int32), lengths[order])
    T = ids.shape[0]
    # turns of 32..511 tokens, the last third of each being the action
    size = rng.integers(32, 512, T // 32 + 2)
    ends = np.cumsum(size)
    turn = np.searchsorted(ends, np.arange(T), side="right")
    return ids, (ends[turn] - np.arange(T) <= size[turn] // 3).astype(np.uint8)


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _prepare_adv(case, seed):
    rng = np.random.default_rng([seed, 1])
    n_task, n_group, size = case["n_task"], case["n_group"], case["group_size"]
    n = n_group * size
    group = np.repeat(np.arange(n_group, dtype=np.int32), size)
    task = (group.astype(np.int64) * n_task // n_group).astype(np.int32)
    if case["scale"]:           # tasks of different reward scales, some with a few outcomes only
        reward = rng.normal(0, 1, n) + rng.normal(0, 2, n_task)[task]
        reward = np.where(task % 2 == 0, rng.random(n) < rng.random(n_task)[task], reward)
    else:                       # success or failure
        reward = rng.random(n) < 0.5
    # lengths from a half to one and a half times the mean, in pairs that keep the total
    lengths = np.full(n, case["mean_len"])
    off = rng.integers(0, case["mean_len"] // 2 + 1, n // 2)
    lengths[:n // 2] += off
    lengths[n - n // 2:] -= off
    ids, mask = _trajectories(rng, n, rng.permutation(lengths))
    return dict(kind="adv", traj_id=_t(ids), mask=_t(mask), task=_t(task),
                group=_t(group) if case["groups"] else None, reward=_t(reward.astype(np.float32)),
                n_task=n_task, n_group=n_group if case["groups"] else 0,
                opt=dict(std_ddof=case["ddof"], drop_uniform_groups=int(case["drop"])))


def _prepare_seqw(case, seed):
    rng = np.random.default_rng([seed, 2])
    T, n = case["T"], case["n_traj"]
    lengths = rng.integers(T // n // 2 + 1, 4 * (T // n) + 1000, n)
    ids, mask = _trajectories(rng, n, lengths)
    return dict(kind="seqw", traj_id=_t(ids[:T]), mask=_t(mask[:T]), n_traj=n)


def _head(case, seed):
    """H, W, mask, sampled targets and behaviour log-probs (zero on observations)."""
    T, V, d = case["T"], case["V"], case["d"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    rng = np.random.default_rng([seed, 3])
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 2 + 1)
    H = torch.randn((T, d), generator=gen, device=DEV).to(dt)
    W = torch.randn((V, d), generator=gen, device=DEV).mul_(W_STD).to(dt)
    mask = _t(_turns(rng, T, case["n_act"]))
    act = torch.nonzero(mask).flatten()
    y = torch.randint(0, V, (T,), generator=gen, device=DEV, dtype=torch.int32)
    logp = torch.zeros(T, device=DEV)
    for rows in act.split(max(64, min(2048, (1 << 28) // V))):
        z = (H.index_select(0, rows) @ W.t()).float()
        # Gumbel: the largest of z - log(-log u) is a sample of softmax(z)
        u = torch.empty_like(z).exponential_(generator=gen).log_()
        s = (z - u).argmax(1)
        y[rows] = s.int()
        logp[rows] = z.gather(1, s[:, None])[:, 0] - z.logsumexp(1)
        del z, u
    return H, W, mask, act, y, logp, gen


def _prepare_logprob(case, seed):
    H, W, mask, act, y, logp, gen = _head(case, seed)
    T, V, d = case["T"], case["V"], case["d"]
    opt = dict(temperature=case["temperature"])
    s = dict(kind="logprob", case=dict(case), H=H, W=W, y=y, mask=mask, opt=B.agrl_options(**opt))
    if case["noalloc"]:
        s["out"] = (torch.empty(T, device=DEV), torch.empty(T, device=DEV))
    else:
        s["plan"] = P.TokenLogprob(T, d, V, H.dtype, max_act=case["n_act"], opt=opt)
    return s


def _prepare_loss(case, seed):
    H, W, mask, act, y, logp, gen = _head(case, seed)
    T, V, d, n_act = case["T"], case["V"], case["d"], case["n_act"]
    old = torch.zeros(T, device=DEV)
    old[act] = logp[act] + case["noise"] * torch.randn(n_act, generator=gen, device=DEV)
    # one normalised advantage per trajectory: about 700 tokens each
    traj = torch.arange(T, device=DEV) // 700
    adv = torch.randn(int(traj[-1]) + 1, generator=gen, device=DEV)[traj] * mask
    opt = dict(temperature=case["temperature"], dw_accumulate=int(case["accumulate"]),
               g_chunk_bytes=case["chunk_bytes"], kl_beta=case["kl"])
    s = dict(kind="loss", case=dict(case), H=H, W=W, y=y, mask=mask, old=old, adv=adv)
    if case["kl"]:
        s["ref"] = torch.where(mask.bool(), logp + 0.1 * torch.randn(T, generator=gen, device=DEV), old)
        opt["ref_logp"] = s["ref"].data_ptr()
    if case["weighted"]:
        s["seq"] = P.sequence_mean_weights(traj.int(), mask, int(traj[-1]) + 1)
        opt["token_weight"] = s["seq"][1].data_ptr()
    s["plan"] = P.PolicyLoss(T, d, V, H.dtype, max_act=n_act if case["bound"] else 0,
                             eps_low=case["eps_lo"], eps_high=case["eps_hi"], opt=opt)
    if case["accumulate"]:      # the gradient of the micro-batches before this one
        s["plan"].dW.normal_(generator=gen).mul_(1 / math.sqrt(n_act * V))
    return s


_PREPARE = dict(adv=_prepare_adv, seqw=_prepare_seqw, logprob=_prepare_logprob, loss=_prepare_loss)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


# ------------------------------------------------------------------ one pass
_ADV_OUT = ("act_count", "task_count", "task_mean", "task_std", "adv_traj", "adv_tok")


def run(s):
    if s["kind"] == "adv":
        out = P.task_adv_norm(s["traj_id"], s["mask"], s["task"], s["group"], s["reward"], s["n_task"],
                              s["n_group"], opt=s["opt"])
        return {k: out[k] for k in _ADV_OUT}
    if s["kind"] == "seqw":
        return P.sequence_mean_weights(s["traj_id"], s["mask"], s["n_traj"])
    if s["kind"] == "logprob":
        if "plan" in s:
            return s["plan"](s["H"], s["W"], s["y"], s["mask"])
        c = s["case"]
        B.agrl_token_logprob_noalloc(c["T"], c["n_act"], c["d"], c["V"], B.AGRL_BF16, s["H"], s["W"], s["y"],
                                     s["mask"], s["opt"], s["out"][0], s["out"][1])
        return s["out"]
    args = s["H"], s["W"], s["y"], s["mask"], s["adv"], s["old"]
    loss, logp, lse, n_clip = s["plan"].forward(*args)
    dH, dW = s["plan"].backward(*args)
    out = dict(loss=loss, logp=logp, lse=lse, dH=dH, dW=dW)
    # The two clip counts move by one where a ratio lies within its rounding of a clip bound,
    # which a large batch has now and then; as two whole numbers they are compared where not.
    if s["case"]["T"] <= 8192:
        out["n_clip"] = n_clip
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    k = case["kind"]
    if k == "adv":
        n, T = case["n_group"] * case["group_size"], case["n_group"] * case["group_size"] * case["mean_len"]
        return dict(bytes=T * (4 + 1 + 4) + n * (4 + 4 * case["groups"] + 4 + 4 + 4) + case["n_task"] * 16, flops=0)
    if k == "seqw":
        return dict(bytes=case["T"] * (4 + 1 + 4) + case["n_traj"] * 4, flops=0)
    T, N, V, d = case["T"], case["n_act"], case["V"], case["d"]
    e = 2 if case["dtype"] == "bf16" else 4
    once = N * d * e + V * d * e + T * (1 + 4 + 4) + N * 4      # H's action rows, W, mask, logp, lse, ids
    if k == "logprob":
        return dict(bytes=once, flops=2 * N * V * d)
    extra = N * 4 * (2 + bool(case["kl"]) + case["weighted"])
    grads = T * d * 4 + V * d * 4 * (2 if case["accumulate"] else 1)
    # logits, dH and dW; that the logits are formed twice is the library's choice
    return dict(bytes=once + extra + grads, flops=6 * N * V * d)


def tolerance(case):
    if case["kind"] in ("adv", "seqw"):     # the header fixes the order of every sum
        return "exact"
    if case["kind"] == "logprob":           # fp32 sums of exact products
        return {"rel": 5e-7}
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    return {"rel": 7e-3}                    # the logit gradient is rounded to bf16


# ------------------------------------------------------------------ the same in 64 bits
def _exact_adv(s):
    ids, mask = s["traj_id"].cpu().numpy(), s["mask"].cpu().numpy()
    task, reward = s["task"].cpu().numpy(), s["reward"].cpu().numpy().astype(np.float64)
    ddof, eps = s["opt"]["std_ddof"], float(np.float32(1e-6))
    n, n_task = task.shape[0], s["n_task"]
    count = np.bincount(ids[mask != 0], minlength=n)
    a, kept = reward.copy(), np.ones(n, bool)
    if s["group"] is not None:
        group = s["group"].cpu().numpy()
        for g in range(s["n_group"]):
            m = np.nonzero(group == g)[0]
            r = reward[m]
            if s["opt"]["drop_uniform_groups"] and (r == r[0]).all():
                kept[m] = False
                a[m] = 0
            elif len(m) > ddof:
                a[m] = (r - r.mean()) / (math.sqrt(((r - r.mean()) ** 2).sum() / (len(m) - ddof)) + eps)
            else:
                a[m] = 0
    N, mean, std, out = (np.zeros(n_task, t) for t in (np.int64, np.float64, np.float64, np.float64))
    out = np.zeros(n)
    for i in range(n_task):
        m = np.nonzero((task == i) & kept)[0]
        N[i] = count[m].sum()
        if N[i] == 0:
            continue
        mean[i] = (count[m] * a[m]).sum() / N[i]
        if N[i] > ddof:
            std[i] = math.sqrt((count[m] * (a[m] - mean[i]) ** 2).sum() / (N[i] - ddof))
        out[m] = (a[m] - mean[i]) / (std[i] + eps)
    return dict(act_count=count.astype(np.int32), task_count=N, task_mean=mean, task_std=std, adv_traj=out,
                adv_tok=out[ids] * mask)


def _exact_seqw(s):
    ids, mask = s["traj_id"].cpu().numpy(), s["mask"].cpu().numpy()
    count = np.bincount(ids[mask != 0], minlength=s["n_traj"])
    w = np.where(mask != 0, 1.0 / ((count > 0).sum() * np.maximum(count[ids], 1)), 0.0)
    return count.astype(np.int32), w


def _exact_head(s):
    c = s["case"]
    T, V = c["T"], c["V"]
    it = 1.0 if c["temperature"] == 0 else 1.0 / float(np.float32(c["temperature"]))
    act = torch.nonzero(s["mask"]).flatten()
    y = s["y"].long()[act]
    H = s["H"][act].double()
    blocks = [(v, min(V, v + 8192)) for v in range(0, V, 8192)]
    lse = torch.full((len(act),), -math.inf, dtype=torch.float64, device=DEV)
    zy = torch.zeros_like(lse)
    for v0, v1 in blocks:
        z = (H @ s["W"][v0:v1].double().t()).mul_(it)
        lse = torch.logaddexp(lse, z.logsumexp(1))
        here = (y >= v0) & (y < v1)
        zy[here] = z[here, y[here] - v0]
        del z
    spread = lambda a: torch.zeros(T, dtype=torch.float64, device=DEV).index_put_((act,), a)  # noqa: E731
    return act, y, H, blocks, it, lse, zy - lse, spread


def _exact_loss(s):
    c, o = s["case"], s["plan"].opt
    act, y, H, blocks, it, lse, logp, spread = _exact_head(s)
    N = len(act)
    A, old = s["adv"][act].double(), s["old"][act].double()
    lo, hi = (float(np.float32(c[k])) for k in ("eps_lo", "eps_hi"))
    rho = (logp - old).exp()
    f = torch.minimum(rho * A, rho.clamp(1 - lo, 1 + hi) * A)
    cut_hi, cut_lo = (A > 0) & (rho > 1 + hi), (A < 0) & (rho < 1 - lo)
    w = s["seq"][1][act].double() if c["weighted"] else torch.full_like(A, 1.0 / N)
    g = torch.where(cut_hi | cut_lo, torch.zeros_like(A), -A * rho)
    if c["kl"]:
        u, beta = s["ref"][act].double() - logp, float(o.kl_beta)
        f = f - beta * (torch.expm1(u) - u)
        g = g - beta * torch.expm1(u)
    loss, g = -(w * f).sum().reshape(1), w * g * it
    dH = torch.zeros_like(H)
    dW = s["plan"].dW.double() if c["accumulate"] else torch.zeros_like(s["plan"].dW, dtype=torch.float64)
    for v0, v1 in blocks:
        Wb = s["W"][v0:v1].double()
        G = (H @ Wb.t()).mul_(it).sub_(lse[:, None]).exp_().mul_(-g[:, None])
        here = torch.nonzero((y >= v0) & (y < v1)).flatten()
        G[here, y[here] - v0] += g[here]
        dH += G @ Wb
        dW[v0:v1] += G.t() @ H
        del G, Wb
    full = torch.zeros(c["T"], c["d"], dtype=torch.float64, device=DEV)
    full[act] = dH
    out = dict(loss=loss, logp=spread(logp), lse=spread(lse), dH=full, dW=dW)
    if c["T"] <= 8192:
        out["n_clip"] = torch.stack([cut_hi.sum(), cut_lo.sum()])
    return out


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "adv":
        return _exact_adv(s)
    if case["kind"] == "seqw":
        return _exact_seqw(s)
    if case["kind"] == "logprob":
        _, _, _, _, _, lse, logp, spread = _exact_head(s)
        return spread(logp), spread(lse)
    return _exact_loss(s)
