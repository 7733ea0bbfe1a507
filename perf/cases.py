"""Timed cases: the calls a PS-PPO training program makes, over the sizes it makes them at.

Paths
  update   one whole update pass (``pipeline.Step``): draw the cutoffs, pack the prefixes, LM-head
           PPO loss forward + backward
  loss     the loss call alone on tokens that are already packed (micro-batches, gradient accumulation)
  proxy    the output-head score proxy over completion tokens (forward only)
  pack     cutoff sampling + prefix packing with the gather of the hidden rows
  weights  the per-step weights of the cutoff design
  design   the budgeted monotone solve for the survival tables

Sizes are those of the repository's own workloads (``synth.CONFIGS``) with batches from a few
completions to the whole one, and generic ragged ones.  Target ids follow a 1/rank law, as the
tokens of real text do, and the hidden rows carry a component along their target's head row, so
that log-probs spread from near 0 to -log V.
"""
import math
import statistics

import numpy as np
import torch

from paper_2606_29758_amd import pipeline, pspo, synth

DEV = "cuda"
EPS = 0.1
PHILOX = 11      # seed of the cutoff draws
W_STD = 0.02
# successes of the K = 8 completions of prompt 0, 1, 2, ...: every count equally often (a prompt's
# success rate is uniform), so 2 prompts of 9 have equal rewards and zero advantages
SUCCESSES = (3, 6, 1, 8, 4, 7, 2, 5, 0)


def listed():
    return [
        # the smallest whole pass (the `tiny` workload): launches and latency
        dict(name="update_tiny", path="update", P=2, K=4, d=128, V=2048, median=80, sigma=0.4, lo=32, hi=128,
             sigma_lp=0.05, logp=True),
        # two prompts on the 1.5B-shaped head: a data-parallel rank's share of a small batch, ragged V
        dict(name="update_1p5b_short", path="update", P=2, K=8, d=1536, V=151936, median=512, sigma=0.5, lo=64,
             hi=4096, sigma_lp=0.05, logp=True),
        # the benchmark's batch (`qwen7b`): the largest
        dict(name="update_7b", path="update", P=8, K=8, d=3584, V=152064, median=2048, sigma=0.5, lo=128, hi=8192,
             sigma_lp=0.1, logp=False),
        # a few short completions on the 7B-shaped head: the smallest call on a real vocabulary
        dict(name="loss_7b_short", path="loss", tokens=200, seqs=8, d=3584, V=152064, sigma_lp=0.1, logp=True,
             accumulate=False, keep=False),
        # one micro-batch of a gradient-accumulation loop on the 7B-shaped head
        dict(name="loss_7b_micro", path="loss", tokens=2048, seqs=16, d=3584, V=152064, sigma_lp=0.1, logp=False,
             accumulate=True, keep=False),
        # a middle-sized batch with the opt-in kept logits
        dict(name="loss_7b_keep", path="loss", tokens=16001, seqs=32, d=3584, V=152064, sigma_lp=0.1, logp=False,
             accumulate=False, keep=True),
        # odd sizes everywhere: no tile, K step or chunk comes out even
        dict(name="loss_ragged", path="loss", tokens=4999, seqs=24, d=1000, V=50021, sigma_lp=0.1, logp=True,
             accumulate=False, keep=False),
        # computing xi on the 7B-shaped head: the proxy over the completion tokens of one prompt
        dict(name="proxy_7b", path="proxy", tokens=20480, d=3584, V=152064, p_sq=False),
        # the proxy of one short completion on the 1.5B-shaped head, with every output
        dict(name="proxy_1p5b_short", path="proxy", tokens=1501, d=1536, V=151936, p_sq=True),
        # sampling and packing of the long-reasoning batch (`qwen7b_long`): a gather, bound by memory
        dict(name="pack_7b_long", path="pack", P=4, K=8, d=3584, median=8192, sigma=0.5, lo=1024, hi=16384),
        # the design weights of the benchmark's batch, top-16 lists
        dict(name="weights_7b", path="weights", P=8, K=8, topk=16, median=2048, sigma=0.5, lo=128, hi=8192),
        # the survival tables of the benchmark's batch
        dict(name="design_7b", path="design", P=8, K=8, median=2048, sigma=0.5, lo=128, hi=8192, variant=0,
             kept=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choices(["update", "loss", "proxy", "pack", "weights", "design"], [3, 5, 3, 2, 2, 2])[0]
    d = max(128, min(4096, _log_int(rng, 128, 4096)))
    d = d // 8 * 8 if rng.random() < 0.5 else max(128, d // 128 * 128)
    V = _log_int(rng, 2000, 152064)
    if rng.random() < 0.4:
        V = rng.choice([2048, 32000, 128256, 151936, 152064])
    K = rng.choice([2, 4, 8, 16])
    P = rng.choice([1, 2, 3, 5, 8, 16])
    most = 2e13 / (float(V) * d)     # a third of the largest listed case's products
    if path == "loss":
        tokens = min(_log_int(rng, 48, 60000), int(most))
        return dict(path="loss", tokens=tokens, seqs=max(1, min(tokens // 8, P * K)), d=d, V=V,
                    sigma_lp=rng.choice([0.05, 0.1]), logp=rng.random() < 0.5, accumulate=rng.random() < 0.4,
                    keep=rng.random() < 0.2)
    if path == "proxy":
        return dict(path="proxy", tokens=min(_log_int(rng, 48, 100000), int(2 * most)), d=d, V=V,
                    p_sq=rng.random() < 0.3)
    median = _log_int(rng, 64, 8192)
    if path == "update":
        median = max(24, min(median, int(most / (P * K))))
        return dict(path="update", P=P, K=K, d=d, V=V, median=median, sigma=0.5, lo=max(8, median // 8),
                    hi=median * 4, sigma_lp=rng.choice([0.05, 0.1]), logp=rng.random() < 0.5)
    if path == "pack":
        median = min(median, int(3e5 / (P * K)))
        return dict(path="pack", P=P, K=K, d=d, median=median, sigma=0.5, lo=max(8, median // 8), hi=median * 4)
    median = min(median, int(6e5 / (P * K)))
    if path == "weights":
        return dict(path="weights", P=P, K=K, topk=rng.choice([5, 8, 16]), median=median, sigma=0.5,
                    lo=max(8, median // 8), hi=min(median * 4, 16384))
    return dict(path="design", P=P, K=K, median=median, sigma=0.5, lo=max(8, median // 8),
                hi=min(median * 4, 16384), variant=rng.choice([0, 0, 0, 1, 2, 3]), kept=rng.uniform(0.2, 0.8))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _lengths(case, rng):
    """Completion lengths: the quantiles of the clipped log-normal law in random order."""
    R = case["P"] * case["K"]
    q = [statistics.NormalDist().inv_cdf((i + 0.5) / R) for i in range(R)]
    raw = np.rint(case["median"] * np.exp(case["sigma"] * np.array(q)))
    return rng.permutation(np.clip(raw, case["lo"], case["hi"])).astype(np.int32)


def _rewards(P, K, rng):
    r = np.zeros((P, K))
    for p in range(P):
        n = round(SUCCESSES[p % len(SUCCESSES)] * K / 8)
        r[p, rng.permutation(K)[:n]] = 1.0
    return r


def _rollouts(case):
    """Lengths, survival tables (a Beta law over the prefix fraction, per prompt), rewards, advantages.
    Part of the case (output shapes follow from them); everything else is drawn from the seed."""
    rng = np.random.default_rng(1)
    P, K = case["P"], case["K"]
    lengths = _lengths(case, rng)
    horizon = lengths.reshape(P, K).max(axis=1)
    off = np.zeros(P + 1, dtype=np.int64)
    off[1:] = np.cumsum(horizon)
    ab = rng.uniform(1.0, 4.0, size=(P, 2))
    xi = np.concatenate([synth.beta_survival_table(ab[p, 0], ab[p, 1], int(horizon[p])) for p in range(P)])
    rewards = _rewards(P, K, rng)
    adv = (rewards - rewards.mean(axis=1, keepdims=True)).reshape(-1).astype(np.float32)
    return dict(lengths=lengths, xi=xi, xi_off=off, rewards=rewards.reshape(-1), advantage=adv)


def _targets(g, n, V):
    """Token ids with P(rank r) ~ 1/r, the ranks spread over the vocabulary."""
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    rank = torch.exp(u * math.log(V + 1.0)).long().clamp_(1, V) - 1
    perm = torch.randperm(V, generator=g, device=DEV)
    return perm[rank].to(torch.int32)


def _head(g, V, d):
    return (torch.randn((V, d), generator=g, device=DEV) * W_STD).to(torch.bfloat16)


def _hidden(g, n, d, w, tgt):
    """N(0, 1) rows plus a component along the target's head row that raises its logit by 0 .. log V + 4."""
    h = torch.empty((n, d), dtype=torch.bfloat16, device=DEV)
    for a in range(0, n, 16384):
        b = min(n, a + 16384)
        wo = w[tgt[a:b].long()].float()
        boost = torch.rand(b - a, generator=g, device=DEV) * (math.log(w.shape[0]) + 4.0)
        x = torch.randn((b - a, d), generator=g, device=DEV)
        h[a:b] = (x + (boost / wo.square().sum(1))[:, None] * wo).to(torch.bfloat16)
    return h


def _logp_old(g, h, w, tgt, sigma):
    """Log-probs of an old policy: the head's own (to about 1e-4) plus N(0, sigma^2), no ratio within
    1e-3 of a clip bound, so that no rounding decides whether a token is clipped."""
    n = h.shape[0]
    lp = torch.empty(n, dtype=torch.float32, device=DEV)
    for a in range(0, n, 4096):
        b = min(n, a + 4096)
        o = tgt[a:b].long()[:, None]
        z = (h[a:b] @ w.t()).float()
        zo = (h[a:b].float() * w[o[:, 0]].float()).sum(1)
        z.scatter_(1, o, zo[:, None])
        lp[a:b] = zo - torch.logsumexp(z, dim=1)
    noise = sigma * torch.randn(n, generator=g, device=DEV)
    for bound in (-math.log1p(EPS), -math.log1p(-EPS)):
        near = (noise - bound).abs() < 1e-3
        noise = torch.where(near, noise + 2e-3, noise)
    return lp + noise


def _dev(a, dt):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device=DEV, dtype=dt)


def _loss_inputs(case, seed):
    g, rng = _gen(seed), np.random.default_rng([seed, 2])
    n, R, d, V = case["tokens"], case["seqs"], case["d"], case["V"]
    w = _head(g, V, d)
    tgt = _targets(g, n, V)
    h = _hidden(g, n, d, w, tgt)
    old = _logp_old(g, h, w, tgt, case["sigma_lp"])
    # kept prefixes of R completions, their weights those of a cutoff uniform on 1 .. 1.5 H
    share = rng.uniform(0.3, 1.7, R)
    cu = np.rint(np.concatenate([[0.0], np.cumsum(share / share.sum())]) * n).astype(np.int64)
    seq = np.repeat(np.arange(R, dtype=np.int32), np.diff(cu))
    t = np.arange(n) - cu[seq]
    T = np.ceil(1.5 * np.diff(cu))[seq]
    adv = _rewards((R + 7) // 8, 8, rng)
    adv = (adv - adv.mean(axis=1, keepdims=True)).reshape(-1)[:R].astype(np.float32)
    return dict(hidden=h, w_head=w, target=tgt, logp_old=old, weight=_dev(T / (T - t), torch.float32),
                seq_id=_dev(seq, torch.int32), advantage=_dev(adv, torch.float32))


def _update_inputs(case, seed):
    r, g = _rollouts(case), _gen(seed)
    S, d, V = int(r["lengths"].sum()), case["d"], case["V"]
    w = _head(g, V, d)
    tgt = _targets(g, S, V)
    h = _hidden(g, S, d, w, tgt)
    r.update(w_head=w, target=tgt, hidden=h, total=S, logp_old=_logp_old(g, h, w, tgt, case["sigma_lp"]))
    return r


def _proxy_inputs(case, seed):
    g = _gen(seed)
    w = _head(g, case["V"], case["d"])
    tgt = _targets(g, case["tokens"], case["V"])
    return dict(w_head=w, target=tgt, hidden=_hidden(g, case["tokens"], case["d"], w, tgt))


def _weights_inputs(case, seed):
    """Top-k lists in the shape a rollout engine reports them: k distinct ids a row, from a pool of 64
    per prompt so that the completions' lists overlap; mass 0.5 .. 0.95, decreasing."""
    r, g = _rollouts(case), _gen(seed)
    P, K, k = case["P"], case["K"], case["topk"]
    S = int(r["lengths"].sum())
    full = np.concatenate([[0], np.cumsum(r["lengths"])]).astype(np.int32)
    pool = torch.stack([torch.randperm(151936, generator=g, device=DEV)[:64] for _ in range(P)])
    prompt = _dev(np.repeat(np.arange(P * K) // K, r["lengths"]), torch.int64)
    pick = torch.rand((S, 64), generator=g, device=DEV).topk(k, dim=1).indices
    ids = torch.gather(pool[prompt], 1, pick).to(torch.int32)
    e = (-torch.log(torch.rand((S, k), generator=g, device=DEV) + 1e-9)) ** 3
    e = (e / e.sum(1, keepdim=True)).sort(dim=1, descending=True).values
    mass = 0.5 + 0.45 * torch.rand((S, 1), generator=g, device=DEV)
    logp = torch.log((e * mass).clamp_min(1e-30)).float()
    gamma = 3584.0 * torch.exp(0.6 * torch.randn(S, generator=g, device=DEV))
    return dict(gamma=gamma, ids=ids, logp=logp, lengths=_dev(r["lengths"], torch.int32), full=_dev(full, torch.int32),
                rewards=_dev(r["rewards"], torch.float32), xi_off=_dev(r["xi_off"], torch.int64),
                total=int(r["xi_off"][-1]), host=r)


def _design_inputs(case, seed):
    """Noisy per-step weights that fall along a completion; exactly zero once the completions still
    running share a reward, and everywhere for a prompt whose completions all do."""
    r = _rollouts(case)
    rng = np.random.default_rng([seed, 3])
    w, off = np.empty(int(r["xi_off"][-1])), r["xi_off"]
    rew, lens = r["rewards"].reshape(case["P"], case["K"]), r["lengths"].reshape(case["P"], case["K"])
    for p in range(case["P"]):
        T = int(off[p + 1] - off[p])
        t = np.arange(T)
        good, bad = lens[p][rew[p] > 0.5], lens[p][rew[p] <= 0.5]
        both = min(good.max(initial=0), bad.max(initial=0))
        w[off[p]:off[p + 1]] = 3584.0 * np.exp(0.6 * rng.standard_normal(T) - rng.uniform(0, 3) * t / T)
        w[off[p]:off[p + 1]] *= np.where(t < both, rng.uniform(0.05, 0.5, T), 0.0)
    return dict(w=w, xi_off=off, budget=case["kept"] * float(np.diff(off).mean()), lam=2.0 / case["median"])


# ---------------------------------------------------------------------------
# the measured pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    path = case["path"]
    if path == "loss":
        s = _loss_inputs(case, seed)
        n, d, V = case["tokens"], case["d"], case["V"]
        s["flags"] = ((pspo.PSPO_ACCUMULATE_DW if case["accumulate"] else 0)
                      | (pspo.PSPO_KEEP_LOGITS if case["keep"] else 0))
        s["d_w"] = torch.zeros((V, d), dtype=torch.float32, device=DEV)
        s["d_h"] = torch.empty((n, d), dtype=torch.float32, device=DEV)
        s["ws"] = torch.empty(max(pspo.loss_workspace_bytes(n, d, V, s["flags"]), 256), dtype=torch.uint8, device=DEV)
    elif path == "update":
        r = _update_inputs(case, seed)
        dw = pipeline.DeviceWorkload(
            P=case["P"], K=case["K"], d=case["d"], V=case["V"], capacity=r["total"], xi=_dev(r["xi"], torch.float64),
            xi_off=_dev(r["xi_off"], torch.int64), lengths=_dev(r["lengths"], torch.int32),
            advantage=_dev(r["advantage"], torch.float32), target_full=r["target"], logp_old_full=r["logp_old"],
            hidden_full=r["hidden"], w_head=r["w_head"], eps_low=EPS, eps_high=EPS,
            loss_scale=1.0 / (case["P"] * case["K"]))
        s = dict(step=pipeline.Step(dw), philox=PHILOX)
    elif path == "proxy":
        s = _proxy_inputs(case, seed)
        need = pspo.score_proxy_workspace_bytes(case["tokens"], case["d"], case["V"])
        s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
    elif path == "pack":
        r, g = _rollouts(case), _gen(seed)
        S = int(r["lengths"].sum())
        s = dict(xi=_dev(r["xi"], torch.float64), xi_off=_dev(r["xi_off"], torch.int64),
                 lengths=_dev(r["lengths"], torch.int32), total=S, philox=PHILOX, err=torch.zeros(1, dtype=torch.int32, device=DEV),
                 target=torch.randint(0, 152064, (S,), generator=g, device=DEV, dtype=torch.int32),
                 logp_old=-torch.rand(S, generator=g, device=DEV) * 12,
                 hidden=torch.randn((S, case["d"]), generator=g, device=DEV).to(torch.bfloat16))
    elif path == "weights":
        s = _weights_inputs(case, seed)
    else:
        s = _design_inputs(case, seed)
        s["total"] = int(s["xi_off"][-1])
        s["w"], s["xi_off"] = _dev(s["w"], torch.float64), _dev(s["xi_off"], torch.int64)
    s["case"] = dict(case)
    return s


def run(s):
    c = s["case"]
    path = c["path"]
    if path == "loss":
        o = pspo.loss_fwd_bwd(s["hidden"], s["w_head"], s["target"], s["logp_old"], s["weight"], s["seq_id"],
                              s["advantage"], c["tokens"], EPS, EPS, 1.0 / c["seqs"], flags=s["flags"],
                              d_w_head=s["d_w"], d_hidden=s["d_h"], workspace=s["ws"], want_logp=c["logp"])
        return {k: o[k] for k in ("loss", "d_hidden", "d_w_head", "logp_new", "stats")}
    if path == "update":
        o = s["step"](s["philox"], want_logp=c["logp"])
        n = o["N"]
        return dict({k: o[k] for k in ("loss", "d_hidden", "d_w_head", "logp_new", "stats", "cutoffs")},
                    src_row=o["pack"]["src_row"][:n], weight=o["pack"]["weight"][:n])
    if path == "proxy":
        o = pspo.score_proxy(s["hidden"], s["w_head"], s["target"], c["tokens"], want_p_sq=c["p_sq"],
                             workspace=s["ws"])
        return {k: o[k] for k in ("gamma", "logp", "p_sq")}
    if path == "pack":
        cut = pspo.sample_cutoffs(s["xi"], s["xi_off"], s["lengths"], c["P"], c["K"], s["philox"], err_flag=s["err"])
        pk = pspo.pack_prefixes(cut, s["lengths"], s["xi"], s["xi_off"], c["P"], c["K"], s["total"],
                                target_full=s["target"], logp_old_full=s["logp_old"], hidden_full=s["hidden"],
                                err_flag=s["err"])
        n = int(pk["n_tokens"].item())   # what sizes the loss call that follows
        return dict(cutoffs=cut, cu_seqlens=pk["cu_seqlens"], err=s["err"],
                    **{k: pk[k][:n] for k in ("src_row", "seq_id", "weight", "target", "logp_old", "hidden")})
    if path == "weights":
        return pspo.design_weights(s["gamma"], s["ids"], s["logp"], s["lengths"], s["full"], s["rewards"],
                                   s["xi_off"], c["P"], c["K"], s["total"], want_parts=True)
    return pspo.design_cutoffs(s["w"], s["xi_off"], c["P"], s["total"], s["budget"], variant=c["variant"],
                               lam=s["lam"])


# ---------------------------------------------------------------------------
# work and tolerances
# ---------------------------------------------------------------------------

# shares of the tokens: kept by the cutoffs, of completions with a non-zero advantage, and of those
# not clipped
KEPT, NONZERO, UNCLIPPED = 0.65, 0.78, 0.85


def work(case):
    path = case["path"]
    if path in ("loss", "update"):
        d, V = case["d"], case["V"]
        n = case["tokens"] if path == "loss" else KEPT * _mean_tokens(case)
        fwd = n if case["logp"] else NONZERO * n
        flops = (2 * fwd + 4 * NONZERO * UNCLIPPED * n) * V * d
        by = V * d * (2 + 4 + (4 if case.get("accumulate") else 0)) + n * d * (2 + 4) + n * 20
        if path == "update":
            by += n * (2 + 2) * d + n * 36
        return dict(bytes=by, flops=flops)
    if path == "proxy":
        n, d, V = case["tokens"], case["d"], case["V"]
        return dict(bytes=2 * d * (V + n) + 16 * n, flops=2.0 * n * V * d)
    n = _mean_tokens(case)
    if path == "pack":
        return dict(bytes=KEPT * n * (4 * case["d"] + 36), flops=0.0)
    steps = 1.8 * n / case["K"]      # the longest completion of each prompt
    if path == "weights":
        return dict(bytes=n * (8 * case["topk"] + 4) + 24 * steps, flops=0.0)
    return dict(bytes=16 * steps, flops=0.0)


def _mean_tokens(case):
    return case["P"] * case["K"] * case["median"] * math.exp(case["sigma"] ** 2 / 2)


def tolerance(case):
    path = case["path"]
    if path == "pack":
        return "exact"
    if path in ("weights", "design"):
        return dict(rel=1e-12, max=1e-10)      # float64 sums in another order
    if path == "proxy":
        return dict(rel=1e-5, max=1e-4)        # float32 sums
    # bf16 logit gradients with exact target entries: up to 5e-5 from the 64-bit result
    return dict(rel=2e-4, max=0.03)


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------

def _exact_loss(h, w, tgt, old, weight, seq, adv, scale, want_logp):
    f32 = lambda x: float(np.float32(x))   # noqa: E731  (the call takes its scalars in float32)
    lo, hi, sc = f32(EPS), f32(EPS), f32(scale)
    n, d = h.shape
    w64 = w.double()
    dw = torch.zeros_like(w64)
    dh = torch.zeros((n, d), dtype=torch.float64, device=DEV)
    logp = torch.empty(n, dtype=torch.float64, device=DEV)
    tot = torch.zeros(5, dtype=torch.float64, device=DEV)
    wt64 = w64.t()
    for a in range(0, n, 2048):
        b = min(n, a + 2048)
        hc, o = h[a:b].double(), tgt[a:b].long()
        z = hc @ wt64
        lse = torch.logsumexp(z, dim=1)
        lp = z.gather(1, o[:, None])[:, 0] - lse
        logp[a:b] = lp
        A, c = adv[seq[a:b].long()].double(), weight[a:b].double()
        rho = torch.exp(lp - old[a:b].double())
        s = torch.minimum(rho * A, rho.clamp(1 - lo, 1 + hi) * A)
        mu = ((A > 0) & (rho <= 1 + hi)) | ((A < 0) & (rho >= 1 - lo))
        delta = torch.where(mu, -sc * c * rho * A, torch.zeros_like(A))
        tot += torch.stack([(c * s).sum(), (c * s).abs().sum(), ((A != 0) & ~mu).double().sum(),
                            (A == 0).double().sum(), (delta != 0).double().sum()])
        act = delta != 0
        if bool(act.any()):
            G = z[act].sub_(lse[act][:, None]).exp_().mul_(-delta[act][:, None])
            G.scatter_add_(1, o[act][:, None], delta[act][:, None])
            dh[a:b][act] = G @ w64
            dw.addmm_(G.t(), hc[act])
        del z
    t = tot.tolist()
    stats = torch.tensor([sc * t[1], t[2], t[3], float(weight[:n].max()), t[4]], dtype=torch.float64)
    return dict(loss=torch.tensor([-sc * t[0]], dtype=torch.float64), d_hidden=dh, d_w_head=dw,
                logp_new=logp if want_logp else None, stats=stats)


def _philox_word0(ctr, seed):
    """Word 0 of Philox4x32-10 (Salmon et al., SC'11) with counter (r, 0, 0, 0), the key from `seed`."""
    m = np.uint64(0xFFFFFFFF)
    s32 = np.uint64(32)
    x = [ctr.astype(np.uint64)] + [np.zeros_like(ctr, dtype=np.uint64) for _ in range(3)]
    k = [seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF]
    for _ in range(10):
        a, b = x[0] * np.uint64(0xD2511F53), x[2] * np.uint64(0xCD9E8D57)
        x = [(b >> s32) ^ x[1] ^ np.uint64(k[0]), b & m, (a >> s32) ^ x[3] ^ np.uint64(k[1]), a & m]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    return x[0]


def _exact_pack(r, P, K, philox):
    """Cutoffs, source rows, completion ids and weights of the kept tokens."""
    q = np.maximum(np.floor(r["xi"] * 2.0 ** 32), 1.0)
    x = _philox_word0(np.arange(P * K, dtype=np.uint64), philox).astype(np.float64)
    off, lens = r["xi_off"], r["lengths"]
    cut = np.array([min(int(lens[i]), int((x[i] < q[off[i // K]:off[i // K + 1]]).sum())) for i in range(P * K)])
    full = np.concatenate([[0], np.cumsum(lens)])
    src = np.concatenate([full[i] + np.arange(cut[i]) for i in range(P * K)]).astype(np.int64)
    weight = np.concatenate([2.0 ** 32 / q[off[i // K]:off[i // K] + cut[i]] for i in range(P * K)])
    return cut.astype(np.int32), src, np.repeat(np.arange(P * K), cut), weight.astype(np.float32)


def exact(case, seed):
    path = case["path"]
    if path == "loss":
        if work(case)["flops"] > 4e14:
            return None
        s = _loss_inputs(case, seed)
        return _exact_loss(s["hidden"], s["w_head"], s["target"], s["logp_old"], s["weight"], s["seq_id"],
                           s["advantage"], 1.0 / case["seqs"], case["logp"])
    if path == "update":
        if work(case)["flops"] > 4e14:
            return None
        r = _update_inputs(case, seed)
        cut, src, seq, weight = _exact_pack(r, case["P"], case["K"], PHILOX)
        at = _dev(src, torch.int64)
        o = _exact_loss(r["hidden"][at], r["w_head"], r["target"][at], r["logp_old"][at], _dev(weight, torch.float32),
                        _dev(seq, torch.int64), _dev(r["advantage"], torch.float32), 1.0 / (case["P"] * case["K"]),
                        case["logp"])
        return dict(o, cutoffs=cut, src_row=src.astype(np.int32), weight=weight)
    if path == "proxy":
        s = _proxy_inputs(case, seed)
        w64 = s["w_head"].double()
        wt64 = w64.t()
        gam, lps, psq = [], [], []
        for a in range(0, case["tokens"], 2048):
            h, o = s["hidden"][a:a + 2048].double(), s["target"][a:a + 2048].long()
            z = h @ wt64
            z -= torch.logsumexp(z, dim=1)[:, None]
            lp = z.gather(1, o[:, None])[:, 0]
            p = z.exp_()
            sq = p.square().sum(1)
            rest = p.scatter_(1, o[:, None], 0.0)
            gam.append(h.square().sum(1) * (rest.sum(1).square() + rest.square().sum(1)))
            lps.append(lp)
            psq.append(sq)
            del z, p, rest
        return dict(gamma=torch.cat(gam), logp=torch.cat(lps), p_sq=torch.cat(psq) if case["p_sq"] else None)
    if path == "pack":
        r = _rollouts(case)
        weight = _exact_pack(r, case["P"], case["K"], PHILOX)[3]
        return dict(cutoffs=None, cu_seqlens=None, err=None, src_row=None, seq_id=None, weight=weight, target=None,
                    logp_old=None, hidden=None)
    if path == "weights":
        return _exact_weights(case, _weights_inputs(case, seed))
    s = _design_inputs(case, seed)
    return _exact_design(s["w"], s["xi_off"], s["budget"], case["variant"], s["lam"])


def _exact_weights(case, s):
    P, K, host = case["P"], case["K"], s["host"]
    full, lens = np.concatenate([[0], np.cumsum(host["lengths"])]), host["lengths"]
    gb, u = [], []
    for p in range(P):
        T = int(host["xi_off"][p + 1] - host["xi_off"][p])
        rows = slice(int(full[p * K]), int(full[(p + 1) * K]))
        names = torch.unique(s["ids"][rows])
        acc = torch.zeros((T, names.numel()), dtype=torch.float64, device=DEV)
        gsum, n, good, rest = (torch.zeros(T, dtype=torch.float64, device=DEV) for _ in range(4))
        for k in range(K):
            r, L = p * K + k, int(lens[p * K + k])
            a = int(full[r])
            sign = 1.0 if host["rewards"][r] > 0.5 else -1.0
            pr = torch.exp(s["logp"][a:a + L].double())
            acc[:L].scatter_add_(1, torch.searchsorted(names, s["ids"][a:a + L].contiguous()), sign * pr)
            rest[:L] += sign * (1.0 - pr.sum(1)).clamp_min(0.0)
            gsum[:L] += s["gamma"][a:a + L].double()
            n[:L] += 1.0
            good[:L] += 1.0 if sign > 0 else 0.0
        uu = (0.5 - 0.5 * (acc.abs().sum(1) + rest.abs()) / n).clamp_min(0.0)
        u.append(torch.where((good == 0) | (good == n), torch.zeros_like(uu), uu))
        gb.append(gsum / n)
    gb, u = torch.cat(gb), torch.cat(u)
    return dict(w=gb * u, gamma_bar=gb, u=u)


def _exact_design(w, off, budget, variant, lam):
    out = np.empty_like(w)
    for p in range(len(off) - 1):
        v = w[off[p]:off[p + 1]]
        T = len(v)
        t = np.arange(T)
        if variant == 2:
            x = (T - t) / T
        elif variant == 3:
            x = np.exp(-lam * t)
        elif budget >= T:
            x = np.ones(T)
        elif not v.any():
            x = np.full(T, budget / T)
        elif variant == 1:
            x = np.minimum.accumulate(np.minimum(1.0, budget * np.sqrt(v) / np.sqrt(v).sum()))
        else:
            W, L = [], []
            for a in v.tolist():
                W.append(a)
                L.append(1)
                while len(W) > 1 and W[-2] * L[-1] < W[-1] * L[-2]:
                    a2, l2 = W.pop(), L.pop()
                    W[-1] += a2
                    L[-1] += l2
            L, sc = np.array(L), np.sqrt(np.array(W) / np.array(L))
            rest = np.cumsum((L * sc)[::-1])[::-1]
            sat, kappa = 0, None
            for m in range(len(L)):
                if rest[m] == 0.0:
                    break
                kappa = (budget - sat) / rest[m]
                if kappa * sc[m] <= 1.0:
                    break
                sat, kappa = sat + int(L[m]), None
            start = np.concatenate([[0], np.cumsum(L)[:-1]])
            if kappa is None:
                x = np.repeat(np.where(start < sat, 1.0, (budget - sat) / max(T - sat, 1)), L)
            else:
                x = np.repeat(np.minimum(1.0, kappa * sc), L)
        out[off[p]:off[p + 1]] = x if variant == 2 else np.maximum(x, 2.0 ** -32)
    return out
