"""GPU: the design weights over the list shapes that choose the group width (lists of 1 to 256 entries,
1 to 64 completions, up to 256 entries a step) or the wave per step (5 completions or more with lists of
up to 4 entries, up to 128 a step: one and two entries a lane, both sides of each limit), step counts that
leave groups and blocks part empty or send such lists to the table (past 1300 steps a completion), lists
that share all their ids (every table slot summed K times), none, or repeat one, and ids past the table's
size; batches on both sides of the 64 prompts that one load finds, with empty prompts among them.
Repeated calls give the same bits.

Both sides add the same float64 terms in another order: at most 256 terms of at most 1, so 1e-13.
"""
import numpy as np
import pytest
import torch

from paper_2606_29758_amd import pspo

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (64, 1), (64, 4), (2, 3), (5, 7), (8, 8), (8, 16), (16, 16), (9, 17), (4, 64), (3, 65), (3, 85),
          (2, 128), (1, 256), (4, 4), (5, 1), (5, 4), (5, 5), (16, 4), (23, 1), (24, 1), (32, 4), (33, 3), (43, 3), (64, 2)]


def _reference(gamma, ids, logp, lengths, rewards, P, K):
    full = np.concatenate([[0], np.cumsum(lengths)])
    w, gb, u = [], [], []
    for p in range(P):
        for t in range(lengths[p * K:(p + 1) * K].max()):
            sums, rest, gs, n, good = {}, 0.0, 0.0, 0, 0
            for r in range(p * K, (p + 1) * K):
                if lengths[r] <= t:
                    continue
                row = full[r] + t
                sign = 1.0 if rewards[r] > 0.5 else -1.0
                pr = np.exp(logp[row].astype(np.float64))
                for i, x in zip(ids[row].tolist(), pr.tolist()):
                    if i >= 0:
                        sums[i] = sums.get(i, 0.0) + sign * x
                rest += sign * max(0.0, 1.0 - pr.sum())
                gs, n, good = gs + float(gamma[row]), n + 1, good + int(sign > 0)
            uu = 0.0 if good in (0, n) else max(0.0, 0.5 - 0.5 * (sum(map(abs, sums.values())) + abs(rest)) / n)
            gb.append(gs / n)
            u.append(uu)
            w.append(gs / n * uu)
    return np.array(w), np.array(gb), np.array(u)


@pytest.mark.parametrize("K,topk", SHAPES)
def test_shapes(K, topk):
    rng = np.random.default_rng(K * 1000 + topk)
    P = 3
    lengths = rng.integers(1, 24, P * K).astype(np.int32)
    rewards = (rng.random(P * K) < 0.5).astype(np.float32)
    S = int(lengths.sum())
    gamma = rng.gamma(2.0, 500.0, S).astype(np.float32)
    logp = np.log(rng.dirichlet(np.ones(topk), S) * rng.uniform(0.3, 1.0, (S, 1)) + 1e-12).astype(np.float32)
    full = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    horizon = lengths.reshape(P, K).max(axis=1)
    off = np.concatenate([[0], np.cumsum(horizon)]).astype(np.int64)
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dt)   # noqa: E731
    for law in ("shared", "spread", "repeats"):
        print(f"[weights] K={K} topk={topk} ids={law}", flush=True)
        if law == "shared":
            ids = np.argsort(rng.random((S, topk)), axis=1)
        elif law == "spread":
            ids = rng.integers(0, 2 ** 31 - 1, (S, topk))
        else:
            ids = rng.integers(-1, 3, (S, topk))     # repeated in a list; negative: no entry
        out = pspo.design_weights(t(gamma, torch.float32), t(ids, torch.int32), t(logp, torch.float32),
                                  t(lengths, torch.int32), t(full, torch.int32), t(rewards, torch.float32),
                                  t(off, torch.int64), P, K, int(off[-1]), want_parts=True)
        again = pspo.design_weights(t(gamma, torch.float32), t(ids, torch.int32), t(logp, torch.float32),
                                    t(lengths, torch.int32), t(full, torch.int32), t(rewards, torch.float32),
                                    t(off, torch.int64), P, K, int(off[-1]), want_parts=True)
        assert all(torch.equal(out[k], again[k]) for k in ("w", "gamma_bar", "u"))
        for got, want in zip((out["w"], out["gamma_bar"], out["u"]), _reference(gamma, ids, logp, lengths, rewards, P, K)):
            scale = 1000.0 if got is out["w"] else 1.0
            np.testing.assert_allclose(got.cpu().numpy(), want, rtol=1e-13, atol=1e-13 * scale)


@pytest.mark.parametrize("P,K,topk,longest", [(64, 2, 3, 6), (65, 2, 3, 6), (65, 24, 2, 4), (131, 8, 4, 5), (3, 5, 3, 2300)])
def test_batches(P, K, topk, longest):
    print(f"[weights] P={P} K={K} topk={topk} longest={longest}", flush=True)
    rng = np.random.default_rng(P * 100 + K)
    lengths = rng.integers(0 if P > 3 else longest - 30, longest, P * K).astype(np.int32)
    if P > 3:
        lengths[[0, 1]] = longest
        for p in (1, 2, P - 2):          # prompts without a step, the last but one among them
            lengths[p * K:(p + 1) * K] = 0
    rewards = (rng.random(P * K) < 0.5).astype(np.float32)
    S = int(lengths.sum())
    gamma = rng.gamma(2.0, 500.0, S).astype(np.float32)
    logp = np.log(rng.dirichlet(np.ones(topk), S) * rng.uniform(0.3, 1.0, (S, 1)) + 1e-12).astype(np.float32)
    ids = rng.integers(0, 12, (S, topk))
    full = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(lengths.reshape(P, K).max(axis=1))]).astype(np.int64)
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dt)   # noqa: E731
    out = pspo.design_weights(t(gamma, torch.float32), t(ids, torch.int32), t(logp, torch.float32),
                              t(lengths, torch.int32), t(full, torch.int32), t(rewards, torch.float32),
                              t(off, torch.int64), P, K, int(off[-1]), want_parts=True)
    for got, want in zip((out["w"], out["gamma_bar"], out["u"]), _reference(gamma, ids, logp, lengths, rewards, P, K)):
        scale = 1000.0 if got is out["w"] else 1.0
        np.testing.assert_allclose(got.cpu().numpy(), want, rtol=1e-13, atol=1e-13 * scale)
