"""GPU: the budgeted solve where its block search can go wrong: step counts around a wave (64), a
work-group (1024), powers of two (the joins of the search) and the LDS limit (13040 steps, beyond
which the blocks lie in the workspace); weights that end in one block, in blocks of one step each, in
one that pools everything at its last step, in ties and zeros, and with trailing zeros; the running
minimum of the heuristic over the same.

Both sides add the same float64 terms (up to 16390 positive ones) in another order, the reference one
after another: at most 16390 * 2^-53 = 1.8e-12 relative, about the root of the count in practice: 1e-12.
"""
import numpy as np
import pytest
import torch

from paper_2606_29758_amd import pspo

pytestmark = pytest.mark.gpu

FLOOR = 2.0 ** -32


def _weights(kind, T, rng):
    t = np.arange(T)
    if kind == "rising":
        return 1.0 + t
    if kind == "falling":
        return 1.0 + (T - t)
    if kind == "spike":      # T - 1 blocks on the stack, all pooled by the last step
        w = 1.0 + (T - t).astype(np.float64)
        w[-1] = 10.0 * w.sum()
        return w
    if kind == "spikes":     # deep stacks that are cut back again and again
        w = 1.0 + (T - t) + 0.0
        w[99::100] *= 1.0 + 40.0 * rng.random(len(w[99::100]))
        return w
    if kind == "ties":
        return rng.integers(0, 3, T).astype(np.float64)
    if kind == "tail":
        return np.where(t < max(1, T // 3), np.exp(rng.standard_normal(T)), 0.0)
    return np.exp(0.6 * rng.standard_normal(T) - 2.0 * t / T)


def _reference(w, budget, heuristic):
    T = len(w)
    if budget >= T:
        return np.ones(T)
    if not w.any():
        return np.full(T, budget / T)
    if heuristic:
        return np.maximum(np.minimum.accumulate(np.minimum(1.0, budget * np.sqrt(w) / np.sqrt(w).sum())), FLOOR)
    W, L = [], []
    for a in w.tolist():
        W.append(a)
        L.append(1)
        while len(W) > 1 and W[-2] * L[-1] < W[-1] * L[-2]:
            a2, l2 = W.pop(), L.pop()
            W[-1] += a2
            L[-1] += l2
    L, sc = np.array(L), np.sqrt(np.array(W) / np.array(L))
    rest = np.cumsum((L * sc)[::-1])[::-1]
    start = np.concatenate([[0], np.cumsum(L)[:-1]])
    kappa = np.divide(budget - start, rest, out=np.full(len(L), -1.0), where=rest > 0)
    m = int(np.argmax((rest == 0) | (kappa * sc <= 1.0)))
    if rest[m] == 0:
        x = np.where(start < start[m], 1.0, (budget - start[m]) / max(T - start[m], 1))
    else:
        x = np.minimum(1.0, kappa[m] * sc)
    return np.maximum(np.repeat(x, L), FLOOR)


@pytest.mark.parametrize("kind", ["rising", "falling", "spike", "spikes", "ties", "tail", "noise"])
def test_tables(kind):
    rng = np.random.default_rng(3)
    sizes = [1, 2, 3, 63, 64, 65, 129, 1000, 1023, 1024, 1025, 4097, 13039, 13040, 13041, 16390]
    w = [_weights(kind, T, rng) for T in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    dw = torch.from_numpy(np.concatenate(w)).to("cuda")
    doff = torch.from_numpy(off).to("cuda")
    for budget in (0.5, 60.0, 900.0, 6000.0):
        for variant in (0, 1):
            print(f"[design] kind={kind} budget={budget} variant={variant}", flush=True)
            x = pspo.design_cutoffs(dw, doff, len(sizes), int(off[-1]), budget, variant=variant).cpu().numpy()
            for p, T in enumerate(sizes):
                want = _reference(w[p], budget, variant == 1)
                np.testing.assert_allclose(x[off[p]:off[p + 1]], want, rtol=1e-12, err_msg=str(T))
