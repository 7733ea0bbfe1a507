"""GPU: merging the vocabulary-tile partials (384 rows each) of the loss and of the score proxy,
where the slices of a merge (1 per token for one tile, 4 up to 8 tiles, then 32; 32 tokens per block)
come out uneven: fewer tiles than slices, exactly as many, one more, several rounds; one token, and
counts around a block.

Tolerances: a log-prob is z_o - M - log(sum), float32 sums of positive terms and logits of float32
products, so about log2(V) * 2^-24 relative on the sum and 2^-24 |z| on the logits: 1e-5 absolute
covers |z| < 40.  gamma is a product of such sums: 2e-5 relative.
"""
import numpy as np
import pytest
import torch

from paper_2606_29758_amd import pspo, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [300, 384, 385, 384 * 4, 384 * 5, 384 * 8, 384 * 8 + 1, 384 * 31, 384 * 32, 384 * 32 + 1, 384 * 65 + 383])
@pytest.mark.parametrize("N", [1, 31, 32, 65])
def test_merge(N, V):
    print(f"[merge] N={N} V={V}", flush=True)
    d, rng = 64, np.random.default_rng(N * 7 + V)
    f = lambda b: (b.astype(np.uint32) << 16).view(np.float32).astype(np.float64)             # noqa: E731
    h = synth.round_to_bf16_bits(rng.normal(0.0, 1.0, (N, d)).astype(np.float32))
    W = synth.round_to_bf16_bits(rng.normal(0.0, 0.3, (V, d)).astype(np.float32))
    tgt = rng.integers(0, V, N).astype(np.int32)
    tgt[0] = V - 1
    z = f(h) @ f(W).T
    p = np.exp(z - z.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    po = p[np.arange(N), tgt].copy()
    bits = lambda b: torch.from_numpy(b.view(np.int16)).to("cuda").view(torch.bfloat16)       # noqa: E731
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dt)   # noqa: E731
    hb, wb, tb = bits(h), bits(W), t(tgt, torch.int32)
    lp_old = t(np.log(po), torch.float32)
    out = pspo.loss_fwd_bwd(hb, wb, tb, lp_old, t(np.ones(N), torch.float32), t(np.zeros(N), torch.int32),
                            t(np.ones(1), torch.float32), N, 0.2, 0.2, 1.0, want_logp=True)
    assert np.max(np.abs(out["logp_new"].double().cpu().numpy() - np.log(po))) < 1e-5
    assert abs(float(out["loss"].item()) + N) < 1e-5 * N      # rho = 1, A = 1, weight 1
    prox = pspo.score_proxy(hb, wb, tb, N, want_p_sq=True)
    sq = (p ** 2).sum(axis=1)
    p[np.arange(N), tgt] = 0.0
    gamma = (f(h) ** 2).sum(axis=1) * ((1.0 - po) ** 2 + (p ** 2).sum(axis=1))
    assert np.max(np.abs(prox["logp"].double().cpu().numpy() - np.log(po))) < 1e-5
    assert np.max(np.abs(prox["gamma"].double().cpu().numpy() / gamma - 1.0)) < 2e-5
    assert np.max(np.abs(prox["p_sq"].double().cpu().numpy() / sq - 1.0)) < 2e-5
