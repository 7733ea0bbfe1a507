"""GPU: the backward of few tokens in one vocabulary chunk against the chunked one (the same call in a
workspace 256 bytes short of the one-chunk plan), around the row tile (384) and up to the token block
(768) and on widths whose chunks are narrow (d = 4096: 6144 rows; 13,001 rows are two chunks and a
partial tile).  The logits and their gradient are the same bits on both; dW rows and d_hidden rows are
float32 sums over tokens and over the vocabulary in another order: 2e-6 of the row's norm covers sums
of 13,001 terms that are added 32 at a time.
"""
import numpy as np
import pytest
import torch

from paper_2606_29758_amd import pspo, synth

from parity_util import loss_in

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("N", [1, 383, 385, 767, 768])
def test_one_chunk(N, accumulate):
    print(f"[one chunk] N={N} accumulate={accumulate}", flush=True)
    d, V, R = 4096, 13001, 3
    rng = np.random.default_rng(N)
    bits = lambda a: torch.from_numpy(synth.round_to_bf16_bits(a.astype(np.float32)).view(np.int16)).to("cuda").view(torch.bfloat16)   # noqa: E731
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dt)   # noqa: E731
    args = (bits(rng.normal(0.0, 1.0, (N, d))), bits(rng.normal(0.0, 0.02, (V, d))),
            t(rng.integers(0, V, N), torch.int32), t(-9.0 + 0.1 * rng.normal(size=N), torch.float32),
            t(1.0 + rng.random(N), torch.float32), t(np.sort(rng.integers(0, R, N)), torch.int32),
            t([1.0, -1.0, 0.5], torch.float32), N, 0.9, 0.9, 0.25)
    need = pspo.loss_workspace_bytes(N, d, V, 0)
    start = torch.randn((V, d), device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    outs = []
    for size, chunks in ((need, 1), (need - 256, 2)):
        out, ran = loss_in(size, *args, flags=pspo.PSPO_ACCUMULATE_DW if accumulate else 0, d_w_head=start.clone())
        assert ran == chunks
        outs.append((out["loss"], out["logp_new"], out["d_hidden"], out["d_w_head"] - start if accumulate else out["d_w_head"]))
    (l0, p0, h0, w0), (l1, p1, h1, w1) = outs
    assert torch.equal(l0, l1) and torch.equal(p0, p1)
    for a, b in ((h0, h1), (w0, w1)):
        a, b = a.double(), b.double()
        # (adding to O(1) values rounds each sum to 2^-24 of them)
        slack = 2e-6 * b.norm(dim=1) + (1.2e-7 * 4 * d ** 0.5 if accumulate and a.shape[0] == V else 1e-30)
        assert bool(((a - b).norm(dim=1) <= slack).all())
