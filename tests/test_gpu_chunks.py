"""GPU: the chunked backward against the float64 oracle, just past the 768 tokens up to which one chunk
serves and beyond, where the vocabulary splits unevenly (d = 4096: 16 row tiles of 384 a chunk before the
split is evened out; 13,401 rows are chunks of 18 and 17 tiles, 14,101 of 13, 13 and 11), each with a
partial last tile; with every flag of the call.

Every row is compared.  A d_w_head row is the float32 target entries plus bf16-rounded other entries
(2^-9 relative each at most, over hidden rows of independent directions), so it is off by less than 2^-8
of its other part; d_hidden rows likewise: GRAD_REL_L2 (1e-2) of the row covers both.  Kept logits are
rounded to fp16 offsets, which moves an entry by less than its bf16 rounding.  Added to O(1) values, a row's
sum is rounded to 2^-24 of them.
"""
import numpy as np
import pytest
import torch

from oracle import ppo_head as ohead
from paper_2606_29758_amd import pspo, synth

from parity_util import GRAD_REL_L2, LOGP_ATOL, LOSS_RTOL, f32, loss_in

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,V,chunks", [(769, 13401, 2), (900, 14101, 3), (1537, 13401, 2)])
def test_uneven_chunks(N, V, chunks):
    d, R = 4096, 5
    rng = np.random.default_rng(N)
    h = synth.round_to_bf16_bits(rng.normal(0.0, 1.0, (N, d)).astype(np.float32))
    W = synth.round_to_bf16_bits(rng.normal(0.0, 0.02, (V, d)).astype(np.float32))
    tgt = rng.integers(0, V, N).astype(np.int32)
    tgt[:4] = (0, V - 1, V - 384, V // 2)
    seq = np.sort(rng.integers(0, R, N)).astype(np.int32)
    adv = np.array([1.0, -1.0, 0.0, 0.5, -0.7], dtype=np.float32)
    weight = (1.0 + rng.random(N)).astype(np.float32)
    lp_old = (ohead.target_logprob(h, W, tgt) + rng.normal(0.0, 0.05, N)).astype(np.float32)
    ref = ohead.loss_fwd_bwd(h, W, tgt, lp_old, weight, seq, adv, f32(0.9), f32(0.9), f32(0.25))
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dt)   # noqa: E731
    bits = lambda b: torch.from_numpy(b.view(np.int16)).to("cuda").view(torch.bfloat16)       # noqa: E731
    args = (bits(h), bits(W), t(tgt, torch.int32), t(lp_old, torch.float32), t(weight, torch.float32),
            t(seq, torch.int32), t(adv, torch.float32), N, 0.9, 0.9, 0.25)
    start = torch.randn((V, d), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    for flags in (0, pspo.PSPO_ACCUMULATE_DW, pspo.PSPO_KEEP_LOGITS, pspo.PSPO_ACCUMULATE_DW | pspo.PSPO_KEEP_LOGITS):
        print(f"[chunks] N={N} V={V} flags={flags}", flush=True)
        add = bool(flags & pspo.PSPO_ACCUMULATE_DW)
        out, ran = loss_in(pspo.loss_workspace_bytes(N, d, V, flags), *args, flags=flags, d_w_head=start.clone())
        assert ran == chunks
        assert abs(float(out["loss"].item()) - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
        assert np.max(np.abs(out["logp_new"].double().cpu().numpy() - ref["logp_new"])) <= LOGP_ATOL
        dw = (out["d_w_head"].double() - start.double() if add else out["d_w_head"].double()).cpu().numpy()
        for got, want, slack in ((out["d_hidden"].double().cpu().numpy(), ref["d_hidden"], 0.0),
                                 (dw, ref["d_w"], 2.0 ** -24 * 4 * d ** 0.5 if add else 0.0)):
            off = np.linalg.norm(got - want, axis=1)
            bound = GRAD_REL_L2 * np.linalg.norm(want, axis=1) + slack
            assert np.all(off <= bound), (int(np.argmax(off - bound)), off.max())
