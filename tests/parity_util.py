"""Helpers shared by the GPU parity tests: run the oracle on a workload and compare."""
import os

import numpy as np

from oracle import cutoffs as ocut
from oracle import ppo_head as ohead
from paper_2606_29758_amd import synth

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")

# Tolerances for bf16 inputs with fp32 accumulation (the loss is reduced in fp64).
LOSS_RTOL = 1e-4
GRAD_REL_L2 = 1e-2
LOGP_ATOL = 2e-4


def f32(x):
    """The float32 value the kernels see for a scalar parameter, as a float64."""
    return float(np.float32(x))


def oracle_logp_old(wl):
    """logp_old = logp_new + noise with logp_new from the float64 oracle (small workloads)."""
    return (ohead.target_logprob(wl.hidden_bits, wl.w_bits, wl.target_full) + wl.lp_noise).astype(np.float32)


def logp_old_for(wl):
    try:
        return synth.load_stored_logp_old(wl, GOLDEN)
    except FileNotFoundError:
        if wl.total_tokens * wl.cfg.V * wl.cfg.d > 5e12:
            raise
        return oracle_logp_old(wl)


def oracle_sample_pack(wl, logp_old_full, seed, offset=0):
    cfg = wl.cfg
    H = ocut.sample_cutoffs(wl.xi, wl.xi_off, wl.lengths, cfg.P, cfg.K, seed, offset)
    pk = ocut.pack_prefixes(H, wl.lengths, wl.xi, wl.xi_off, cfg.P, cfg.K, wl.target_full, logp_old_full)
    return H, pk


def oracle_loss(wl, pk, advantage=None, want_grads=True):
    cfg = wl.cfg
    adv = wl.advantage if advantage is None else advantage
    return ohead.loss_fwd_bwd(wl.hidden_bits[pk["src_row"]], wl.w_bits, pk["target"], pk["logp_old"],
                              pk["weight"], pk["seq_id"], adv, f32(cfg.eps_low), f32(cfg.eps_high),
                              f32(cfg.loss_scale), want_grads=want_grads)


def rel_l2(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / nb if nb > 0 else np.linalg.norm(a)


def ambiguous_clip(ref, eps_low, eps_high, band=1e-5):
    """Tokens whose ratio sits so close to a clip bound that float32 and float64 may disagree."""
    rho = ref["rho"]
    return (np.abs(rho - (1 + f32(eps_high))) < band) | (np.abs(rho - (1 - f32(eps_low))) < band)


def loss_in(workspace_bytes, hidden, w_head, target, logp_old, weight, seq_id, advantage, N, eps_low, eps_high,
            loss_scale, flags=0, d_w_head=None, want_logp=True):
    """pspo_loss_fwd_bwd in a workspace of the given size, straight through the library: the
    binding asks for the full size, the library also takes the smaller one of the chunked plan.
    Returns the outputs and the vocabulary chunks that the backward ran in."""
    import torch

    from paper_2606_29758_amd import pspo
    V, d = w_head.shape
    new = lambda shape, dt=torch.float32: torch.empty(shape, dtype=dt, device="cuda")   # noqa: E731
    out = dict(loss=new(1, torch.float64), d_hidden=new((N, d)), d_w_head=new((V, d)) if d_w_head is None else d_w_head,
               logp_new=new(N) if want_logp else None, stats=new(5, torch.float64))
    ws = new(workspace_bytes, torch.uint8)
    lib, ptr = pspo.load(), (lambda x: None if x is None else x.data_ptr())
    pspo.timing_start(256)
    rc = lib.pspo_loss_fwd_bwd(*[ptr(x) for x in (hidden, w_head, target, logp_old, weight, seq_id, advantage)], N, d, V,
                               advantage.shape[0], eps_low, eps_high, loss_scale, flags, ptr(out["loss"]),
                               ptr(out["d_hidden"]), ptr(out["d_w_head"]), ptr(out["logp_new"]), ptr(out["stats"]), None,
                               ptr(ws), workspace_bytes, torch.cuda.current_stream().cuda_stream)
    chunks = pspo.timing_stop()["logit_grad"]["count"]
    assert rc == 0, lib.pspo_last_error()
    torch.cuda.synchronize()
    return out, chunks


def loss_chunked(step, pk, N, want_logp=True):
    """A loss call of few tokens without the room for one vocabulary chunk: the chunked backward."""
    from paper_2606_29758_amd import pspo
    dw = step.dw
    size = pspo.loss_workspace_bytes(N, dw.d, dw.V, 0) - 256
    return loss_in(size, pk["hidden"], dw.w_head, pk["target"], pk["logp_old"], pk["weight"], pk["seq_id"], dw.advantage,
                   N, dw.eps_low, dw.eps_high, dw.loss_scale, want_logp=want_logp)
