"""GPU: the gather of the kept hidden rows on both sides of its line (the capacity's rows read and
written past 160 MB, in rows of more than 64 16-byte pieces), with rows that end inside a round of
8 x 64 pieces, completions that keep nothing, everything, or a prefix, and a capacity at, below and
above the kept count.
The bytes are those of the rows.
"""
import numpy as np
import pytest
import torch

from paper_2606_29758_amd import pspo

pytestmark = pytest.mark.gpu

# d, kept rows: 81,920 rows of 64 pieces would be 160 MB; 10,922 of 480 pieces just are not, 10,923 are
CASES = [(8, 5000), (512, 90000), (520, 80000), (520, 81000), (3592, 2000), (3592, 13000), (3840, 10922), (3840, 10923), (4104, 11000)]


@pytest.mark.parametrize("d,kept", CASES)
@pytest.mark.parametrize("short", [0, 7, -30000])   # capacity against the kept rows
def test_rows(d, kept, short):
    print(f"[pack rows] d={d} kept={kept} capacity short by {short}", flush=True)
    rng = np.random.default_rng(d + kept)
    lengths = np.array([kept // 2, 40, 0, kept - kept // 2 + 300, 17], dtype=np.int32)
    cut = np.array([kept // 2, 0, 0, kept - kept // 2 - 5, 5], dtype=np.int32)
    T = int(lengths.max())
    t = lambda a, dt: torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dt)   # noqa: E731
    S = int(lengths.sum())
    full = torch.from_numpy(rng.integers(0, 2 ** 16, (4096, d)).astype(np.uint16).view(np.int16)).to("cuda")
    full = full[torch.arange(S, device="cuda") * 2654435761 % 4096].view(torch.bfloat16)
    out = pspo.pack_prefixes(t(cut, torch.int32), t(lengths, torch.int32), torch.ones(T, dtype=torch.float64, device="cuda"),
                             t([0, T], torch.int64), 1, 5, kept - short, hidden_full=full)
    n = min(kept, kept - short)
    rows = np.concatenate([f + np.arange(c) for f, c in zip(np.concatenate([[0], np.cumsum(lengths)]), cut)])[:n]
    assert int(out["n_tokens"].item()) == n
    assert torch.equal(out["hidden"].view(torch.int16)[:n], full.view(torch.int16)[t(rows, torch.int64)])
