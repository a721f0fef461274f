"""Reshape search where its mask pass, column counts and row counts change their shape: tensors that end inside a
word, a window or a piece, periods that are no multiple of 32, single divisors and many groups of them, several
copies of the histograms.  Checked against a count of every reshape with torch on the GPU (64-bit integers), costs in
binary64 on the host: the sums differ from the kernel's in the order of at most 513 terms and in log2's last bit,
513 * 2^-52 < 2e-13 relative."""
import math

import numpy as np
import pytest
import torch

from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


def _costs(sym: torch.Tensor, domain):
    T = sym.numel()
    nz = sym != 0
    hv = torch.bincount(sym[nz].long(), minlength=256)
    nnz = int(nz.sum())
    out = []
    for n in domain:
        K = T // n
        m = nz.view(n, K)
        d = torch.zeros(max(257, K + 1), dtype=torch.long, device=sym.device)
        d[:256] += hv
        d[:K] += m.sum(0)
        d[:K + 1] += torch.bincount(m.sum(1), minlength=K + 1)
        c = d.cpu().numpy().astype(np.float64)
        c = c[c > 0]
        p = c / (2 * nnz + n)
        out.append(float(-(2 * nnz + n) * np.sum(p * np.log2(p))))
    return out


@pytest.mark.parametrize("T,Q,density", [
    (31, 8, 0.5), (33, 8, 0.5), (4095, 8, 0.3), (4097, 8, 0.9), (8192 + 15, 6, 0.4), (3 * 331 * 32, 8, 0.4),
    (199 * 211 * 223, 8, 0.3),           # divisors without a common period, one group each
    (729 * 8191, 8, 0.5),                # odd: no row count by words, windows at every bit position
    (1012 * 32 * 61 + 32, 8, 0.3),       # just past whole pieces
    (240 * 251 * 169 * 2, 8, 0.35),      # many divisors, several groups
    (100003, 8, 0.5), (2 * 50021, 6, 0.1),  # K = 1 alone, and one beside it: no columns or rows to count, and hardly any
    (32 * 1024 * 17 * 31, 8, 0.97),         # counters of a column near the most their fields take
    (32 * 256 * 784 + 784 * 16, 8, 0.25), (5 * (1 << 20) - 4, 4, 0.05), (1 << 23, 8, 1.0),
])
def test_costs_at_the_edges(T, Q, density):
    print(f"[case] reshape edges T={T} Q={Q} d={density}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    sym = torch.randint(1, 1 << Q, (T,), device="cuda", generator=g, dtype=torch.uint8)
    sym *= torch.rand(T, device="cuda", generator=g) < density
    res = B.search_reshape(sym, Q)
    nmin = max(math.isqrt(T) + 1, -(-T // (1 << Q)))
    domain = [T // k for k in range(1, (1 << Q) + 1) if T % k == 0 and T // k >= nmin]
    assert list(res.cand_rows[:res.n_candidates]) == domain
    want = _costs(sym, domain)
    got = list(res.cand_cost[:res.n_candidates])
    assert got == pytest.approx(want, rel=2e-13, abs=1e-9)
    assert res.cost_bits == min(got[:res.n_evaluated]) and res.rows == domain[got.index(res.cost_bits)]
    stop = next((i + 1 for i in range(1, len(got)) if got[i] > got[i - 1]), len(got))
    assert res.n_evaluated == stop
    # unaligned symbols take the byte loads
    shifted = torch.empty(T + 1, dtype=torch.uint8, device="cuda")[1:]
    shifted.copy_(sym)
    again = B.search_reshape(shifted, Q)
    assert bytes(again) == bytes(res)
