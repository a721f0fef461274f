"""Containers of few streams (the encoder form with one coding wave per work-group) and tables of large alphabets,
byte by byte against the CPU oracle.  Needs an MI355X (-m gpu)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


def _compare(x, q, m, mode, cols, s, cs, dtype=0):
    n = x.numel()
    p = B.make_params(q, m, n // cols, cols, mode, s, cs, dtype)
    print(f"[case] n={n} Q={q} M={m} mode={mode} K={cols} S={s} cs={cs}", flush=True)
    ref, _ = oracle.compress(x.numpy(), oracle.make_params(q, m, n // cols, cols, mode, s, cs, dtype))
    codec = B.Codec(p, n)
    nbytes = codec.compress(x.cuda())
    assert codec.container(nbytes) == ref
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    codec.decompress(nbytes, codec.header(nbytes), out)
    _, _, y = oracle.decompress(ref)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), np.asarray(y, np.float32).view(np.uint32))


def _relu(n, seed):
    return torch.relu(torch.randn(n, generator=torch.Generator().manual_seed(seed)))


# tiles of 24 rows, 8 of them per feeding wave: row counts around both, with and without a ragged last row
@pytest.mark.parametrize("rows", [1, 7, 8, 9, 23, 24, 25, 47, 48, 49, 72, 73])
@pytest.mark.parametrize("s,rem", [(64, 0), (33, 1), (70, 69)])
def test_tile_edges(rows, s, rem):
    n = rows * s + rem
    _compare(_relu(n, rows), 8, 12, B.MODE_DENSE, n, s, 0)
    if n % 5 == 0:
        _compare(_relu(n, rows), 6, 12, B.MODE_CSR, 5, s, 0)


# dense chunks of four to ten tiles: the feeding waves request two tiles at a time, four make a turn
@pytest.mark.parametrize("rows", [95, 96, 97, 119, 120, 121, 144, 145, 168, 169, 192, 193, 217])
@pytest.mark.parametrize("s,rem,cs", [(64, 0, 0), (33, 1, 0), (70, 69, 70 * 96)])
def test_turns_of_four_tiles(rows, s, rem, cs):
    n = rows * s + rem
    _compare(_relu(n, rows), 8, 12, B.MODE_DENSE, n, s, cs)


# word areas that run full again and again, one stream, and chunks whose last one is short
@pytest.mark.parametrize("n,q,m,mode,cols,s,cs", [
    (30011, 8, 12, 0, 1, 3, 0), (30011, 8, 14, 0, 1, 1, 0), (50000, 8, 12, 1, 50, 2, 0), (40000, 8, 12, 1, 8, 64, 64 * 300),
    (40000, 8, 12, 0, 8, 64, 64 * 300), (24000, 4, 5, 0, 4, 16, 0), (24000, 2, 7, 1, 100, 16, 16 * 25)])
def test_long_streams_and_short_tables(n, q, m, mode, cols, s, cs):
    _compare(_relu(n, n), q, m, mode, cols, s, cs)


def test_table_with_inexact_multipliers():
    x = torch.zeros(20000)
    x[::37] = _relu(len(x[::37]), 5) + 0.1  # one symbol above half of the table
    for m in (11, 12, 13, 14, 15):
        _compare(x, 8, m, B.MODE_DENSE, 1, 48, 0)


# alphabets on both sides of 513, 4096 (table in registers), 5120 (entries in LDS) and 8192; few counts in a small
# table, so that nearly every symbol is raised to 1 and the frequent ones pay
@pytest.mark.parametrize("cols,m", [(511, 10), (512, 10), (3000, 12), (4094, 12), (4096, 13), (5119, 13), (5120, 13), (8190, 13), (8192, 14)])
def test_large_alphabets(cols, m):
    n = cols * 12
    _compare(_relu(n, cols) * (torch.rand(n, generator=torch.Generator().manual_seed(1)) < 0.5), 8, m, B.MODE_CSR, cols, 32, 0)


# tables of 513 to 4096 symbols whose deficit one symbol pays, a few do, or all of the frequent ones, with ties among them
@pytest.mark.parametrize("cols,n_rows,m,keep", [(784, 4, 12, 0.05), (784, 5, 12, 0.5), (784, 40, 10, 0.5), (600, 3, 11, 0.02),
                                                (1023, 9, 11, 0.9), (2000, 30, 12, 0.3), (4000, 7, 12, 0.6)])
@pytest.mark.parametrize("levels", [2, 200])
def test_who_pays_the_deficit(cols, n_rows, m, keep, levels):
    n = cols * n_rows
    g = torch.Generator().manual_seed(n + levels)
    x = (torch.randint(1, levels, (n,), generator=g).float() * (torch.rand(n, generator=g) < keep)) if levels > 2 else (torch.rand(n, generator=g) < keep).float()
    x[0], x[1] = 0.0, float(levels - 1)
    _compare(x, 8, m, B.MODE_CSR, cols, 64, 64 * 16)
