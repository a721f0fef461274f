"""Tables of up to 512 symbols, which every encoder work-group builds for itself: who takes the surplus, who pays the deficit,
on both sides of one symbol a thread, byte by byte against the CPU oracle.  Needs an MI355X (-m gpu)."""
import pytest
import torch

import oracle
from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


def _tensor(kind, levels, n, seed):
    g = torch.Generator().manual_seed(seed)
    if kind == "flat":        # equal counts: ties everywhere
        x = torch.arange(n) % levels
    elif kind == "steep":     # one very frequent symbol, the others rare
        x = torch.randint(0, levels, (n,), generator=g) * (torch.rand(n, generator=g) < 0.05)
    elif kind == "steps":     # frequencies 1, 2, 4, ... : several pay
        x = torch.clamp((torch.rand(n, generator=g).log2() * -levels / 16).floor(), 0, levels - 1)
    else:                     # "few": all levels once or twice, two symbols share the rest
        x = torch.where(torch.arange(n) < 2 * levels, torch.arange(n) % levels, 1 + (torch.arange(n) & 1))
    x = x.float()
    x[0], x[1] = 0.0, float(levels - 1)
    return x[torch.randperm(n, generator=g)]


def _compare(x, q, m, cols, s, cs, kernel, launched_kernels):
    n, mode = x.numel(), B.MODE_CSR if cols else B.MODE_DENSE
    print(f"[case] Q={q} K={cols} M={m} S={s} n={n}", flush=True)
    codec = B.Codec(B.make_params(q, m, n // (cols or n), cols or n, mode, s, cs, B.F32), n)
    xd = x.cuda()
    assert {"k_encode", "k_encode_feed"} & launched_kernels(lambda: codec.compress(xd, check=False)) == {kernel}
    status = B.rans_last_status(codec.ws)
    try:
        ref, _ = oracle.compress(x.numpy(), oracle.make_params(q, m, n // (cols or n), cols or n, mode, s, cs, 0))
    except oracle.OracleError as e:
        assert status == e.code and int(codec.nbytes.item()) == 0
        return
    assert status == 0 and codec.container(int(codec.nbytes.item())) == ref


# M from the fewest slots the present symbols fit up; 2^6 slots are too few for most of the 8-bit tensors
@pytest.mark.parametrize("kind", ["flat", "steep", "steps", "few"])
@pytest.mark.parametrize("q,cols", [(1, 0), (3, 0), (8, 0), (6, 63), (8, 255), (8, 256), (8, 301), (8, 511)])
def test_small_tables(kind, q, cols, launched_kernels):
    x = _tensor(kind, 1 << q, (cols or 97) * 41, q + cols)
    other = "k_encode" if cols else "k_encode_feed"
    for m in (6, 8, 9, 10, 12, 15):
        for s, cs, kernel in ((64, 64 * 40, "k_encode_feed"), (300, 0, other), (1088, 0, "k_encode")):
            _compare(x, q, m, cols, s, cs, kernel, launched_kernels)


# k_encode on dense chunks long enough for the lines that it requests beside the table build (16 and 32 rows), ragged at the end
@pytest.mark.parametrize("kind", ["flat", "steep", "steps", "few"])
@pytest.mark.parametrize("s,rows,chunks", [(1088, 11, 3), (4096, 31, 4), (4096, 33, 4), (64, 40, 513)])
def test_small_tables_beside_touched_lines(kind, s, rows, chunks, launched_kernels):
    x = _tensor(kind, 256, s * rows * chunks - 5, rows)
    for m in (8, 9, 12):
        _compare(x, 8, m, 0, s, s * rows, "k_encode", launched_kernels)
