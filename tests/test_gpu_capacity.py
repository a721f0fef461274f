"""A container that does not fit in a call with more work-groups than are resident at once: the groups that start after an early
one has found out leave at their start, and the size still has to say 0.  Needs an MI355X (-m gpu)."""
import pytest
import torch

import oracle
from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


# encoder, elements, row length, mode, streams, chunk: work-groups of the encoder that places its words itself (building its
# table, and with k_normalize's), of the fed one likewise, and of the gather kernel behind grids above 16384
@pytest.mark.parametrize("kernel,n,cols,mode,s,chunk", [
    ("k_encode", 8192 * 1024, 1024, B.MODE_DENSE, 256, 1024),
    ("k_encode", 3 << 20, 64, B.MODE_CSR, 256, 1024),
    ("k_encode", 3 << 20, 1024, B.MODE_CSR, 256, 1024),
    ("k_encode_feed", 6000000, 16, B.MODE_CSR, 64, 64 * 256),
    ("k_encode_feed", 6000000, 750, B.MODE_CSR, 64, 64 * 256),
    ("k_gather", 66 * 65536, 65536, B.MODE_DENSE, 65536, 65536)])
def test_size_is_zero_when_later_groups_find_the_error(kernel, n, cols, mode, s, chunk, launched_kernels):
    g = torch.Generator().manual_seed(n + cols)
    x = torch.randint(1, 256, (n,), generator=g).float()  # no zeros but one: D is as long as the grid is sized for
    x[0] = 0
    p = B.make_params(8, 12, n // cols, cols, mode, s, chunk, B.F32)
    codec = B.Codec(p, n)
    xd = x.cuda()
    sizes = [codec.nbytes]  # the one behind it lies in pinned host memory, which the call may write too
    sizes.append(torch.empty(1, dtype=torch.int64, pin_memory=True))
    alphabet = max(256, cols + 1) if mode == B.MODE_CSR else 256
    chunks = -(-(2 * n + n // cols if mode == B.MODE_CSR else n) // chunk)
    room = 128 + 2 * alphabet + 8 * (chunks + 1) + 3 * 10 * s  # header, table, directory, and a few chunks at most
    small = codec.stream[:room]
    for size in sizes:
        for _ in range(3):
            size.fill_(0x7777)
            print(f"[case] {kernel} n={n} K={cols} mode={mode} S={s} room={room}", flush=True)
            names = launched_kernels(lambda: B.rans_compress(xd, n, p, small, size, codec.ws))
            assert kernel in names
            assert B.rans_last_status(codec.ws) == B.ERR_CAPACITY
            assert int(size.item()) == 0
    ref, _ = oracle.compress(x.numpy(), oracle.make_params(8, 12, n // cols, cols, mode, s, chunk, 0))
    assert codec.container(codec.compress(xd)) == ref
