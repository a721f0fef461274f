"""Which form of a kernel a call takes on the two sides of the lines between them, from the launches the library
records, and the containers at those sizes byte by byte against the CPU oracle.  Needs an MI355X (-m gpu)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


def _launched(call):
    """Names of the kernels `call` launches."""
    B.rans_profile_reset()
    B.rans_profile_enable("all")
    try:
        call()
        torch.cuda.synchronize()
        return set(B.rans_profile_read())
    finally:
        B.rans_profile_enable(None)
        B.rans_profile_reset()


def _relu(n, zeros, seed=7):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(n, generator=g).abs() + 0.01
    x *= torch.rand(n, generator=g) >= zeros
    x[0] = 0
    return x


# streams, symbols of a stream in a chunk, coding waves of 64 streams; the fed coder pays for long streams and while its
# work-groups find room: a compute unit holds two of them
@pytest.mark.parametrize("s,rows,waves,fed", [
    (64, 3, 64, False), (64, 4, 64, True), (64, 4, 256, True), (16, 23, 64, False), (16, 24, 64, True), (4096, 11, 128, False),
    (4096, 12, 128, True), (4096, 32, 256, False), (4096, 48, 256, True), (64, 24, 288, True), (64, 23, 288, False),
    (256, 64, 288, False), (256, 96, 288, True), (1024, 128, 320, False), (1024, 192, 320, True),
    (64, 24, 512, True), (64, 23, 512, False), (32, 48, 512, True), (32, 47, 512, False), (256, 128, 512, True),
    (256, 96, 512, False), (64, 128, 513, False)])
def test_dense_encoder_form(s, rows, waves, fed):
    n = waves // -(-s // 64) * s * rows
    print(f"[case] dense S={s} rows={rows} waves={waves} n={n}", flush=True)
    x = _relu(n, 0.0)
    codec = B.Codec(B.make_params(8, 12, n, 1, B.MODE_DENSE, s, s * rows, B.F32), n)
    xd = x.cuda()
    names = _launched(lambda: codec.compress(xd))
    assert ("k_encode_feed" in names) == fed and ("k_encode" in names) != fed
    ref, _ = oracle.compress(x.numpy(), oracle.make_params(8, 12, n, 1, B.MODE_DENSE, s, s * rows, 0))
    assert codec.container(int(codec.nbytes.item())) == ref


# CSR, where D may be as long as the grid is sized for: 2 n + rows symbols without zeros
@pytest.mark.parametrize("zeros", [0.0, 0.3, 0.7])
@pytest.mark.parametrize("s,rows,waves,cols,fed", [
    (64, 64, 256, 4, True), (64, 64, 288, 16, True), (64, 64, 600, 4, False), (64, 64, 768, 64, False), (1024, 64, 512, 64, False),
    (256, 128, 288, 300, True), (256, 128, 288, 1500, False), (64, 256, 288, 1500, True), (64, 32, 700, 6000, False),
    (16, 256, 768, 16, True), (16, 256, 769, 16, False)])
def test_csr_encoder_form(s, rows, waves, cols, fed, zeros):
    chunk = s * rows
    n = int(waves // -(-s // 64) * chunk / (2 + 1 / cols)) // cols * cols
    print(f"[case] csr S={s} rows={rows} waves={waves} K={cols} zeros={zeros} n={n}", flush=True)
    x = _relu(n, zeros)
    codec = B.Codec(B.make_params(8, 13, n // cols, cols, B.MODE_CSR, s, chunk, B.F32), n)
    xd = x.cuda()
    names = _launched(lambda: codec.compress(xd))
    assert ("k_encode_feed" in names) == fed and ("k_encode" in names) != fed
    ref, _ = oracle.compress(x.numpy(), oracle.make_params(8, 13, n // cols, cols, B.MODE_CSR, s, chunk, 0))
    assert codec.container(int(codec.nbytes.item())) == ref


# streams, symbols of a stream, chunks: the form with the short chain is for streams that outlast its refill, while all its
# work-groups are resident (with a 32 KB table and 64 streams three on a compute unit), and not
# for a few lanes in many work-groups
@pytest.mark.parametrize("s,rows,chunks,lean", [
    (64, 31, 20, False), (64, 32, 20, True), (256, 24, 100, False), (256, 64, 100, True), (64, 64, 768, True), (64, 64, 769, False),
    (1, 64, 512, True), (8, 40, 600, False), (9, 40, 600, True), (1, 200, 700, False)])
def test_decoder_form(s, rows, chunks, lean):
    n = s * rows * chunks
    print(f"[case] decode S={s} rows={rows} chunks={chunks} n={n}", flush=True)
    x = _relu(n, 0.3)
    p = B.make_params(8, 12, n, 1, B.MODE_DENSE, s, s * rows, B.F32)
    codec = B.Codec(p, n)
    nbytes = codec.compress(x.cuda())
    hdr = codec.header(nbytes)
    out = torch.empty(n, dtype=torch.float32, device="cuda")
    names = _launched(lambda: codec.decompress(nbytes, hdr, out))
    assert ("k_decode_lean" in names) == lean and ("k_decode" in names) != lean
    _, _, y = oracle.decompress(codec.container(nbytes))
    assert np.array_equal(out.cpu().numpy().view(np.uint32), np.asarray(y, np.float32).view(np.uint32))
