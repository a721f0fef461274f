"""CSR decode around the line below which the expand kernel adds up the row counts itself (32768 rows, 256 tiles), and
the symbols' way back to floats at sizes that are no multiple of its vectors."""
import numpy as np
import pytest
import torch

from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(1, 5), (7, 3), (9, 513), (2047, 1), (2048, 2), (32767, 4), (32768, 4), (32769, 4), (32768, 16),
                                       (32764, 17), (8200, 64), (2056, 255), (513, 1024)])
@pytest.mark.parametrize("out", [torch.float32, torch.float16])
def test_csr_round_trip(oracle, rows, cols, out):
    n = rows * cols
    print(f"[case] expand {rows} x {cols} {out}", flush=True)
    rng = np.random.default_rng(n)
    x = (rng.standard_normal(n).clip(0) * (rng.random(n) < 0.8)).astype(np.float32)
    x[: n // 3] = 0  # a long stretch of empty rows
    x[n - 1] = 2.5
    p = B.make_params(8, 12, rows, cols, B.MODE_CSR, 64, 4096, B.F32)
    codec = B.Codec(p, n)
    nbytes = codec.compress(torch.from_numpy(x).cuda())
    hdr = codec.header(nbytes)
    want, _ = oracle.quantize(x, 8)
    sym = torch.empty(n, dtype=torch.uint8, device="cuda")
    codec.decode(nbytes, hdr, sym)
    assert np.array_equal(sym.cpu().numpy(), np.asarray(want, np.uint8))
    y = torch.empty(n, dtype=out, device="cuda")
    codec.decompress(nbytes, hdr, y)
    z = torch.empty(n, dtype=out, device="cuda")
    B.rans_dequantize(sym, n, codec.qinfo, B.F16 if out == torch.float16 else B.F32, z)
    _, _, ref = oracle.decompress(codec.container(nbytes))
    ref = torch.from_numpy(np.asarray(ref, np.float32)).to(out)
    assert torch.equal(y.cpu(), ref) and torch.equal(z.cpu(), ref)
