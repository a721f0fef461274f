"""Symbols at and around the rounding boundaries of Eq. 6, to the last bit those of the oracle.  fp16 vectors in dense mode
take a shorter way where the rounded value is certain, the exact one elsewhere and, in a wave that meets many doubtful
values, from the next tile on; everything else takes the exact way throughout."""
import numpy as np
import pytest
import torch

from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


def _values(lo, hi, Q, n, seed):
    """Values whose x / s + z lies on a half-integer, up to 40 units of the last place (or 2^-14 ... 2^-10 steps) off it."""
    rng = np.random.default_rng(seed)
    lo, hi = np.float32(lo), np.float32(hi)
    s = np.float32(hi - lo) / np.float32(2 ** Q - 1)
    z = np.float64(np.rint(np.float32(-lo / s)))
    k = rng.integers(-1, 2 ** Q + 1, n) + 0.5
    x = ((k - z) * np.float64(s) + np.where(rng.random(n) < 0.5, 0.0, rng.choice([-1, 1], n) * 2.0 ** -rng.uniform(10, 14, n)) * s)
    x = x.astype(np.float32)
    x = (x.view(np.int32) + rng.integers(-40, 41, n).astype(np.int32)).view(np.float32)
    x = np.clip(np.nan_to_num(x, nan=0.0, posinf=0.0, neginf=0.0), lo, hi).astype(np.float32)
    x[0], x[-1] = lo, hi
    return x


@pytest.mark.parametrize("lo,hi", [(-1.0, 1.0), (0.0, 3.7), (-92.0, 87.3), (-5.1, 0.0), (1e-6, 2.3e-6), (100.0, 101.0),
                                   (0.4999, 128.0), (-3e8, 2e8), (-1e-9, 1e-9), (255.0, 511.0), (256.5, 511.5)])
@pytest.mark.parametrize("Q,dtype,mode", [(8, "fp32", "dense"), (6, "fp32", "csr"), (8, "fp16", "csr"), (3, "fp16", "dense"), (8, "fp16", "dense"), (6, "fp16", "dense")])
@pytest.mark.parametrize("n", [4096 * 4 + 7, 1 << 20])
def test_symbols_at_the_halves(oracle, lo, hi, Q, dtype, mode, n):
    x = _values(lo, hi, Q, n, 5)
    if dtype == "fp16":
        with np.errstate(over="ignore"):
            x = x.astype(np.float16)
        if not np.isfinite(x).all() or x.max() == x.min():
            pytest.skip("outside binary16")
    print(f"[case] halves [{lo}, {hi}] Q={Q} {dtype} {mode} n={n}", flush=True)
    p = B.make_params(Q, 12, n, 1, B.MODE_CSR if mode == "csr" else B.MODE_DENSE, 64, 4096, B.F16 if dtype == "fp16" else B.F32)
    codec = B.Codec(p, n)
    sym = torch.empty(n, dtype=torch.uint8, device="cuda")
    codec.quantize(torch.from_numpy(x).cuda(), sym)
    want, _ = oracle.quantize(x, Q)
    assert np.array_equal(sym.cpu().numpy(), np.asarray(want, np.uint8))


# scales that put the few values of binary16 on halves, so that waves change to the exact way: after one tile of many,
# in tensors that end inside a tile and inside a vector
@pytest.mark.parametrize("top", [255 / 64, 255 / 32, 4.98046875, 5.1])
@pytest.mark.parametrize("n", [256 * 32768 * 2 + 32768 * 3 + 8 * 1000 + 5, 32768 * 300 + 4099])
def test_many_values_on_halves(oracle, top, n):
    print(f"[case] on halves top={top} n={n}", flush=True)
    x = torch.randn(n, generator=torch.Generator().manual_seed(n % 1000)).abs().clamp_(max=top).to(torch.float16)
    x[0], x[1] = top, 0
    p = B.make_params(8, 12, n, 1, B.MODE_DENSE, 1024, 1 << 18, B.F16)
    codec = B.Codec(p, n)
    sym = torch.empty(n, dtype=torch.uint8, device="cuda")
    codec.quantize(x.cuda(), sym)
    want, _ = oracle.quantize(x.numpy(), 8)
    assert np.array_equal(sym.cpu().numpy(), np.asarray(want, np.uint8))
