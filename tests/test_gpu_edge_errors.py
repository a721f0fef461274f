"""The edge side as one call reports a tensor that cannot be quantised, although it waits for no status before its end."""
import pytest
import torch

from paper_2511_11664_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_edge_side_refuses_non_finite_values(value):
    x = torch.rand(128 * 784, device="cuda")
    x[777] = value
    with pytest.raises(B.RansError) as e:
        B.compress_with_search(x, 8, 12, 64, 4096)
    assert e.value.code == -6
    x[777] = 0.5
    stream, p, _ = B.compress_with_search(x, 8, 12, 64, 4096)
    assert stream.numel() > 0 and p.rows * p.cols == x.numel()
