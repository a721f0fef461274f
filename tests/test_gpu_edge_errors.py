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


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("search_fails", [False, True])
def test_a_refused_tensor_leaves_no_error_behind(value, search_fails, monkeypatch):
    """The workspaces of a refused call hold no unread error when they are given back: a later call may get that memory."""
    used = []

    def noting(name, at):
        entry = getattr(B, name)
        monkeypatch.setattr(B, name, lambda *a: (used.append(a[at]), entry(*a))[1])
    noting("rans_quantize", 5)
    noting("rans_encode", 6)
    if search_fails:
        monkeypatch.setattr(B, "rans_search_reshape", lambda *a: B.ERR_HIP)
    x = torch.rand(128 * 784, device="cuda")
    x[5] = value
    with pytest.raises(B.RansError):
        B.compress_with_search(x, 8, 12, 64, 4096)
    assert len(used) == (1 if search_fails else 2)
    assert [B.rans_last_status(ws) for ws in used] == [0] * len(used)
