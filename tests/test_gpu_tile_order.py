"""The longest-first tile order at the edges of a work-group's round: every
tile once, list lengths falling by powers of two."""
import numpy as np
import pytest

from _gpu_helpers import say

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["empty", "same", "mixed"])
@pytest.mark.parametrize("n", [1, 63, 64, 1023, 1025, 8191, 8192, 8193, 16384, 16385, 70000])
def test_tile_order(gpu, n, kind):
    from paper_2509_12138_amd import _lib
    from paper_2509_12138_amd.ops import _ptr, call, stream_handle
    say("tile order", n, kind)
    rng = np.random.default_rng(n)
    lens = {"empty": np.zeros(n, np.int64), "same": np.full(n, 37),
            "mixed": (2.0 ** rng.uniform(0, 15, n)).astype(np.int64) * rng.integers(0, 2, n)}[kind]
    end = np.cumsum(lens)
    ranges = torch.as_tensor(np.stack([end - lens, end], 1).astype(np.uint32).view(np.int32)).cuda()
    order = torch.full((n + 1,), -7, dtype=torch.int32, device="cuda")
    ws = torch.zeros(_lib.load().gs_tile_order_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    call("gs_tile_order", _ptr(ranges), n, _ptr(ws), ws.numel(), _ptr(order), stream_handle())
    got = order.cpu().numpy()
    assert got[n] == -7
    np.testing.assert_array_equal(np.sort(got[:n]), np.arange(n))
    bucket = np.floor(np.log2(lens[got[:n]] + 1.0))
    assert np.all(np.diff(bucket) <= 0)
