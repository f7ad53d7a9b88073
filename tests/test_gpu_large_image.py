"""GPU parity of a weight whose dense operand image passes 2 GiB while its 4:2
image, the one with a limit, does not (524,404 x 4096: 32 windows x 32,776
channel tiles, 2.00 and 1.06 GiB), on every kernel and both input layouts,
through the C ABI: stored blocks in the first and the last windows and tiles,
the last of them ragged. Bars as in test_gpu_parity.py (int32: bit-exact).
"""
import numpy as np
import pytest

import oracle
from test_gpu_parity import say

pytestmark = pytest.mark.gpu

T = 1  # SL_LAYOUT_T16X32
N, K, M = 16 * 32775 + 4, 4096, 130


@pytest.fixture(scope="module")
def big(hip):
    rng = np.random.default_rng(21)
    w = np.zeros((N // 4, 4, K), np.int8)
    g = np.arange(N // 4)
    # 24 blocks a block-row anywhere, one in the first and two in the last window
    for lo, hi, blocks in ((0, K, 24), (0, 128, 1), (K - 128, K, 2)):
        for _ in range(blocks):
            w[g, :, rng.integers(lo, hi, N // 4)] = rng.integers(1, 128, (N // 4, 4), dtype=np.int8)
    w = w.reshape(N, K)
    pw = hip.PackedWeight.pack(w, np.full(N, 0.01, np.float32))
    x = rng.integers(-127, 128, (M, K), dtype=np.int8)
    # channels of the first, the last and some other tiles
    tiles = np.concatenate([[0, 1, 32774, 32775], rng.integers(2, 32774, 200)])
    sel = np.unique((tiles[:, None] * 16 + np.arange(16)).ravel())
    sel = sel[sel < N]
    yield pw, x, sel, oracle.acc(x, np.ascontiguousarray(w[sel]))
    pw.free()


@pytest.mark.parametrize("path", ["", "split", "panel", "tile", "direct", "staged"])
def test_dense_image_over_2_gib(hip, big, monkeypatch, path):
    import torch
    pw, x, sel, ref = big
    if path:
        monkeypatch.setenv("SL_PATH", path)
    for xl in (0, T):
        if path == "staged" and xl == T:
            continue
        xd = torch.from_numpy(np.ascontiguousarray(hip.to_t16x32(x, fill=3)) if xl == T else x).cuda()
        say(f"dense image over 2 GiB path={path} x_layout={xl}")
        y = pw.run(xd, 0.02, 0, x_layout=xl, m_tokens=M)
        torch.cuda.synchronize()
        assert hip.last_path().startswith(path), hip.last_path()
        got = y[:, torch.from_numpy(sel).cuda()].cpu().numpy()
        assert np.array_equal(got, ref), f"{path} {hip.last_path()} x_layout={xl}"
        del y
    torch.cuda.empty_cache()
