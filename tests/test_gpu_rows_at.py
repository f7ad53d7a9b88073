"""GPU parity for token rows at any alignment, through the C ABI: row widths
that are no multiple of 4 or 16 and views of X that start at any byte, on the
split-reduction, weight-stationary and direct kernels (which load such rows
into registers, by whole words or by the words around them and a shift) and
on the staged kernel (which copies them byte by byte), with X ending where
its last row does. Bars as in test_gpu_parity.py.
"""
import numpy as np
import pytest

from test_gpu_panel import T, _refs
from test_gpu_parity import KINDS, _case, check, say

pytestmark = pytest.mark.gpu


def _view(torch, x, off):
    """A CUDA copy of x that starts `off` bytes into its allocation."""
    flat = torch.empty(x.size + off, dtype=torch.int8, device="cuda")
    v = flat[off:].view(x.shape)
    v.copy_(torch.from_numpy(x))
    return v


def _run_all(hip, pw, xd, refs, m, n, what, want=None):
    import torch
    for name, kind in KINDS.items():
        so, ref = refs[kind]
        for yl in (0, T) if kind in (3, 4) else (0,):
            say(f"rows at {what} {name} y={yl}")
            y = pw.run(xd, 0.02, kind, out_scale=so, y_layout=yl, m_tokens=m)
            torch.cuda.synchronize()
            if want:
                assert hip.last_path().startswith(want), hip.last_path()
            got = hip.from_t16x32(y.cpu().numpy(), m, n) if yl == T else y.cpu().numpy()
            check(kind, got, ref, f"{what} {name} y={yl} {hip.last_path()}")


@pytest.mark.parametrize("path", ["", "split", "panel"])
@pytest.mark.parametrize("m,n,k", [(1, 4, 1), (5, 20, 3), (17, 36, 33), (16, 64, 126), (33, 100, 257), (50, 132, 1001),
                                   (31, 48, 2050), (70, 32, 1004)])
def test_rows_at_every_byte(hip, monkeypatch, path, m, n, k):
    import torch
    if path:
        monkeypatch.setenv("SL_PATH", path)
    w, sw, b, rng = _case(n, k, 0.3, m + 3 * n + k)
    x = rng.integers(-127, 128, (m, k), dtype=np.int8)
    refs = _refs(x, w, sw, b)
    pw = hip.PackedWeight.pack(w, sw, b)
    for off in range(4):
        _run_all(hip, pw, _view(torch, x, off), refs, m, n, f"{path} m={m} n={n} k={k} offset {off}", path)
    pw.free()


@pytest.mark.parametrize("shape", ["8,2,8,2", "4,2,8,2", "2,2,8,4"])
@pytest.mark.parametrize("k", [129, 1022])
def test_rows_at_panel_shapes(hip, monkeypatch, shape, k):
    import torch
    m, n = 700, 132
    monkeypatch.setenv("SL_PATH", "panel")
    monkeypatch.setenv("SL_PTILE", shape)
    monkeypatch.setenv("SL_PSLICES", "1")
    w, sw, b, rng = _case(n, k, 0.2, n + k)
    x = rng.integers(-127, 128, (m, k), dtype=np.int8)
    refs = _refs(x, w, sw, b)
    pw = hip.PackedWeight.pack(w, sw, b)
    for off in (0, 3):
        _run_all(hip, pw, _view(torch, x, off), refs, m, n, f"{shape} k={k} offset {off}", f"panel {shape} ")
    pw.free()


# what runs by default on either side of the alignment rules, above the few
# tokens that the split-reduction kernel takes
@pytest.mark.parametrize("m,n,k,off,want", [
    (700, 1000, 1001, 0, "panel"), (700, 1000, 1004, 0, "panel"), (700, 1000, 1004, 2, "panel"),
    (1400, 1000, 2500, 0, "direct"), (1400, 1000, 2501, 0, "panel"), (1400, 1000, 2500, 4, "direct"),
    (1400, 1000, 5001, 0, "staged")])
def test_rows_at_choice(hip, monkeypatch, m, n, k, off, want):
    import torch
    monkeypatch.delenv("SL_PATH", raising=False)
    w, sw, b, rng = _case(n, k, 0.1, n + k)
    x = rng.integers(-127, 128, (m, k), dtype=np.int8)
    rows = np.concatenate([np.arange(0, m - 20, 97), np.arange(m - 20, m)])
    refs = _refs(np.ascontiguousarray(x[rows]), w, sw, b)
    pw = hip.PackedWeight.pack(w, sw, b)
    xd = _view(torch, x, off)
    for name, kind in KINDS.items():
        so, ref = refs[kind]
        say(f"rows at choice {n}x{k} offset {off} {name}")
        y = pw.run(xd, 0.02, kind, out_scale=so)
        torch.cuda.synchronize()
        assert hip.last_path().startswith(want), hip.last_path()
        check(kind, y.cpu().numpy()[rows], ref, f"{n}x{k} offset {off} {name}")
    pw.free()
