"""GPU parity of the weight-stationary kernel's 8-tile shapes and of its int8
stores (16 bytes a lane at any multiple of 4), through the C ABI: every
epilogue kind and layout pairing at the edges of its tiles -- a ragged last
channel tile, channel group, token group and window, row widths that are no
multiple of 16, an output that is only 4-byte aligned, one window and several
token groups a wave -- and which shape runs by default on either side of its
rules. Bars as in test_gpu_parity.py.
"""
import numpy as np
import pytest

from test_gpu_panel import T, _refs
from test_gpu_parity import KINDS, _case, check, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["8,2,8,2", "8,2,12,2", "6,2,8,2"])
@pytest.mark.parametrize("m,n,k", [(1, 4, 16), (33, 128, 128), (70, 132, 272), (64, 256, 768), (850, 144, 1024)])
def test_wide_shapes(hip, monkeypatch, shape, m, n, k):
    import torch
    w, sw, b, rng = _case(n, k, 0.25, 5 * m + n + k)
    x = rng.integers(-127, 128, (m, k), dtype=np.int8)
    refs = _refs(x, w, sw, b)
    pw = hip.PackedWeight.pack(w, sw, b)
    xd = {0: torch.from_numpy(x).cuda(), T: torch.from_numpy(np.ascontiguousarray(hip.to_t16x32(x, fill=77))).cuda()}
    monkeypatch.setenv("SL_PATH", "panel")
    monkeypatch.setenv("SL_PTILE", shape)
    monkeypatch.setenv("SL_PSLICES", "1")
    for xl, yl in [(0, 0), (T, 0), (T, T), (0, T)]:
        for name, kind in KINDS.items():
            if yl == T and kind not in (3, 4):
                continue
            so, ref = refs[kind]
            for off in (0, 4) if yl == 0 and kind in (3, 4) else (0,):
                say(f"panel {shape} m={m} n={n} k={k} layouts=({xl},{yl}) {name} offset {off}")
                out = None
                if off:
                    out = torch.empty(m * n + off, dtype=torch.int8, device="cuda")[off:].view(m, n)
                y = pw.run(xd[xl], 0.02, kind, out_scale=so, x_layout=xl, y_layout=yl, m_tokens=m, out=out)
                torch.cuda.synchronize()
                assert hip.last_path().startswith(f"panel {shape} "), hip.last_path()
                got = hip.from_t16x32(y.cpu().numpy(), m, n) if yl == T else y.cpu().numpy()
                check(kind, got, ref, f"{shape} {name} m={m} n={n} k={k} layouts=({xl},{yl}) offset {off}")
    pw.free()


# (n, k, m, kind, block layouts): int8 and fp32 rows, and blocks whose 6-tile
# groups leave a remainder or not
@pytest.mark.parametrize("n,k,m,kind,blocks,want", [
    (2304, 768, 4096, 3, False, "panel 8,2,8,2"), (2308, 768, 4096, 1, False, "panel 6,2"),
    (4096, 1024, 8192, 3, True, "panel 8,2,12,2"), (3072, 768, 4096, 3, True, "panel 6,2,12,2"),
    (768, 768, 4096, 3, True, "panel"), (768, 768, 4096, 1, False, "panel"),
    # one token group a wave of the 4-tile shape, or of the 2-tile one with GELU,
    # from rows; a wave's second group of 6 tiles against its first of 8
    (4096, 1024, 700, 1, False, "panel 4,2,8,2"), (4096, 1024, 1000, 2, False, "panel 4,2,8,2"),
    (3072, 1024, 255, 2, False, "panel 2,2,8,4"), (3072, 1024, 700, 2, False, "panel 4,2,8,2"),
    (3072, 1024, 255, 1, False, "panel 4,2,8,2"), (3072, 768, 1500, 1, False, "panel 6,2"),
    (4096, 1024, 1537, 1, False, "panel 8,2,12,2"), (3072, 768, 2228, 2, True, "panel 8,2,12,2"),
    # int8 from rows: few token groups, or a short reduction into blocks
    (2048, 512, 384, 4, False, "panel 4,2,8,2"), (624, 128, 1700, 4, False, "panel 4,2,8,2"),
    (2400, 96, 1400, 4, False, "panel 8,2,8,2"), (3072, 768, 1024, 3, False, "panel 8,2,8,2")])
def test_wide_choice(hip, monkeypatch, n, k, m, kind, blocks, want):
    import torch
    monkeypatch.delenv("SL_PATH", raising=False)
    monkeypatch.delenv("SL_PTILE", raising=False)
    w, sw, b, rng = _case(n, k, 0.2, n + m)
    x = rng.integers(-127, 128, (m, k), dtype=np.int8)
    rows = np.arange(0, m, 61)
    pw = hip.PackedWeight.pack(w, sw, b)
    xl = T if blocks else 0
    xd = torch.from_numpy(np.ascontiguousarray(hip.to_t16x32(x)) if blocks else x).cuda()
    so, ref = _refs(np.ascontiguousarray(x[rows]), w, sw, b)[kind]
    yl = xl if kind in (3, 4) else 0
    y = pw.run(xd, 0.02, kind, out_scale=so, x_layout=xl, y_layout=yl, m_tokens=m)
    torch.cuda.synchronize()
    assert hip.last_path().startswith(want), hip.last_path()
    got = hip.from_t16x32(y.cpu().numpy(), m, n) if yl else y.cpu().numpy()
    check(kind, got[rows], ref, f"{n}x{k} m={m} {hip.last_path()}")
    pw.free()
