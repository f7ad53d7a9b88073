"""GPU parity of the tile kernel (128 tokens x 6 or 8 channel tiles, the
reduction's halves split over its waves), through the C ABI: every epilogue
kind and layout pairing at the edges of its tiles -- ragged tokens, channels
and last window, fewer and more windows than its ring holds, several channel
groups -- and which kernel runs by default on either side of its rules. Bars as
in test_gpu_parity.py.
"""
import numpy as np
import pytest

import oracle
from test_gpu_panel import T, _refs
from test_gpu_parity import KINDS, _case, check, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt", [6, 8])
@pytest.mark.parametrize("m,n,k", [(1, 4, 16), (128, 96, 128), (130, 132, 400), (129, 256, 512), (300, 100, 656),
                                   (257, 200, 1040), (140, 128, 2048)])
def test_tile_shapes(hip, monkeypatch, nt, m, n, k):
    import torch
    w, sw, b, rng = _case(n, k, 0.25, 5 * m + n + k)
    x = rng.integers(-127, 128, (m, k), dtype=np.int8)
    refs = _refs(x, w, sw, b)
    pw = hip.PackedWeight.pack(w, sw, b)
    xd = {0: torch.from_numpy(x).cuda(), T: torch.from_numpy(np.ascontiguousarray(hip.to_t16x32(x, fill=77))).cuda()}
    monkeypatch.setenv("SL_PATH", "tile")
    monkeypatch.setenv("SL_TILE", f"{nt},0,0,0,0")
    for xl, yl in [(0, 0), (T, 0), (T, T), (0, T)]:
        for name, kind in KINDS.items():
            if yl == T and kind not in (3, 4):
                continue
            so, ref = refs[kind]
            for off in (0, 4) if yl == 0 and kind in (3, 4) else (0,):
                say(f"tile {nt} m={m} n={n} k={k} layouts=({xl},{yl}) {name} offset {off}")
                out = None
                if off:
                    out = torch.empty(m * n + off, dtype=torch.int8, device="cuda")[off:].view(m, n)
                y = pw.run(xd[xl], 0.02, kind, out_scale=so, x_layout=xl, y_layout=yl, m_tokens=m, out=out)
                torch.cuda.synchronize()
                assert hip.last_path().startswith(f"tile 128,{nt}"), hip.last_path()
                got = hip.from_t16x32(y.cpu().numpy(), m, n) if yl == T else y.cpu().numpy()
                check(kind, got, ref, f"tile {nt} {name} m={m} n={n} k={k} layouts=({xl},{yl}) offset {off}")
    pw.free()


@pytest.mark.parametrize("n,k,m,kind,xl,yl,want", [
    (768, 3072, 4096, 1, 0, 0, "tile 128,6"), (768, 3072, 4096, 3, T, 0, "tile 128,6"),
    (768, 3072, 4096, 3, T, T, "direct"), (768, 3072, 4096, 3, 0, T, "tile 128,6"),
    (768, 3072, 2048, 1, 0, 0, "staged"), (1024, 4096, 4096, 1, T, 0, "tile 128,8"),
    (1024, 4096, 4096, 1, 0, 0, "tile 128,8"), (768, 768, 4096, 1, 0, 0, "panel"),
    # more rounds of workgroups: short reductions stay with the kernels that
    # overlap finishing a tile, long ones and int8 rows do not
    (4096, 1408, 8192, 1, 0, 0, "staged"), (1072, 1184, 11821, 0, 0, 0, "staged"),
    (4096, 1040, 8192, 2, 0, 0, "staged"), (1072, 1040, 4096, 1, 0, 0, "tile 128,6"),
    (1024, 4096, 12000, 1, 0, 0, "tile 128,8"), (4096, 1040, 4096, 3, 0, 0, "tile 128,8"),
    (4096, 1040, 4096, 4, 0, T, "direct"), (1024, 1152, 8192, 4, 0, T, "tile 128,8"),
    (4096, 1040, 2048, 1, T, 0, "direct"), (4096, 1040, 4096, 3, T, T, "direct"),
    (4096, 1040, 4096, 3, T, 0, "tile 128,8")])
def test_tile_choice(hip, monkeypatch, n, k, m, kind, xl, yl, want):
    import torch
    monkeypatch.delenv("SL_PATH", raising=False)
    w, sw, b, rng = _case(n, k, 0.2, n + m)
    x = rng.integers(-127, 128, (m, k), dtype=np.int8)
    rows = np.arange(0, m, 61)
    pw = hip.PackedWeight.pack(w, sw, b)
    xd = torch.from_numpy(np.ascontiguousarray(hip.to_t16x32(x)) if xl == T else x).cuda()
    so, ref = _refs(np.ascontiguousarray(x[rows]), w, sw, b)[kind]
    y = pw.run(xd, 0.02, kind, out_scale=so, x_layout=xl, y_layout=yl, m_tokens=m)
    torch.cuda.synchronize()
    assert hip.last_path().startswith(want), hip.last_path()
    got = hip.from_t16x32(y.cpu().numpy(), m, n) if yl == T else y.cpu().numpy()
    check(kind, got[rows], ref, f"{n}x{k} m={m} {hip.last_path()}")
    pw.free()


def test_more_tiles_than_a_launch_takes(hip, monkeypatch):
    """2,063,872 x 66,720 int8 outputs (137 GB) would be 8.4 million tile
    workgroups, over the 2^32 threads of one launch: another kernel runs them."""
    import torch
    m, n, k = 2063872, 66720, 1040
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of free GPU memory")
    monkeypatch.delenv("SL_PATH", raising=False)
    rng = np.random.default_rng(5)
    w = np.zeros((n // 4, 4, k), np.int8)
    for _ in range(16):
        w[np.arange(n // 4), :, rng.integers(0, k, n // 4)] = rng.integers(1, 128, (n // 4, 4), dtype=np.int8)
    w = w.reshape(n, k)
    sw = rng.uniform(0.001, 0.01, n).astype(np.float32)
    pw = hip.PackedWeight.pack(w, sw)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randint(-127, 128, (m, k), dtype=torch.int8, device="cuda", generator=g)
    say(f"tile launch limit m={m} n={n} k={k}")
    y = pw.run(x, 0.02, 3, out_scale=0.05)
    torch.cuda.synchronize()
    assert not hip.last_path().startswith("tile"), hip.last_path()
    rows = torch.cat([torch.arange(0, m, m // 40), torch.arange(m - 3, m)]).cuda()
    got, xs = y[rows].cpu().numpy(), x[rows].cpu().numpy()
    check(3, got, oracle.linear(xs, w, 0.02, sw, None, 3, so=0.05), f"{n}x{k} m={m} {hip.last_path()}")
    pw.free()
    del x, y
    torch.cuda.empty_cache()

