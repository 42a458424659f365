"""Parity of the tiles that single products take when their grid leaves the
chip idle: 64 x 64 and 64 x 128 (MXFP4 forward), 128 x 64 (NVFP4 forward), 64 x
128 (dX), 256 x 128 (NVFP4 forward and dX) and 128 x 128 after a thin second
round of large tiles; and those of experts of a few tokens each, 32 x 128 and
64 x 128.  Ragged in every dimension, on both sides of each limit,
against the oracle per element; a grouped call of the same expert, whose tiles
differ, gives the same bits."""

import pytest
import torch

from conftest import ensure_library, gpu_ready
from test_gpu_gemm import make_layer, to_dev
from test_gpu_thin import check

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def sq():
    ensure_library()
    from paper_2609_04526_amd import sq as _sq
    return _sq


def tiles(M, N):
    return -(-M // 128) * -(-N // 128)


SHAPES = [
    ("mx", 65, 72, 256), ("nv", 65, 72, 272),              # one tile, one row over 64
    ("mx", 193, 200, 1024), ("nv", 193, 200, 528),
    ("mx", 1270, 2040, 256), ("mx", 1290, 2040, 256),       # 160 and 176 tiles: 64 x 64, 64 x 128
    ("mx", 1020, 3704, 256), ("mx", 1540, 2440, 256),       # 232 and 260: 64 x 128
    ("mx", 1020, 3720, 256), ("mx", 2030, 2040, 256),       # 240 and 256: 128 x 128
    ("mx", 2800, 2040, 256), ("mx", 2820, 2056, 256),       # 352 and 391: 64 x 128, 128 x 128
    ("nv", 1020, 2040, 272), ("nv", 1030, 2056, 272),       # 128 and 153: 128 x 64, 128 x 128
    ("mx", 1000, 264, 2040 // 32 * 32), ("nv", 1030, 264, 2032),   # dX: 128 tiles and more
    ("nv", 2040, 4104, 2064), ("mx", 1290, 2056, 4128),     # 256 x 128 tiles over long sums
    ("nv", 346, 12296, 2064), ("mx", 346, 2056, 12320),     # not where they would be a third padding
    ("mx", 1290, 14344, 64), ("nv", 1290, 14344, 64),       # 342 large tiles: a thin second round
]


def test_the_limits_are_on_both_sides():
    n = {f"{fmt} fwd": sorted(tiles(T, O) for f, T, O, I in SHAPES if f == fmt) for fmt in ("mx", "nv")}
    for at in (160, 176, 232, 240, 256, 260, 352, 391):
        assert at in n["mx fwd"], at
    assert {128, 153} <= set(n["nv fwd"])
    dx = {tiles(T, I) for f, T, O, I in SHAPES}
    assert 128 in dx and any(128 < t < 160 for t in dx)


@pytest.mark.parametrize("fmt,T,O,I", SHAPES)
def test_parity_and_grouped_bits(sq, fmt, T, O, I):
    X, dY, codes, sb, ws2 = make_layer(fmt, T, O, I, seed=9700 + T + O)
    Xc, dYc, c, s = to_dev(X, dY, codes, sb)
    print(f"[narrow] fmt={fmt} T={T} O={O} I={I} tiles fwd {tiles(T, O)} dx {tiles(T, I)}", flush=True)
    Y, dX = sq.sq_fwd(fmt, Xc, c, s, ws2), sq.sq_bwd_dx(fmt, dYc, c, s, ws2)
    Yb, dXb = (sq.sq_fwd(fmt, Xc, c, s, ws2, torch.bfloat16), sq.sq_bwd_dx(fmt, dYc, c, s, ws2, torch.bfloat16))
    check(fmt, X, dY, codes, sb, ws2, Y.cpu().numpy(), dX.cpu().numpy(), f"{fmt} {T}x{O}x{I}")
    assert torch.equal(Yb, Y.to(torch.bfloat16)) and torch.equal(dXb, dX.to(torch.bfloat16))
    Yg = sq.sq_fwd_grouped(fmt, [Xc, Xc[:70]], [c, c], [s, s], [ws2, ws2])
    dXg = sq.sq_bwd_dx_grouped(fmt, [dYc, dYc[:70]], [c, c], [s, s], [ws2, ws2])
    assert torch.equal(Yg[0], Y) and torch.equal(dXg[0], dX)


def grouped_tile(kind, fmt, Ts, O, I):
    """The tile that a grouped call of few-token experts takes (csrc/sq_gemm.hip, grouped_sized)."""
    Ts = [T for T in Ts if T]                              # empty experts are left out before
    n, N = len(Ts), O if kind == "fwd" else I
    r32, r64, r128 = (sum(-(-T // r) for T in Ts) for r in (32, 64, 128))
    cols = -(-N // 128)
    if kind == "dx":
        few = sum(Ts) <= 16 * n and r32 == r64 and (I <= 2304 or r32 * cols <= 256)
        return "32x128" if few else "64x256" if sum(Ts) <= 96 * n else None
    if fmt == "mx" and I % 256 == 0:                       # registers dequantise
        return "32x128" if sum(Ts) <= 16 * n and (r32 == r64 or r32 * cols <= 512) else "64x256"
    if sum(Ts) <= 8 * n:
        return "32x128"
    return "64x128" if sum(Ts) <= 96 * n and (5 * r64 <= 7 * r128 or r64 * cols <= 256) else "128x128"


# (experts' tokens, O, I, forward tile MXFP4, NVFP4, dX tile)
FEW = [
    ([1, 0, 5, 33, 2, 7, 0], 136, 416, "64x128", "64x128", "64x256"),        # 9.6 tokens an expert, one over 32
    ([1, 5, 31, 2, 7, 2, 8], 264, 512, "32x128", "32x128", "32x128"),        # exactly 8, registers (MXFP4)
    ([1, 5, 32, 2, 7, 2, 8], 264, 512, "32x128", "64x128", "32x128"),        # one token more
    ([3, 0, 9, 12, 8], 264, 528, "32x128", "32x128", "32x128"),              # exactly 8, through LDS
    ([32, 32, 1, 2, 30, 4, 11], 264, 512, "32x128", "64x128", "32x128"),     # exactly 16, the most
    ([32, 32, 1, 2, 30, 4, 12], 264, 512, "64x256", "64x128", "64x256"),     # one token more
    ([33, 30, 1, 2, 30, 4, 12], 264, 512, "32x128", "64x128", "64x256"),     # 16, one expert over 32: few tiles
    ([33, 1, 2, 1] * 32, 520, 256, "64x256", "64x128", "64x256"),            # the same where they fill the chip
    ([1, 5, 31, 2, 7, 2, 8], 136, 416, "32x128", "32x128", "32x128"),        # exactly 8, MXFP4 through LDS
    ([3, 1, 2, 1] * 16, 96, 2560, None, None, "64x256"),                     # dX over long rows, 1280 tiles (forward: strips)
    ([40, 65, 96, 1, 129, 30], 264, 528, "64x256", "64x128", "64x256"),
    ([96, 90, 100, 98], 264, 528, "64x256", "64x128", "64x256"),             # exactly 96: 64 x 128 one to a CU
    ([96, 90, 100, 99], 264, 528, "64x256", "128x128", None),
    ([100, 90, 80, 70] * 16, 1032, 80, "128x128", "128x128", "64x256"),      # 64-row tiles twice the 128-row ones
]


def test_the_few_token_tiles_are_all_taken():
    for Ts, O, I, mx, nv, dx in FEW:
        Im = I - I % 32
        assert I > 2048 or (grouped_tile("fwd", "mx", Ts, O, Im), grouped_tile("fwd", "nv", Ts, O, I)) == (mx, nv), Ts
        assert grouped_tile("dx", "mx", Ts, O, Im) == grouped_tile("dx", "nv", Ts, O, I) == dx, Ts
    assert {(mx, (I - I % 32) % 256 == 0) for _, _, I, mx, _, _ in FEW} >= {("32x128", True), ("64x256", True), ("32x128", False), ("64x128", False)}


@pytest.mark.parametrize("fmt", ["mx", "nv"])
@pytest.mark.parametrize("Ts,O,I", [c[:3] for c in FEW], ids=lambda v: str(v)[:24])
def test_few_tokens_per_expert(sq, fmt, Ts, O, I):
    I -= I % 32 if fmt == "mx" else 0
    L = [make_layer(fmt, T, O, I, seed=9800 + 7 * e) for e, T in enumerate(Ts)]
    Xs, dYs = [x[0].cuda() for x in L], [x[1].cuda() for x in L]
    cs, ss = [torch.from_numpy(x[2]).cuda() for x in L], [torch.from_numpy(x[3]).cuda() for x in L]
    ws2 = [x[4] for x in L]
    print(f"[few per expert] fmt={fmt} T={Ts[:8]} O={O} I={I} fwd {grouped_tile('fwd', fmt, Ts, O, I)} "
          f"dx {grouped_tile('dx', fmt, Ts, O, I)}", flush=True)
    for out in (torch.float32, torch.bfloat16):
        Ys = sq.sq_fwd_grouped(fmt, Xs, cs, ss, ws2, out)
        dXs = sq.sq_bwd_dx_grouped(fmt, dYs, cs, ss, ws2, out)
        for e, T in enumerate(Ts):
            if T:
                assert torch.equal(Ys[e], sq.sq_fwd(fmt, Xs[e], cs[e], ss[e], ws2[e], out)), (e, T)
                assert torch.equal(dXs[e], sq.sq_bwd_dx(fmt, dYs[e], cs[e], ss[e], ws2[e], out)), (e, T)
            if out == torch.float32 and T and e < 8:
                check(fmt, *L[e], Ys[e].cpu().numpy(), dXs[e].cpu().numpy(), f"expert {e}")
