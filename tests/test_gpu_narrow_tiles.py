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


@pytest.mark.parametrize("fmt", ["mx", "nv"])
@pytest.mark.parametrize("Ts,O,I", [
    ([1, 0, 5, 33, 2, 7, 1], 136, 416),                    # 8 tokens on average and less: 32 x 128
    ([32, 31, 1, 0, 64, 3, 1, 2], 264, 512),               # 16: the most for 32 x 128 forward (MXFP4) and dX
    ([40, 65, 96, 1, 129, 30], 264, 528),                  # NVFP4 and 4-byte planes: 64 x 128
])
def test_few_tokens_per_expert(sq, fmt, Ts, O, I):
    I -= I % 32 if fmt == "mx" else 0
    L = [make_layer(fmt, T, O, I, seed=9800 + 7 * e) for e, T in enumerate(Ts)]
    Xs, dYs = [x[0].cuda() for x in L], [x[1].cuda() for x in L]
    cs, ss = [torch.from_numpy(x[2]).cuda() for x in L], [torch.from_numpy(x[3]).cuda() for x in L]
    ws2 = [x[4] for x in L]
    print(f"[few per expert] fmt={fmt} T={Ts} O={O} I={I}", flush=True)
    for out in (torch.float32, torch.bfloat16):
        Ys = sq.sq_fwd_grouped(fmt, Xs, cs, ss, ws2, out)
        dXs = sq.sq_bwd_dx_grouped(fmt, dYs, cs, ss, ws2, out)
        for e, T in enumerate(Ts):
            if T:
                assert torch.equal(Ys[e], sq.sq_fwd(fmt, Xs[e], cs[e], ss[e], ws2[e], out)), (e, T)
                assert torch.equal(dXs[e], sq.sq_bwd_dx(fmt, dYs[e], cs[e], ss[e], ws2[e], out)), (e, T)
            if out == torch.float32 and e in (0, 3):
                check(fmt, *L[e], Ys[e].cpu().numpy(), dXs[e].cpu().numpy(), f"expert {e}")
