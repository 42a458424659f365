"""GPU parity of the few-token strips (csrc/sq_thin.h): calls of up to 64 tokens
over contractions longer than 2048, and grouped calls of such experts whose
strips leave the chip idle.  Sizes sit at the edges of the 16-token tiles, of
the 16-, 32- and 64-column strips and of the steps of 128 to 512 terms, and
take every strip the dispatch can launch (asserted).  Every element is held to
the summation bound of tests/parity_check.py against the oracle.  Strips add in
the tiles' order: a call equals the same rows of a longer call, and an expert of
a grouped call its single call, bit for bit, whichever of the two each takes."""

import os
import re

import numpy as np
import pytest
import torch

from conftest import ROOT, ensure_library, gpu_ready
from oracle import linear
from parity_check import assert_elements
from test_gpu_gemm import TOL, abs_sums, depths, make_layer, normwise, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

CUS = 256


@pytest.fixture(scope="module")
def sq():
    ensure_library()
    from paper_2609_04526_amd import sq as _sq
    return _sq


def source():
    with open(os.path.join(ROOT, "paper_2609_04526_amd", "csrc", "sq_gemm.hip")) as f:
        return f.read()


def fwd_shapes():
    m = re.search(r"kThinFwdShapes\[\] = \{(.*?)\};", source())
    return [(int(a), int(b), float(u)) for a, b, u in re.findall(r"\{(\d), (\d), ([\d.]+)\}", m.group(1))]


def wgs(Ts, N, mt, nt):
    return sum(-(-T // (16 * mt)) for T in Ts) * -(-N // (16 * nt))


def fwd_strip(fmt, Ts, O, I, grouped):
    """(MT, NT) of the strips that a forward of these experts takes, None for tiles."""
    if I <= 2048 or max(Ts) > 64:
        return None
    mt, nt, _ = min(fwd_shapes(), key=lambda c: c[2] * -(-wgs(Ts, O, c[0], c[1]) // CUS))
    if grouped and wgs(Ts, O, mt, nt) > (1 if fmt == "mx" else 2) * CUS:
        return None
    return mt, nt


def dx_strip(Ts, O, I):
    if O <= 2048 or max(Ts) > 64:
        return None
    mt = 1 if max(Ts) <= 16 else 2 if max(Ts) <= 32 or wgs(Ts, I, 2, 2) <= CUS else 3 if max(Ts) <= 48 else 4
    return (mt, 2) if wgs(Ts, I, mt, 2) <= 2 * CUS else None


def check(fmt, X, dY, codes, sb, ws2, Y, dX, what):
    Xd, dYd = X.double().numpy(), dY.double().numpy()
    W = linear.dequant(fmt, codes, sb, ws2)
    T, I = Xd.shape
    aY, adX, _ = abs_sums(fmt, Xd, dYd, codes, W)
    kY, kX, _ = depths(fmt, T, W.shape[0], I)
    for got, ref, a, k, name in ((Y, linear.forward(Xd, W), aY, kY, "Y"), (dX, linear.backward_dx(dYd, W), adX, kX, "dX")):
        assert normwise(got, ref) <= TOL
        assert_elements(got, ref, a, k, f"{what} {name}")


SINGLE = [
    ("mx", 1, 8, 2080), ("nv", 1, 2056, 16),             # the narrowest strips, one token
    ("mx", 16, 40, 2208), ("nv", 15, 2072, 144),         # a token tile and one row less, ragged strips and steps
    ("mx", 17, 2056, 2304), ("nv", 17, 2056, 2064),      # long contractions both ways, one row over a tile
    ("mx", 33, 2064, 2176), ("nv", 33, 4104, 2096),
    ("mx", 64, 2056, 4128), ("nv", 64, 2072, 4112),      # the most tokens; NVFP4 rows ending inside a step's chunk
    ("nv", 48, 2080, 4224),
    ("mx", 64, 4096, 2048), ("nv", 64, 4096, 2048),      # dX here, the forward on tiles
    ("mx", 7, 8200, 2080), ("nv", 16, 8200, 2064),       # 1 x 4 strips of the forward
    ("mx", 18, 14344, 2080), ("nv", 32, 14344, 2064),    # 2 x 4
    ("mx", 48, 14344, 2304), ("nv", 47, 14344, 2064),    # 3 x 4; all sizes of the widest linear, ragged
    ("mx", 64, 14344, 2080), ("nv", 63, 14344, 2064),    # 4 x 4
    ("mx", 3, 4104, 2304), ("nv", 9, 4104, 2064),        # 1 x 2
    ("mx", 33, 4104, 2304),                              # 2 x 2
    ("mx", 48, 2056, 4160), ("nv", 40, 2056, 4176),      # dX of 3 token tiles, and of 4
    ("mx", 50, 2056, 8160), ("nv", 64, 2056, 8176),
    ("mx", 5, 2056, 16416), ("nv", 5, 2056, 16400),      # dX strips past two workgroups per CU: tiles
]


def test_every_strip_is_taken():
    """The parametrisations reach each strip of the dispatch, both formats."""
    for fmt in ("mx", "nv"):
        assert {fwd_strip(f, [T], O, I, False) for f, T, O, I in SINGLE if f == fmt} == {s[:2] for s in fwd_shapes()} | {None}
        assert {dx_strip([T], O, I) for f, T, O, I in SINGLE if f == fmt} == {(m, 2) for m in (1, 2, 3, 4)} | {None}
        grouped = {fwd_strip(fmt, [t for t in Ts if t], O, I, True) for Ts, O, I in GROUPED}
        assert grouped == {s[:2] for s in fwd_shapes()} | {None}
        assert {dx_strip([t for t in Ts if t], O, I) for Ts, O, I in GROUPED} == {(m, 2) for m in (1, 2, 3, 4)} | {None}


@pytest.mark.parametrize("fmt,T,O,I", SINGLE)
def test_parity(sq, fmt, T, O, I):
    X, dY, codes, sb, ws2 = make_layer(fmt, T, O, I, seed=9000 + T + O)
    Xc, dYc, c, s = to_dev(X, dY, codes, sb)
    print(f"[thin] fmt={fmt} T={T} O={O} I={I} fwd {fwd_strip(fmt, [T], O, I, False)} dx {dx_strip([T], O, I)}", flush=True)
    Y, dX = sq.sq_fwd(fmt, Xc, c, s, ws2), sq.sq_bwd_dx(fmt, dYc, c, s, ws2)
    check(fmt, X, dY, codes, sb, ws2, Y.cpu().numpy(), dX.cpu().numpy(), f"{fmt} {T}x{O}x{I}")
    # bf16 outputs are the fp32 ones, rounded
    assert torch.equal(sq.sq_fwd(fmt, Xc, c, s, ws2, torch.bfloat16), Y.to(torch.bfloat16))
    assert torch.equal(sq.sq_bwd_dx(fmt, dYc, c, s, ws2, torch.bfloat16), dX.to(torch.bfloat16))
    # the same rows among 130: the tiles give the same bits
    Xl, dYl = Xc.repeat(130 // T + 1, 1)[:130].contiguous(), dYc.repeat(130 // T + 1, 1)[:130].contiguous()
    assert torch.equal(sq.sq_fwd(fmt, Xl, c, s, ws2)[:T], Y)
    assert torch.equal(sq.sq_bwd_dx(fmt, dYl, c, s, ws2)[:T], dX)
    # planes at the least alignment the entry points take (codes 4 bytes, scales any)
    cb = torch.empty(codes.size + 4, dtype=torch.uint8, device="cuda")[4:].view(codes.shape)
    ub = torch.empty(sb.size + 1, dtype=torch.uint8, device="cuda")[1:].view(sb.shape)
    cb.copy_(c)
    ub.copy_(s)
    Yu = sq.sq_fwd(fmt, Xc, cb, ub, ws2)
    if fmt == "nv" or I % 256:                           # (else the aligned call adds in the register path's order)
        assert torch.equal(Yu, Y)
    assert torch.equal(sq.sq_fwd(fmt, Xl, cb, ub, ws2)[:T], Yu)
    assert torch.equal(sq.sq_bwd_dx(fmt, dYc, cb, ub, ws2), dX)


GROUPED = [
    ([1, 16, 7, 5], 520, 2112),                          # 16-output strips; dX of up to 2048 terms on tiles
    ([1, 16, 7, 5], 2056, 2304),
    ([1, 16, 17, 64, 33, 5], 264, 2112),
    ([40, 33, 64], 1032, 2304),
    ([64, 33], 2056, 2304),                              # mixed token tiles
    ([16, 3], 4096, 2304),
    ([48, 40, 33], 4104, 2336),
    ([3, 16, 0, 7], 4104, 2080),                         # 64-output strips, an expert without tokens
    ([20, 32, 17, 9], 4096, 2304),
    ([64, 50, 60], 4104, 2336),
    ([48, 40, 33], 2056, 4128),
    ([64, 61, 60], 2056, 4160),
    ([5] * 40, 2056, 2304),                              # enough strips to fill the chip: tiles
    ([64, 33, 2, 17] * 8, 2056, 2304),
    ([1, 16, 17, 65, 64, 200, 9], 2056, 2304),           # among larger experts: tiles
    ([16, 17, 300, 1, 129], 264, 512),
    ([2200, 12, 2100], 2056, 2304),                      # beside experts on the long or large tiles
]


@pytest.mark.parametrize("fmt", ["mx", "nv"])
@pytest.mark.parametrize("Ts,O,I", GROUPED, ids=lambda v: str(v)[:24])
def test_grouped_equals_single(sq, fmt, Ts, O, I):
    E = len(Ts)
    L = [make_layer(fmt, T, O, I, seed=9300 + 7 * e) for e, T in enumerate(Ts)]
    Xs, dYs = [x[0].cuda() for x in L], [x[1].cuda() for x in L]
    cs, ss = [torch.from_numpy(x[2]).cuda() for x in L], [torch.from_numpy(x[3]).cuda() for x in L]
    ws2 = [float(np.float32(x[4] / (1 + e % 2))) for e, x in enumerate(L)]
    used = [t for t in Ts if t]
    print(f"[thin grouped] fmt={fmt} T={Ts} O={O} I={I} fwd {fwd_strip(fmt, used, O, I, True)} dx {dx_strip(used, O, I)}", flush=True)
    Ys = sq.sq_fwd_grouped(fmt, Xs, cs, ss, ws2)
    dXs = sq.sq_bwd_dx_grouped(fmt, dYs, cs, ss, ws2)
    for e in range(E):
        if Ts[e] == 0:
            continue
        assert torch.equal(Ys[e], sq.sq_fwd(fmt, Xs[e], cs[e], ss[e], ws2[e])), (e, Ts[e])
        assert torch.equal(dXs[e], sq.sq_bwd_dx(fmt, dYs[e], cs[e], ss[e], ws2[e])), (e, Ts[e])
    check(fmt, L[0][0], L[0][1], L[0][2], L[0][3], ws2[0], Ys[0].cpu().numpy(), dXs[0].cpu().numpy(), "expert 0")


@pytest.mark.parametrize("fmt,T,O,I", [("nv", 20, 2056, 2064), ("mx", 20, 2056, 2080)])
def test_nan_and_infinite_inputs_stay_in_their_rows(sq, fmt, T, O, I):
    """A NaN scale reaches exactly its output column of the forward and its
    block's columns of dX; an infinite activation its row."""
    X, dY, codes, sb, ws2 = make_layer(fmt, T, O, I, seed=9500)
    codes[5, :] = 0x22
    sb[5, -1] = 0xFF if fmt == "mx" else 0x7F
    X[3, 17] = float("inf")
    X[3, 18:] = 1.0
    Xc, dYc, c, s = to_dev(X, dY, codes, sb)
    Y = sq.sq_fwd(fmt, Xc, c, s, ws2).cpu().numpy()
    bad = ~np.isfinite(Y)
    assert np.isnan(Y[:, 5]).all()
    want = np.zeros_like(bad)
    want[3, :] = True
    want[:, 5] = True
    assert (bad <= want).all() and bad[3].any()
    dX = sq.sq_bwd_dx(fmt, dYc, c, s, ws2).cpu().numpy()
    B = 32 if fmt == "mx" else 16
    assert np.isnan(dX[:, I - B:]).all() and np.isfinite(dX[:, :I - B]).all()
