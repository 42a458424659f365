"""GPU parity of the few-token forward and dX (csrc/sq_thin.h): calls and
experts of up to 64 tokens over contractions longer than 2048.  Sizes sit at the edges of the 16-token tiles, of
the 16-, 32- and 64-column strips and of the 128-deep (forward) and 64-deep
(dX) steps that the 8 waves share; every element is held to the summation
bound of tests/parity_check.py against the oracle, and every expert of a
grouped call equals its single call bit for bit."""

import numpy as np
import pytest
import torch

from conftest import ensure_library, gpu_ready
from oracle import linear
from paper_2609_04526_amd import inputs
from parity_check import assert_elements
from test_gpu_gemm import TOL, abs_sums, depths, make_layer, normwise, to_dev

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def sq():
    ensure_library()
    from paper_2609_04526_amd import sq as _sq
    return _sq


def takes(T, K):
    return K > 2048 and T <= 64


def check(fmt, X, dY, codes, sb, ws2, Y, dX, what):
    Xd, dYd = X.double().numpy(), dY.double().numpy()
    W = linear.dequant(fmt, codes, sb, ws2)
    T, I = Xd.shape
    aY, adX, _ = abs_sums(fmt, Xd, dYd, codes, W)
    kY, kX, _ = depths(fmt, T, W.shape[0], I)
    for got, ref, a, k, name in ((Y, linear.forward(Xd, W), aY, kY, "Y"), (dX, linear.backward_dx(dYd, W), adX, kX, "dX")):
        assert normwise(got, ref) <= TOL
        assert_elements(got, ref, a, k, f"{what} {name}")


@pytest.mark.parametrize("fmt,T,O,I", [
    ("mx", 1, 8, 2080), ("nv", 1, 2056, 16),             # the narrowest strips, one token
    ("mx", 16, 40, 2208), ("nv", 15, 2072, 144),         # a token tile and one row less, ragged strips and steps
    ("mx", 17, 2056, 2080), ("nv", 17, 2056, 2064),      # long contractions both ways, one row over a tile
    ("mx", 33, 2064, 2176), ("nv", 33, 4104, 2096),
    ("mx", 64, 2056, 4128), ("nv", 64, 2072, 4112),      # the most tokens; NVFP4 rows ending inside a 32-code chunk
    ("nv", 48, 2080, 4224),                              # whole scale words per step
    ("mx", 64, 4096, 2048), ("nv", 64, 4096, 2048),      # dX here, the forward on tiles
])
def test_parity(sq, fmt, T, O, I):
    X, dY, codes, sb, ws2 = make_layer(fmt, T, O, I, seed=9000 + T + O)
    Xc, dYc, c, s = to_dev(X, dY, codes, sb)
    print(f"[thin] fmt={fmt} T={T} O={O} I={I}", flush=True)
    Y, dX = sq.sq_fwd(fmt, Xc, c, s, ws2), sq.sq_bwd_dx(fmt, dYc, c, s, ws2)
    check(fmt, X, dY, codes, sb, ws2, Y.cpu().numpy(), dX.cpu().numpy(), f"{fmt} {T}x{O}x{I}")
    # bf16 outputs are the fp32 ones, rounded
    assert torch.equal(sq.sq_fwd(fmt, Xc, c, s, ws2, torch.bfloat16), Y.to(torch.bfloat16))
    assert torch.equal(sq.sq_bwd_dx(fmt, dYc, c, s, ws2, torch.bfloat16), dX.to(torch.bfloat16))
    # planes at the least alignment the entry points take (codes 4 bytes, scales any)
    cb = torch.empty(codes.size + 4, dtype=torch.uint8, device="cuda")[4:].view(codes.shape)
    ub = torch.empty(sb.size + 1, dtype=torch.uint8, device="cuda")[1:].view(sb.shape)
    cb.copy_(c)
    ub.copy_(s)
    if takes(T, I):                                      # (the tiles' MXFP4 forward sums in another order there)
        assert torch.equal(sq.sq_fwd(fmt, Xc, cb, ub, ws2), Y)
    assert torch.equal(sq.sq_bwd_dx(fmt, dYc, cb, ub, ws2), dX)


@pytest.mark.parametrize("fmt", ["mx", "nv"])
@pytest.mark.parametrize("Ts,O,I", [
    ([1, 16, 17, 64, 33, 5], 2056, 2112),                # only few-token experts, mixed tiles
    ([3, 16, 0, 7], 96, 2208),
    ([1, 16, 17, 65, 64, 200, 9], 2056, 2304),           # among larger experts: a launch of their own
    ([16, 17, 300, 1, 129], 264, 512),
    ([2200, 12, 2100], 2056, 2304),                      # beside experts on the long or large tiles
])
def test_grouped_equals_single(sq, fmt, Ts, O, I):
    E = len(Ts)
    L = [make_layer(fmt, T, O, I, seed=9300 + 7 * e) for e, T in enumerate(Ts)]
    Xs, dYs = [x[0].cuda() for x in L], [x[1].cuda() for x in L]
    cs, ss = [torch.from_numpy(x[2]).cuda() for x in L], [torch.from_numpy(x[3]).cuda() for x in L]
    ws2 = [float(np.float32(x[4] / (1 + e % 2))) for e, x in enumerate(L)]
    print(f"[thin grouped] fmt={fmt} T={Ts} O={O} I={I}", flush=True)
    Ys = sq.sq_fwd_grouped(fmt, Xs, cs, ss, ws2)
    dXs = sq.sq_bwd_dx_grouped(fmt, dYs, cs, ss, ws2)
    for e in range(E):
        if Ts[e] == 0:
            continue
        assert torch.equal(Ys[e], sq.sq_fwd(fmt, Xs[e], cs[e], ss[e], ws2[e])), (e, Ts[e])
        assert torch.equal(dXs[e], sq.sq_bwd_dx(fmt, dYs[e], cs[e], ss[e], ws2[e])), (e, Ts[e])
    check(fmt, L[0][0], L[0][1], L[0][2], L[0][3], ws2[0], Ys[0].cpu().numpy(), dXs[0].cpu().numpy(), "expert 0")


def test_nan_and_infinite_inputs_stay_in_their_rows(sq):
    """A NaN scale reaches exactly its output column; an infinite activation its row."""
    fmt, T, O, I = "nv", 20, 2056, 2064
    X, dY, codes, sb, ws2 = make_layer(fmt, T, O, I, seed=9500)
    codes[5, :] = 0x22
    sb[5, -1] = 0x7F
    X[3, 17] = float("inf")
    X[3, 18:] = 1.0
    Xc, _, c, s = to_dev(X, dY, codes, sb)
    Y = sq.sq_fwd(fmt, Xc, c, s, ws2).cpu().numpy()
    bad = ~np.isfinite(Y)
    assert np.isnan(Y[:, 5]).all()
    want = np.zeros_like(bad)
    want[3, :] = True
    want[:, 5] = True
    assert (bad <= want).all() and bad[3].any()
