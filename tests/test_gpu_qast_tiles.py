"""The QAST kernels at the edges of their 16 x 16 matrix-core blocks: ranks on
both sides of the 4-, 16- and 32-rank steps, planes narrower than a block, one
column over a wave's or a workgroup's tile, rows that end inside a block, and
planes at the least alignment the entry points take.  Scale bytes and masks
equal the oracle's bit for bit; every factor gradient is within the fp32
summation bound (tests/parity_check.py)."""

import numpy as np
import pytest
import torch

from conftest import ensure_library, gpu_ready
from oracle import qast
from paper_2609_04526_amd import inputs
from parity_check import assert_elements
from test_gpu_qast import factors, plane

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def sq():
    ensure_library()
    from paper_2609_04526_amd import sq as _sq
    return _sq


def shifted(t, nbytes):
    """A copy of t whose first byte sits nbytes past an aligned address."""
    raw = torch.empty(t.numel() * t.element_size() + nbytes, dtype=torch.uint8, device="cuda")
    v = raw[nbytes:].view(t.dtype).view(t.shape)
    v.copy_(t)
    return v


CASES = [("mx", 8, 1, 1), ("nv", 15, 15, 2), ("mx", 16, 16, 4), ("nv", 17, 17, 5), ("mx", 63, 32, 16), ("nv", 65, 33, 17),
         ("mx", 64, 48, 33), ("nv", 128, 64, 64), ("mx", 129, 65, 58), ("nv", 40, 80, 34),
         # enough 16 x 16 blocks for the wide kernel at ranks 8 (6144), 2 (12,288) and 1 to a load (24,576 up to rank 8)
         ("nv", 8200, 196, 24), ("mx", 8200, 197, 64), ("mx", 28200, 97, 30), ("nv", 12300, 252, 58), ("mx", 12300, 256, 61),
         ("nv", 24600, 256, 7),
         # and launches that stay on the narrow one
         ("mx", 16400, 97, 30), ("nv", 49200, 20, 7), ("nv", 8200, 197, 63), ("mx", 8200, 196, 61), ("nv", 28200, 97, 5),
         ("mx", 8200, 196, 64), ("nv", 100, 1000, 40), ("mx", 120, 13201, 3),
         # narrow, factors through LDS by 8, 2 and 1 (over 512 workgroups), and a rank per load beside them
         ("mx", 8192, 130, 48), ("nv", 8192, 130, 20), ("mx", 8192, 130, 41), ("nv", 8192, 130, 19),
         # dA columns in runs (narrow dS rows, 4096 workgroups and more), both column counts
         ("nv", 1100, 16001, 5), ("mx", 1100, 8001, 40)]


@pytest.mark.parametrize("fmt,O,G,r", CASES)
def test_scales_and_gradients(sq, fmt, O, G, r):
    print(f"[qast tiles] fmt={fmt} O={O} G={G} r={r}", flush=True)
    base, ws2 = plane(fmt, O, G, 7700 + O + G)
    B, A = factors(fmt, base, ws2, r, 7701 + r, push=3.0 if r < 20 else 30.0)
    c = 0.5
    want, mask = qast.qast_scales(fmt, base, B, A, c, ws2)
    bd, Bd, Ad = torch.from_numpy(base).cuda(), B.cuda(), A.cuda()
    g = inputs.rng(7702)
    dS = g.standard_normal((O, G)).astype(np.float32)
    m = (g.random((O, G)) > 0.3).astype(np.uint8)
    dd, md = torch.from_numpy(dS).cuda(), torch.from_numpy(m).cuda()
    wB, wA = qast.factor_grads(dS, m, B, A, c)
    aB, aA = qast.factor_grads(np.abs(dS), m, B.abs(), A.abs(), c)
    got = []
    for low in (False, True):
        b, Bx, Ax, d, mm = ((shifted(bd, 1), shifted(Bd, 2), shifted(Ad, 2), shifted(dd, 4), shifted(md, 1)) if low
                            else (bd, Bd, Ad, dd, md))
        out, mk = sq.sq_qast_scales(fmt, b, Bx, Ax, c, ws2)
        assert np.array_equal(out.cpu().numpy(), want) and np.array_equal(mk.cpu().numpy(), mask)
        dB, dA = sq.sq_qast_factor_grads(d, mm, Bx, Ax, c)
        assert_elements(dB.cpu().numpy(), wB, aB, G + 2, "dB")
        assert_elements(dA.cpu().numpy(), wA, aA, O + 2, "dA")
        got.append((dB, dA))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])   # one order for every alignment
