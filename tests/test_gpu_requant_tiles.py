"""sq_qat_requant at the edges of its 16 x 128 wave tiles and 16-rank groups:
one row or one block over a tile, NVFP4 rows ending in a lane's first block,
ranks around the group size, planes at the least alignment the entry point
takes, NaN scales and adapters, and weights that overflow to infinity.  Codes and scale bytes equal the oracle's bit for bit."""

import numpy as np
import pytest
import torch

from conftest import ensure_library, gpu_ready
from oracle import qat
from paper_2609_04526_amd import inputs
from test_gpu_qast_tiles import plane, shifted

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def sq():
    ensure_library()
    from paper_2609_04526_amd import sq as _sq
    return _sq


@pytest.mark.parametrize("fmt,O,I,r", [("mx", 16, 128, 16), ("mx", 24, 160, 17), ("nv", 72, 144, 15), ("nv", 64, 128, 33),
                                       ("mx", 8, 96, 64), ("nv", 136, 400, 48), ("nv", 8, 16, 3), ("mx", 200, 288, 4)])
def test_codes_and_scales(sq, fmt, O, I, r):
    print(f"[requant tiles] fmt={fmt} O={O} I={I} r={r}", flush=True)
    codes = inputs.codes_uniform(8800 + O, O, I)
    sb, ws2 = plane(fmt, O, I // (32 if fmt == "mx" else 16), 8801 + I)
    g = inputs.rng(8802)
    B = torch.from_numpy(g.standard_normal((O, r)).astype(np.float32) * 0.05).to(torch.bfloat16)
    A = torch.from_numpy(g.standard_normal((r, I)).astype(np.float32) * 0.05).to(torch.bfloat16)
    if O > 16:
        sb[3, 0] = 0xFF if fmt == "mx" else 0x7F                 # a NaN block
        B[9, :], A[0, :16] = 1e38, 1e30                          # weights that overflow to infinity
        A[1, 20] = float("nan")                                  # a NaN weight in every row's second block
    c = 0.75
    wc, ws = qat.requant(fmt, codes, sb, ws2, B, A, c)
    cd, sd = torch.from_numpy(codes).cuda(), torch.from_numpy(sb).cuda()
    Bd, Ad = B.cuda(), A.cuda()
    for cc, ss, bb in ((cd, sd, Bd), (shifted(cd, 4), shifted(sd, 1), shifted(Bd, 2))):
        oc, osc = torch.empty_like(cc), torch.empty_like(ss)
        got = sq.sq_qat_requant(fmt, cc, ss, bb, Ad, c, ws2, shifted(oc, 4), shifted(osc, 3))
        assert np.array_equal(got[0].cpu().numpy(), wc) and np.array_equal(got[1].cpu().numpy(), ws)
