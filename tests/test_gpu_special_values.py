"""Special values through the matrix-core scale step, factor gradients and
re-quantiser: fp32-subnormal products, partial sums and scales, sums that cross
2^-126, bf16-subnormal factors and weights, terms of mixed magnitude (which show
any other order of the rank sum), NaN and infinities.

Factors have three mantissa bits and exponents that keep every product a whole
multiple of 2^-149, so that a product rounded on its own and one inside a fused
multiply-add are the same number, and the bytes equal the oracle's.  The shapes
take the narrow and the wide scale kernel, word and byte planes."""

import numpy as np
import pytest
import torch

from conftest import ensure_library, gpu_ready
from oracle import qast, qat
from paper_2609_04526_amd import inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def sq():
    ensure_library()
    from paper_2609_04526_amd import sq as _sq
    return _sq


def short(g, shape, lo, hi):
    """bf16 values m 2^e of random sign: m = 4 .. 7 quarters, e from lo to hi (values under
    the normal range only as far as they are exact)."""
    m = np.ldexp(g.integers(4, 8, shape).astype(np.float64), -2)
    v = np.ldexp(m, g.integers(lo, hi + 1, shape)) * g.choice([-1.0, 1.0], shape)
    t = torch.from_numpy(v.astype(np.float32)).to(torch.bfloat16)
    assert np.array_equal(t.float().numpy().astype(np.float64), v)
    return t


# name: exponents of B, of A, alpha / r
RANGES = {"subnormal products": (-72, -66, -70, -64, 1.0), "sums across 2^-126": (-68, -62, -66, -62, 1.0),
          "subnormal factors": (-131, -126, -8, 0, 1.0), "subnormal after alpha": (-60, -56, -60, -56, 2.0 ** -14),
          "mixed magnitudes": (-60, -20, -60, -20, 1.0)}


def make(fmt, O, G, seed, name):
    g = inputs.rng(seed)
    if fmt == "mx":
        lo, hi = (40, 90) if name == "mixed magnitudes" else (0, 4)
        return g, g.integers(lo, hi + 1, (O, G)).astype(np.uint8), 1.0
    ws2 = float(np.float32(2.0 ** (-60 if name == "mixed magnitudes" else -128)))
    return g, g.integers(0, 127, (O, G)).astype(np.uint8), ws2


@pytest.mark.parametrize("fmt", ["mx", "nv"])
@pytest.mark.parametrize("O,G,r", [(72, 64, 3), (200, 65, 33), (8200, 196, 24), (8200, 197, 17)])
@pytest.mark.parametrize("name", list(RANGES))
def test_scales(sq, fmt, O, G, r, name):
    print(f"[special scales] {fmt} O={O} G={G} r={r} {name}", flush=True)
    g, base, ws2 = make(fmt, O, G, 9100 + r, name)
    blo, bhi, alo, ahi, c = RANGES[name]
    B, A = short(g, (O, r), blo, bhi), short(g, (r, G), alo, ahi)
    want, mask = qast.qast_scales(fmt, base, B, A, c, ws2)
    assert not np.array_equal(want, base)
    got, mk = sq.sq_qast_scales(fmt, torch.from_numpy(base).cuda(), B.cuda(), A.cuda(), c, ws2)
    assert np.array_equal(got.cpu().numpy(), want) and np.array_equal(mk.cpu().numpy(), mask)


@pytest.mark.parametrize("fmt", ["mx", "nv"])
@pytest.mark.parametrize("O,I,r", [(72, 160, 3), (136, 416, 33), (512, 2048, 24)])
@pytest.mark.parametrize("name", list(RANGES))
def test_requant(sq, fmt, O, I, r, name):
    print(f"[special requant] {fmt} O={O} I={I} r={r} {name}", flush=True)
    g, sb, ws2 = make(fmt, O, I // (32 if fmt == "mx" else 16), 9200 + r, name)
    codes = inputs.codes_uniform(9201, O, I)
    blo, bhi, alo, ahi, c = RANGES[name]
    B, A = short(g, (O, r), blo, bhi), short(g, (r, I), alo, ahi)
    wc, ws = qat.requant(fmt, codes, sb, ws2, B, A, c)
    W = qat.effective_weight(fmt, codes, sb, ws2, B, A, c)
    if name != "mixed magnitudes":
        small = np.abs(np.asarray(W, dtype=np.float64))
        assert np.any((small > 0) & (small < 2.0 ** -126))           # bf16-subnormal weights occur
    got = sq.sq_qat_requant(fmt, torch.from_numpy(codes).cuda(), torch.from_numpy(sb).cuda(), B.cuda(), A.cuda(), c, ws2)
    assert np.array_equal(got[0].cpu().numpy(), wc) and np.array_equal(got[1].cpu().numpy(), ws)


def classes(x):
    return np.where(np.isnan(x), 3, np.where(np.isposinf(x), 1, np.where(np.isneginf(x), 2, 0)))


@pytest.mark.parametrize("fmt,O,G,r", [("mx", 40, 20, 5), ("nv", 200, 97, 33), ("mx", 8200, 196, 24), ("nv", 8200, 196, 24),
                                       ("nv", 8200, 197, 17)])
def test_nan_and_infinity(sq, fmt, O, G, r):
    """NaN and infinities stay in the rows and columns they belong to."""
    print(f"[special nan] {fmt} O={O} G={G} r={r}", flush=True)
    g = inputs.rng(9300 + r)
    B, A = short(g, (O, r), -6, 0), short(g, (r, G), -6, 0)
    B[3, 1], B[O - 1, r - 1], B[17, 0] = float("nan"), float("inf"), float("inf")
    A[0, 2], A[r - 1, G - 1] = float("nan"), float("-inf")
    base = g.integers(100, 127, (O, G)).astype(np.uint8)
    base[5, 5] = 0xFF if fmt == "mx" else 0x7F
    ws2 = 1.0 if fmt == "mx" else float(np.float32(1 / 448))
    with np.errstate(all="ignore"):
        want, mask = qast.qast_scales(fmt, base, B, A, 0.5, ws2)
    Bd, Ad = B.cuda(), A.cuda()
    got, mk = sq.sq_qast_scales(fmt, torch.from_numpy(base).cuda(), Bd, Ad, 0.5, ws2)
    assert np.array_equal(got.cpu().numpy(), want) and np.array_equal(mk.cpu().numpy(), mask)
    dS = g.standard_normal((O, G)).astype(np.float32)
    dS[5, 3], dS[O - 2, G - 1], dS[9, 0] = float("nan"), float("inf"), float("-inf")
    m = np.ones((O, G), dtype=np.uint8)
    m[20:, 1] = 0
    with np.errstate(all="ignore"):
        wB, wA = qast.factor_grads(dS, m, B, A, 0.5)
    dB, dA = sq.sq_qast_factor_grads(torch.from_numpy(dS).cuda(), torch.from_numpy(m).cuda(), Bd, Ad, 0.5)
    assert np.array_equal(classes(dB.cpu().numpy()), classes(wB))
    assert np.array_equal(classes(dA.cpu().numpy()), classes(wA))
