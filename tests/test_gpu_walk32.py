"""The fp32 / fp64 segment walk (forward with fp32 inputs, or unmasked): every
width, tile remainders, one to many segments (walks that sum the records
themselves and ones that read the running sums), against the serial fp64 run.

Bar: the repository's 1e-5 row-wise bar of the fp32 path; rows are judged at
1e-5 of sum |terms| instead where the ratio's denominator is near zero (the
same rule as the other normalised tests)."""
import numpy as np
import pytest

import paper_2510_27258_amd as hla
from oracle import hla2 as O
from oracle import native
from paper_2510_27258_amd import capi
from tests.helpers import dev, gen, rowwise_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masked,normalized", [(1, 0), (1, 1), (0, 0), (0, 1)])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("n,segments", [(1, None), (32, None), (33, 2), (257, None), (320, 8), (321, 9), (1000, 32)])
def test_walk32(d, n, segments, masked, normalized, monkeypatch):
    if segments:
        monkeypatch.setenv("HLA_FUSED_SEGMENTS", str(segments))
    B, H = 1, 3
    for dist in ("scaled", "unit"):
        q, k, v, code = gen(B, H, n, d, d, dist, 11)
        print(f"walk32 d={d} n={n} segments={segments} masked={masked} normalized={normalized} {dist}", flush=True)
        eps = 1e-6
        num, den, _, _ = native.hla2_serial_c(q, k, v, masked=bool(masked), threads=8)
        out = hla.forward(dev(q, code), dev(k, code), dev(v, code), 64, masked=bool(masked),
                          normalized=bool(normalized), eps=eps, algo=capi.HLA_ALGO_CHUNKED).cpu().numpy()
        assert np.isfinite(out).all()
        if normalized:
            good = np.abs(den + eps) >= 0.05 * O.hla2_den_scale(q, k, masked=bool(masked))
            assert rowwise_err(out[good], (num / (den + eps)[..., None])[good]) <= 1e-5
        else:
            assert rowwise_err(out, num) <= 1e-5


def _plan(n, d, BH, segments, chunk, masked, normalized):
    """(P, cps): the segments of the walk and their 32-token tiles for a requested count, cut to what the workspace
    (two arrays of the general path's chunk states) holds."""
    M, F, chunks = -(-n // 32), 2 * d * d + d, -(-n // min(chunk, 64))
    room = 2 * (-(-BH * chunks * (3 * d * d + 2 * d) * 4 // 256) * 256)
    P = min(segments, M)
    while P > 1 and 4 * ((2 if P > 8 else 1) * BH * P * F + (BH * n if masked and normalized else 0)) > room:
        P -= 1
    cps = -(-M // P)
    return -(-M // cps), cps


@pytest.mark.parametrize("masked,normalized", [(1, 0), (1, 1), (0, 0), (0, 1)])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("n,segments,plan", [(2040, 8, (8, 8)), (2015, 9, (9, 7)), (2101, 22, (22, 3)),
                                             (1120, 18, (18, 2))])
def test_walk32_segments_of_several_tiles(d, n, segments, plan, masked, normalized, monkeypatch):
    """On both sides of the eight segments up to which the walk and the fix-up
    sum the records themselves; more than the sixteen records of one round of
    the running sums, their last round partly empty; segments of an odd number
    of tiles (the fix-up takes two a workgroup from d = 64 on).  fp32 inputs."""
    monkeypatch.setenv("HLA_FUSED_SEGMENTS", str(segments))
    B, H, chunk, eps = 1, 2, 16, 1e-6
    assert _plan(n, d, B * H, segments, chunk, masked, normalized) == plan
    q, k, v, code = gen(B, H, n, d, d, "scaled", 13)
    print(f"walk32 d={d} n={n} segments={segments} masked={masked} normalized={normalized}", flush=True)
    num, den, _, _ = native.hla2_serial_c(q, k, v, masked=bool(masked), threads=8)
    out = hla.forward(dev(q, code), dev(k, code), dev(v, code), chunk, masked=bool(masked),
                      normalized=bool(normalized), eps=eps, algo=capi.HLA_ALGO_CHUNKED).cpu().numpy()
    assert np.isfinite(out).all()
    if normalized:
        good = np.abs(den + eps) >= 0.05 * O.hla2_den_scale(q, k, masked=bool(masked))
        assert rowwise_err(out[good], (num / (den + eps)[..., None])[good]) <= 1e-5
    else:
        assert rowwise_err(out, num) <= 1e-5


def _distance(out, ref):
    return float(np.linalg.norm(out - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("masked", [1, 0])
@pytest.mark.parametrize("d", [64, 128])
def test_walk32_one_long_segment_keeps_its_precision(d, masked, monkeypatch):
    """4096 fp32 tokens in one segment.  A running state takes one rounding at
    its own size a tile, 128 in all: relative to its end (a sum of products of
    either sign grows as the root of the tokens) sqrt(128 / 2) times about
    0.4 * 2^-24 each, for S and for X 2.7e-7 together, and half of that again is
    allowed.  Eight roundings a tile come to 8e-7 by the same count."""
    monkeypatch.setenv("HLA_FUSED_SEGMENTS", "1")
    q, k, v, code = gen(1, 2, 4096, d, d, "scaled", 17)
    num, _, _, _ = native.hla2_serial_c(q, k, v, masked=bool(masked), threads=2)
    out = hla.forward(dev(q, code), dev(k, code), dev(v, code), 64, masked=bool(masked),
                      algo=capi.HLA_ALGO_CHUNKED).cpu().numpy()
    assert _distance(out, num) <= 4e-7


def test_walk32_bounds_unmasked_segments():
    """Unmasked, 140 equal heads of 16384 tokens at d = 128: by the head count
    one segment each, whose 512 tile sums come to 5.4e-7 (twice sqrt(512 / 2)
    0.4 * 2^-24, added in squares); segments of at most 2048 tokens keep the
    running sums of a segment and of the records below half of that each."""
    q, k, v, code = gen(1, 1, 16384, 128, 128, "scaled", 19)
    num, _, _, _ = native.hla2_serial_c(q, k, v, masked=False, threads=1)
    heads = [dev(x, code).expand(1, 140, -1, -1).contiguous() for x in (q, k, v)]
    out = hla.forward(*heads, 64, masked=False, algo=capi.HLA_ALGO_CHUNKED)
    assert bool((out == out[:, :1]).all())
    assert _distance(out[:, 0].cpu().numpy(), num[:, 0]) <= 4e-7


@pytest.mark.parametrize("d,dv,chunk", [(64, 64, 64), (128, 128, 128), (64, 32, 64), (16, 16, 16)])
def test_unmasked_by_default_algorithm(d, dv, chunk):
    """hla.forward(masked=False) without an algorithm on bf16: the workspace it
    allocates is the chunked algorithm's, which the unmasked operator takes
    (at the first three shapes the masked operator takes the fused one)."""
    q, k, v, code = gen(1, 2, 300, d, dv, "unit", 23)
    x = [dev(t, code) for t in (q, k, v)]
    num, _, _, _ = native.hla2_serial_c(q, k, v, masked=False, threads=2)
    out = hla.forward(*x, chunk, masked=False)
    assert (out == hla.forward(*x, chunk, masked=False, algo=capi.HLA_ALGO_CHUNKED)).all()
    assert rowwise_err(out.cpu().numpy(), num) <= 1e-5
