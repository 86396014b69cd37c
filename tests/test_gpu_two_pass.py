"""The two-pass plan of the d = 128 walks (second order, AHLA, prefill): the
prefixes summed by the bracket launch or by their own, brackets formed by one
workgroup or by two, one to several tiles a segment.

Besides the bf16 bar on every row the outputs of every head are held to 3.6e-6 of
the 64-bit result in norm.  Every computed operand of the walks is split into
two bf16 pieces (2^-17 of each element), which leaves 2.5-3.0e-6 at these
lengths; the brackets are formed from three, and two there come to 4.2-4.8e-6
(a product left out or misplaced among the smaller pieces costs more)."""
import math

import numpy as np
import pytest

import paper_2510_27258_amd as hla
from oracle import native
from paper_2510_27258_amd import capi
from tests.helpers import dev, gen, tol_for

pytestmark = pytest.mark.gpu

BAR = 3.6e-6
SUM_MAX, SPLIT_MAX = 17, 128     # segments summed by the bracket launch; (segment, head) pairs of two workgroups


def _plan(BH, n, segments, ratio=0.65):
    """(segments, tiles of a later segment) of the plan; ratio: a summary tile's time over an output tile's."""
    M, Q = -(-n // 64), segments - 1 if segments else 256 // BH
    if Q >= 2 and M >= 3:
        x = math.ceil(M / (Q + ratio))
        rest = M - max(1, int(ratio * x + 0.5))
        if rest > 0:
            x = max(x, -(-rest // Q))
            if -(-rest // x) >= 2:
                return 1 + -(-rest // x), x
    return 1, M


def _inputs(BH, n, normalized, seed):
    q, k, v, code = gen(1, BH, n, 128, 128, "unit", seed)
    if normalized:               # non-negative q and k keep the denominators away from zero
        q, k = np.abs(q), np.abs(k)
    return q, k, v, code


def _close(out, ref, code):
    # row 0 of a head is (q.k)^2 v: r_0 = (q.k) k is rounded at 2^-17 of its size, so (q.k)^2 = q.r_0 keeps an error of
    # 2^-17 |q.k| and the row a relative one of 2^-17 / |q.k|, over the bar where q.k < 4e-3 (one in thirty first rows
    # at d = 128, whose q.k are N(0, 1/128)).  Rows below their head's mean size are therefore held to that size.
    size = np.maximum(np.abs(ref).max(-1), np.sqrt((ref ** 2).mean((2, 3)))[..., None])
    assert (np.abs(out - ref).max(-1) / size).max() <= tol_for(code)
    off = np.linalg.norm(out - ref, axis=(2, 3)) / np.linalg.norm(ref, axis=(2, 3))
    assert off.max() <= BAR, off


def _branch(BH, n, segments, monkeypatch, ratio=0.65):
    """The plan, and whether its prefixes have their own launch and a bracket two workgroups."""
    if segments:
        monkeypatch.setenv("HLA_FUSED_SEGMENTS", str(segments))
    P, cps = _plan(BH, n, segments, ratio)
    return P, cps, P > SUM_MAX, BH * (P - 1) <= SPLIT_MAX


@pytest.mark.parametrize("normalized", [0, 1])
@pytest.mark.parametrize("BH,n,segments,P,cps,own_launch,split", [
    (2, 1900, 13, 11, 3, False, True), (3, 3600, 20, 20, 3, True, True),
    (9, 1900, 24, 16, 2, False, False), (6, 2000, 0, 32, 1, True, False)])
def test_forward(BH, n, segments, P, cps, own_launch, split, normalized, monkeypatch):
    assert _branch(BH, n, segments, monkeypatch) == (P, cps, own_launch, split)
    assert capi.hla2_fused_plan(1, BH, n, 128, 128, 128)[0] == P
    q, k, v, code = _inputs(BH, n, normalized, 31)
    print(f"two-pass forward BH={BH} n={n} P={P} normalized={normalized}", flush=True)
    num, den, _, _ = native.hla2_serial_c(q, k, v, masked=True, threads=8)
    out = hla.forward(*(dev(x, code) for x in (q, k, v)), 128, normalized=bool(normalized), eps=1e-6).cpu().numpy()
    _close(out, num / (den + 1e-6)[..., None] if normalized else num, code)


@pytest.mark.parametrize("BH,n,segments,normalized,P,cps,own_launch,split", [
    (2, 3300, 12, 0, 11, 5, False, True), (2, 3300, 12, 1, 11, 5, False, True), (3, 3600, 20, 1, 20, 3, True, True),
    (13, 2000, 12, 1, 11, 3, False, False), (17, 2900, 10, 0, 10, 5, False, False),
    (2, 3000, 0, 0, 47, 1, True, True), (2, 3000, 0, 1, 47, 1, True, True), (4, 3000, 0, 1, 47, 1, True, False),
    (6, 4000, 0, 0, 32, 2, True, False), (2, 3000, 26, 1, 24, 2, True, True)])
def test_ahla(BH, n, segments, normalized, P, cps, own_launch, split, monkeypatch):
    """Plans that take the two passes: five tiles a segment, three when
    normalised, or many segments of one or two."""
    assert _branch(BH, n, segments, monkeypatch, 0.75) == (P, cps, own_launch, split)
    assert cps >= (3 if normalized else 5) or P > 46 or (cps == 2 and P > (23 if normalized else 31))
    q, k, v, code = _inputs(BH, n, normalized, 37)
    print(f"two-pass ahla BH={BH} n={n} P={P} normalized={normalized}", flush=True)
    num, den, _ = native.ahla_serial_c(q, k, v, threads=8)
    out = hla.ahla_forward(*(dev(x, code) for x in (q, k, v)), 128, normalized=bool(normalized), eps=1e-6).cpu().numpy()
    _close(out, num / (den + 1e-6)[..., None] if normalized else num, code)


@pytest.mark.parametrize("BH,pieces", [(2, (1500, 1337)), (12, (1900, 700))])
def test_chained_prefill(BH, pieces):
    """Outputs and the state's record as a whole, two calls."""
    n = sum(pieces)
    q, k, v, code = _inputs(BH, n, False, 41)
    num, _, fin, _ = native.hla2_serial_c(q, k, v, masked=True, threads=8)
    state, outs, a = hla.State(1, BH, 128, 128), [], 0
    for p in pieces:
        print(f"two-pass prefill BH={BH} n={p} at {a} P={_plan(BH, p, 0)[0]}", flush=True)
        outs.append(hla.prefill(state, *(dev(x[:, :, a:a + p], code) for x in (q, k, v)), 128).cpu().numpy())
        a += p
    _close(np.concatenate(outs, 2), num, code)
    got = state.export().cpu().numpy().astype(np.float64)
    ref = np.concatenate([np.asarray(x).reshape(1, BH, -1) for x in fin], 2)
    assert (np.linalg.norm(got - ref, axis=2) / np.linalg.norm(ref, axis=2)).max() <= BAR
