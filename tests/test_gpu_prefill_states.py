"""Prefill from and into a decode state: the conversions between the packed
record and the walks' (S, C, m, Phi, eta) form and the walks from a carry,
over every shape of the fused path, against one serial fp64 run.

States are compared with the sums' own scale: fp32 storage and sums of bf16
products (2^-16 per computed operand) over a few hundred tokens, 1e-4 of the
field's largest value, as the other state tests of this repository."""
import numpy as np
import pytest
import torch

import paper_2510_27258_amd as hla
from oracle import hla2 as O
from oracle import native
from tests.helpers import dev, gen, rowwise_err, tol_for

pytestmark = pytest.mark.gpu


def _chain(B, H, pieces, d, dv, chunk, normalized, seed):
    n = sum(pieces)
    q, k, v, code = gen(B, H, n, d, dv, "unit", seed)
    eps = 0.5 if normalized else 1e-6
    num, den, fin, _ = native.hla2_serial_c(q, k, v, masked=True, threads=8)
    state = hla.State(B, H, d, dv, normalized=bool(normalized), eps=eps)
    outs, a = [], 0
    for p in pieces:
        print(f"prefill B={B} H={H} n={p} at {a} d={d} dv={dv} chunk={chunk} normalized={normalized}", flush=True)
        outs.append(hla.prefill(state, *(dev(x[:, :, a:a + p], code) for x in (q, k, v)), chunk).cpu().numpy())
        a += p
    got = np.concatenate(outs, 2)
    ref = num
    good = np.ones(den.shape, bool)
    if normalized:
        ref = num / (den + eps)[..., None]
        good = np.abs(den + eps) >= 0.05 * O.hla2_den_scale(q, k)
    if B * H > 16:
        # q.k of some row is far below |q||k| (row 0 is (q.k)^2 v), while the operands that form it are rounded at
        # 2^-17 of |q||r|: over thousands of first rows such a row keeps absolute accuracy only, so rows are held to
        # the size of their head's rows (root mean square) where that is larger
        size = np.sqrt((ref ** 2).mean((2, 3), keepdims=True)) + 0 * ref[..., :1]
        ref_max = np.maximum(np.abs(ref).max(-1), size[..., 0])
        assert (np.abs(got - ref).max(-1) / ref_max)[good].max() <= tol_for(code)
    else:
        assert rowwise_err(got[good], ref[good]) <= tol_for(code)
    for g, e in zip(hla.split_state(state.export(), d, dv), fin):
        e = np.asarray(e)
        assert np.abs(g.cpu().numpy().astype(np.float64) - e).max() <= 1e-4 * np.abs(e).max()


@pytest.mark.parametrize("normalized", [0, 1])
@pytest.mark.parametrize("chunk,d,dv", [(32, 32, 32), (64, 32, 64), (64, 64, 32), (64, 64, 64), (32, 128, 128),
                                        (64, 128, 128)])
def test_chained_prefill(chunk, d, dv, normalized):
    _chain(1, 3, (1, 130, 64, 333), d, dv, chunk, normalized, 3)


@pytest.mark.parametrize("normalized", [0, 1])
@pytest.mark.parametrize("BH,pieces", [((1, 1), (1, 40, 700)), ((2, 3), (64, 129, 1000)), ((2, 64), (300, 150)),
                                       ((5, 40), (70, 200))])
def test_chained_prefill_two_pass(BH, pieces, normalized):
    """d = 128 with outputs: many segments a head, two, and one (128 and 200
    heads: fewer than two walks a head in a launch), pieces of one token, one
    tile and ragged ones."""
    _chain(*BH, pieces, 128, 128, 128, normalized, 5)


@pytest.mark.parametrize("segments", [2, 3, 5])
def test_two_pass_prefill_segments(segments, monkeypatch):
    monkeypatch.setenv("HLA_FUSED_SEGMENTS", str(segments))
    _chain(1, 2, (321, 64, 500), 128, 128, 64, 0, 7)
