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
    assert rowwise_err(got[good], ref[good]) <= tol_for(code)
    for g, e in zip(hla.split_state(state.export(), d, dv), fin):
        e = np.asarray(e)
        assert np.abs(g.cpu().numpy().astype(np.float64) - e).max() <= 1e-4 * np.abs(e).max()


@pytest.mark.parametrize("normalized", [0, 1])
@pytest.mark.parametrize("chunk,d,dv", [(32, 32, 32), (64, 32, 64), (64, 64, 32), (64, 64, 64), (32, 128, 128),
                                        (64, 128, 128)])
def test_chained_prefill(chunk, d, dv, normalized):
    _chain(1, 3, (1, 130, 64, 333), d, dv, chunk, normalized, 3)
