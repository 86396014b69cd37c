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
