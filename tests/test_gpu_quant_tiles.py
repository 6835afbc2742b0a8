"""GPU parity of the transposing quantizer tiles around the sizes where their
shape changes: at and just above 16 MiB (16 or 32 column groups per tile, four or
sixteen groups per max-pass thread), the smallest INT4 tiles (one trip of loads,
taken before the partial maxima are folded), fewer rows than a tile, column groups
and rows that fill the last tile partly.  Codes of both layouts, alpha and scales
are bit-exact against the oracle.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402
from oracle import luq as oluq, int4 as oint4  # noqa: E402
from gpu_util import announce, assert_codes_equal, host, to_dev, transpose_codes  # noqa: E402

SHAPES = [
    (8, 8, "f32"),          # one item
    (8, 1000, "f32"),       # one row block, a partial column tile
    (1184, 1000, "bf16"),   # partial tiles both ways
    (264, 2056, "f32"),     # INT4 tiles of 512 words, one column group over
    (2048, 2048, "f32"),    # 16 MiB exactly
    (2056, 2048, "f32"),    # just above
    (4096, 2048, "bf16"),   # 16 MiB exactly
    (4096, 2056, "bf16"),   # just above
    (70000, 8, "f32"),      # one column group: narrow tiles
]


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_10769_amd as lib
    return lib


def _tensor(rows, cols, dtype, seed, signed=True):
    x = synth.lognormal_grad((rows, cols), -10.0, 2.5, 0.3, [seed, rows, cols])
    x = x if signed else np.abs(x)
    if dtype == "f32":
        return x, x
    bits = synth.to_bf16_bits(x)
    return bits, synth.bf16_bits_to_f32(bits)


@pytest.mark.parametrize("rows,cols,dtype", SHAPES)
def test_luq_tiles(L, rows, cols, dtype):
    dev, ref = _tensor(rows, cols, dtype, 1)
    announce("luq tiles", rows, cols, dtype)
    c, ct, alpha, mx = L.luq_quantize_grad(to_dev(dev), R=4, seed=9, counter=2, codes=True, codes_t=True)
    rc, ra, rm = oluq.luq_quantize(ref, R=4, seed=9, counter=2)
    assert host(alpha)[0].tobytes() == np.float32(ra).tobytes()
    assert host(mx)[0].tobytes() == np.float32(rm).tobytes()
    assert_codes_equal(host(c)[0], rc[0], "codes")
    assert_codes_equal(host(ct)[0], transpose_codes(rc[0], rows, cols), "codes_t")


@pytest.mark.parametrize("rows,cols,dtype", SHAPES)
@pytest.mark.parametrize("signed", [True, False])
def test_int4_tiles(L, rows, cols, dtype, signed):
    dev, ref = _tensor(rows, cols, dtype, 2, signed)
    announce("int4 tiles", rows, cols, dtype, signed)
    c, ct, s = L.int4_quantize(to_dev(dev), is_signed=signed, codes=True, codes_t=True)
    rc, rs = oint4.int4_quantize(ref, is_signed=signed)
    assert host(s)[0].tobytes() == np.float32(rs).tobytes()
    assert_codes_equal(host(c), rc, "codes")
    assert_codes_equal(host(ct), transpose_codes(rc, rows, cols), "codes_t")


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_int4_tiles_nonfinite_and_zero(L, value):
    """A non-finite element (codes 0, scale NaN) and an all-zero tensor, in the
    tile whose first trip is loaded before the maximum is known."""
    x = np.ones((264, 2056), np.float32)
    x[263, 2055] = value
    announce("int4 tiles nonfinite", value)
    _, ct, s = L.int4_quantize(to_dev(x), codes=False, codes_t=True)
    assert np.isnan(host(s)[0]) and not host(ct).any()
    _, ct, s = L.int4_quantize(to_dev(np.zeros_like(x)), codes=False, codes_t=True)
    assert host(s)[0] == 0.0 and not host(ct).any()
