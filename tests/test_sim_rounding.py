"""The two-operation rounding of the simulation profile's 8-bit loop: c1 t
rounded to FP32, then c2 t added exactly, equals round-to-nearest-even of the
FP32 pattern to 3 stored mantissa bits for every significand and both signs
(the operations scale with the exponent, so three exponents stand for the range
in between)."""
import numpy as np
import pytest


def _rn3(bits):
    return ((bits + 0x7FFFF + ((bits >> 20) & 1)) & 0xFFF00000).astype(np.uint32)


@pytest.mark.parametrize("exponent", [-126, 0, 106])
@pytest.mark.parametrize("sign", [0, 1])
def test_two_operation_rounding(exponent, sign):
    m = np.arange(1 << 23, dtype=np.uint64)
    bits = (m | ((exponent + 127) << 23) | (sign << 31)).astype(np.uint64)
    t = bits.astype(np.uint32).view(np.float32)
    c1, c2 = np.float32(-1048575.0), np.float64(1048576.0)
    s = (t * c1).astype(np.float32)                 # one rounding
    got = (t.astype(np.float64) * c2 + s.astype(np.float64)).astype(np.float32)   # exact in fp64: one rounding, as fma
    assert np.array_equal(got.view(np.uint32), _rn3(bits))
