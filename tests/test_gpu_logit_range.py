"""The logit loops at the ends of FP32's range, where the rank-1 matrix
instructions have to round and underflow exactly as the scalar FMA does:
subnormal products, exponents spread over the whole range, signed zeros,
products far beyond the 8-bit format, and lengths and head dimensions at the
edges of the loops' 16-key and 16-channel blocks.  Bit-exact against the
oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2609_39361_amd import lamp
    lamp.lib()
    return lamp


def _inputs(kind, N, d, seed):
    g = torch.Generator("cpu")
    g.manual_seed(seed)
    q, k = torch.randn((1, 2, N, d), generator=g), torch.randn((1, 1, N, d), generator=g)

    def spread(t, lo, hi):
        return t * torch.exp2(torch.randint(lo, hi + 1, t.shape, generator=g).float())

    if kind == "subnormal":      # products around 2^-132: FP32 subnormals
        q, k = q * 2.0 ** -66, k * 2.0 ** -66
    elif kind == "underflow":    # exponents from far below FP32's range up to 1
        q, k = spread(q, -75, 0), spread(k, -75, 0)
    elif kind == "edge":         # subnormal, then ordinary and cancelling channels
        q, k = spread(q, -64, 0), k.clone()
        k[..., 1::2] = k[..., ::2]
        q[..., 1::2] = -q[..., ::2]
        q[..., d // 2:] *= 2.0 ** -63
        k[..., d // 2:] *= 2.0 ** -63
    elif kind == "zeros":        # signed zeros beside ordinary values
        q[torch.rand(q.shape, generator=g) < 0.5] = -0.0
        k[torch.rand(k.shape, generator=g) < 0.5] = 0.0
    elif kind == "large":        # products beyond 2^108, sums finite
        q, k = spread(q, 40, 58), spread(k, 40, 58)
    return q.to(torch.bfloat16), k.to(torch.bfloat16)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("N", [16, 80])
@pytest.mark.parametrize("kind", ["subnormal", "underflow", "edge", "zeros", "large"])
def test_logits_at_the_ends_of_fp32(L, kind, N, d):
    q, k = _inputs(kind, N, d, seed=N + d)
    qb, kb, qg, kg = O.bf16_bits(q), O.bf16_bits(k), q.cuda(), k.cuda()
    for high in (0, 1):
        ref = O.logits_sim(qb, kb, 0, 0, 0, N, high)
        got = L.logits_sim(qg, kg, high, 0, 0, 0, N).cpu().numpy().astype(np.float64)
        assert np.isfinite(ref).all()
        assert np.array_equal(got, ref) and np.array_equal(np.signbit(got), np.signbit(ref)), \
            "%s high=%d: %d values differ" % (kind, high, (got != ref).sum())
    y8 = L.logits8(qg, kg, 0, 0, 0, N).cpu().numpy()
    assert np.array_equal(y8, O.logits8(qb, kb, 0, 0, 0, N))
    y16 = L.logits16(qg, kg, 0, 0, 0, N).cpu().numpy().view(np.uint16)
    assert np.array_equal(y16, O.logits16(qb, kb, 0, 0, 0, N))
