"""The forward pass in the simulation profile at the ends of FP32's range,
against the oracle: logits so small that the 8-bit loop leaves the range of its
fast rounding (the pass that finds out also holds 16-bit sums, and the wave's
later ones take the exact rounding), logits beyond it, and logits far below
every finite number a hardware format knows.  The decisions compare logits on
their own scale, so masks show a misrounded one."""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

SIM = 4
KINDS = ["tiny_tiles", "tiny_first", "huge_tiles", "far_below", "far_below_mixed", "subnormal"]


@pytest.fixture(scope="module")
def L():
    from paper_2609_39361_amd import lamp
    lamp.init(0)
    return lamp


def _inputs(kind, B, Hq, Hkv, N, d, seed):
    """Channels in two halves: `a` of ordinary queries (positive) and `t` of tiny
    ones; the key tiles (64 keys) use one half each, so that a tile's logits
    are negative and ordinary, or of either sign and tiny."""
    g = torch.Generator("cpu")
    g.manual_seed(seed)

    def n(*s):
        return torch.randn(s, generator=g)

    q, k, v = n(B, Hq, N, d), n(B, Hkv, N, d), n(B, Hkv, N, d)
    h = d // 2
    tile = torch.arange(N) // 64

    def rows(t, sel, lo, hi, scale):
        t[:, :, sel, lo:hi] = t[:, :, sel, lo:hi] * scale

    q[..., :h] = q[..., :h].abs() * 0.25 + 0.0625
    if kind in ("tiny_tiles", "tiny_first"):
        # ordinary negative logits, then tiny ones above them (the margin tests
        # fail tile by tile), then ordinary again
        tiny = (tile % 3 == 1) if kind == "tiny_tiles" else (tile < 2)
        q[..., h:] *= 2.0 ** -62
        k[..., :h] = -k[..., :h].abs() * 0.25 - 0.0625
        rows(k, tiny, 0, h, 0.0)
        rows(k, tiny, h, d, 2.0 ** -60)
        rows(k, ~tiny, h, d, 0.0)
    elif kind == "huge_tiles":
        # tiles whose products pass 2^107 between ordinary ones
        q[..., :h] *= 2.0 ** 50
        q[..., h:] = 0.0
        rows(k, tile % 3 == 1, 0, h, 2.0 ** 60)
        rows(k, tile % 3 != 1, 0, h, 2.0 ** -52)
    elif kind == "far_below":
        # every logit between -2^100 and -2^106
        q = q.abs() * 2.0 ** 50 + 2.0 ** 48
        k = -(k.abs() * 2.0 ** 50 + 2.0 ** 48)
    elif kind == "far_below_mixed":
        # the running maximum rises from below -2^100 to ordinary logits
        q = q.abs() + 0.25
        k = -(k.abs() + 0.25)
        rows(k, tile < 3, 0, d, 2.0 ** 101)
    elif kind == "subnormal":
        # every logit around 2^-124, its first partial sums FP32 subnormals
        q, k = n(B, Hq, N, d) * 2.0 ** -62, n(B, Hkv, N, d) * 2.0 ** -61
    return q.to(torch.bfloat16), k.to(torch.bfloat16), v.to(torch.bfloat16)


def _close(a, ref, rel):
    return np.all(np.abs(a - ref) <= rel * np.maximum(np.abs(ref), 1.0))


@pytest.mark.parametrize("tau", [math.inf, 0.5, 2.0 ** -5, 0.0])
@pytest.mark.parametrize("d,bq,N", [(128, 128, 330), (128, 64, 250), (256, 128, 256)])
@pytest.mark.parametrize("kind", KINDS)
def test_sim_forward_at_the_ends_of_fp32(L, kind, d, bq, N, tau):
    q, k, v = _inputs(kind, 1, 2, 1, N, d, seed=N + d)
    o, lse, mask = L.attn_fwd(q.cuda(), k.cuda(), v.cuda(), True, 0, bq, 16, 4, 2.0 ** -8, tau, flags=SIM)
    torch.cuda.synchronize()
    ro, rlse, rmask = O.fwd(O.bf16_bits(q), O.bf16_bits(k), O.bf16_bits(v), 1, 0, bq, 16, 4, 2.0 ** -8, tau, flags=SIM)
    assert np.isfinite(ro).all() and np.isfinite(rlse).all()
    got = mask.cpu().numpy()
    assert np.array_equal(got, rmask), "%d of %d mask bytes differ" % ((got != rmask).sum(), rmask.size)
    assert np.abs(o.cpu().numpy() - ro).max() <= 2e-3 * np.abs(ro).max()
    # lse = mu + ln omega in fp32: half an ulp of it beside the stated 1e-4
    assert _close(lse.cpu().numpy(), rlse, 1e-4)


@pytest.mark.parametrize("tau", [math.inf, 0.5])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("d", [128, 256])
def test_sim_large_grid_equals_its_parts(L, kind, d, tau):
    """640 blocks take 128 query rows per wave, one sequence alone 64."""
    q, k, v = (t.cuda() for t in _inputs(kind, 8, 80, 8, 200, d, seed=d))
    big = L.attn_fwd(q, k, v, tau=tau, flags=SIM)
    for b in (0, 7):
        part = L.attn_fwd(q[b:b + 1].contiguous(), k[b:b + 1].contiguous(), v[b:b + 1].contiguous(), tau=tau, flags=SIM)
        torch.cuda.synchronize()
        assert all(torch.equal(x[b], y[0]) for x, y in zip(big, part))
