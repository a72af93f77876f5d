"""Sliding windows at and beyond the sequence, up to the largest int: the call
is the one without a window, whatever arithmetic the kernels do on it."""
import math

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2609_39361_amd import workloads as W

pytestmark = pytest.mark.gpu

SIM = 4
INT_MAX = 2 ** 31 - 1


@pytest.fixture(scope="module")
def L():
    from paper_2609_39361_amd import lamp
    lamp.init(0)
    return lamp


def _equal(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("tau", [math.inf, 0.5, 0.0])
@pytest.mark.parametrize("d,bq,bk,flags,seed", [(128, 128, 16, 0, None), (64, 64, 16, 0, None), (256, 128, 16, SIM, None),
                                                (128, 128, 16, 0, 5), (128, 128, 64, 0, None), (64, 64, 64, 0, None)])
def test_window_beyond_the_sequence(L, d, bq, bk, flags, seed, tau):
    N = 300
    w = W.small("wl", B=1, Hq=2, Hkv=1, N=N, d=d, causal=1, bq=bq, bk=bk, nk=4, seed=900 + d)
    q, k, v = W.make_inputs(w)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    kw = dict(causal=True, bq=bq, bk=bk, nk=4, tau=tau, flags=flags, sr_seed=seed)
    ref = L.attn_fwd(qd, kd, vd, window=0, **kw)
    ro, rlse, rmask = O.fwd(O.bf16_bits(q), O.bf16_bits(k), O.bf16_bits(v), 1, INT_MAX, bq, bk, 4, w.delta, tau,
                            flags=flags | (O.SR8 if seed is not None else 0), seed=seed or 0)
    assert np.isfinite(ro).all() and np.isfinite(rlse).all()
    for window in (N, N + 1, INT_MAX - N, INT_MAX - 62, INT_MAX):
        got = L.attn_fwd(qd, kd, vd, window=window, **kw)
        torch.cuda.synchronize()
        assert _equal(got, ref), "window %d" % window
        assert np.array_equal(got[2].cpu().numpy(), rmask)
        assert np.abs(got[0].cpu().numpy() - ro).max() <= 2e-3 * np.abs(ro).max()
        assert np.abs(got[1].cpu().numpy() - rlse).max() <= 1e-4


def test_window_beyond_the_sequence_large_grid(L):
    w = W.small("wg", B=8, Hq=80, Hkv=8, N=140, d=128, causal=1, bq=128, bk=16, nk=4, seed=911)
    q, k, v = (t.cuda() for t in W.make_inputs(w))
    assert _equal(L.attn_fwd(q, k, v, window=INT_MAX), L.attn_fwd(q, k, v))


def test_window_beyond_the_cache_decode_and_logits(L):
    w = W.small("wd", B=2, Hq=4, Hkv=2, N=2500, d=128, M=2, causal=1, bq=1, bk=64, nk=1, seed=912)
    q, k, v = (t.cuda() for t in W.make_inputs(w))
    assert _equal(L.attn_decode(q, k, v, window=INT_MAX), L.attn_decode(q, k, v))
    w = W.small("wy", B=1, Hq=2, Hkv=1, N=96, d=64, causal=1, seed=913)
    q, k, v = (t.cuda() for t in W.make_inputs(w))
    for f in (L.logits8, L.logits16, lambda a, b, **kw: L.logits_sim(a, b, 0, **kw).view(torch.int32)):
        assert torch.equal(f(q, k, causal=True, window=INT_MAX), f(q, k, causal=True, window=0))
