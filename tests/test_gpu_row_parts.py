"""The pipelined kernel runs blocks of 128 query rows with 64 rows per wave on
small grids and with 128 on large ones; both give the same results.  Small
grids are compared with the oracle elsewhere: here a large grid (640 blocks of
ragged, windowed or grouped sequences) is compared with its first and last
sequence alone, which take the 64-row form.  Every value has to be equal: the
masks are decisions, lse and O come from the same operations in the same
order."""
import math

import pytest
import torch

from paper_2609_39361_amd import workloads as W

pytestmark = pytest.mark.gpu

SIM = 4


@pytest.fixture(scope="module")
def L():
    from paper_2609_39361_amd import lamp
    lamp.init(0)
    return lamp


@pytest.mark.parametrize("tau", [math.inf, 0.5, 2.0 ** -5, 0.0])
@pytest.mark.parametrize("d,N,causal,window,flags,seed", [
    (128, 1, 1, 0, 0, None), (128, 130, 1, 0, 0, None), (128, 333, 0, 0, 0, None), (128, 300, 1, 70, 0, None),
    (64, 130, 1, 0, 0, None), (64, 200, 0, 0, 0, None), (64, 300, 1, 70, 0, None), (64, 140, 1, 0, 0, 11),
    (256, 200, 1, 0, 0, None), (256, 257, 1, 100, 0, None), (128, 200, 1, 0, SIM, None), (256, 140, 0, 0, SIM, None),
    (128, 200, 1, 0, 1, None), (128, 200, 1, 0, 2, None), (128, 140, 1, 0, 0, 11)])
def test_large_grid_equals_its_parts(L, d, N, causal, window, flags, seed, tau):
    w = W.small(B=8, Hq=80, Hkv=8, N=N, d=d, causal=causal, window=window, bq=128, bk=16, nk=4, seed=N + d)
    q, k, v = (t.cuda() for t in W.make_inputs(w))
    kw = dict(causal=bool(causal), window=window, tau=tau, flags=flags, sr_seed=seed)
    o, lse, mask = L.attn_fwd(q, k, v, **kw)
    torch.cuda.synchronize()
    # the random numbers of stochastic rounding depend on the sequence's index
    for b in (0,) if seed is not None else (0, 7):
        po, pl, pm = L.attn_fwd(q[b:b + 1].contiguous(), k[b:b + 1].contiguous(), v[b:b + 1].contiguous(), **kw)
        torch.cuda.synchronize()
        assert torch.equal(mask[b], pm[0])
        assert torch.equal(lse[b], pl[0])
        assert torch.equal(o[b], po[0]), float((o[b] - po[0]).abs().max())
