"""GPU parity of the forward kernels' own observables, through the C ABI.

* the 8-bit logit codes the forward kernel computes (Alg. 1, low-precision
  accumulation; Sec. 4.1 recursion), and the 16-bit codes of the sub-blocks it
  recomputes, written by the kernel for observed query blocks, against the
  oracle's logits byte for byte;
* the instantiation that writes them gives bit-identical O, lse, mask and
  statistics to the one that does not (the one the benchmark times);
* the statistics words (stage counts, tile histogram, saturated 8-bit and
  16-bit logits) against the oracle's, exactly;
* the non-finite input check and the caller-provided workspace.
"""
import math
import sys

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2609_39361_amd import workloads as W

pytestmark = pytest.mark.gpu


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_39361_amd import lamp
    lamp.init(0)
    return lamp


def _dev(w, seed_kind=None):
    q, k, v = W.make_inputs(w)
    return q, k, v, q.cuda(), k.cuda(), v.cuda()


def _check_observables(L, w, tau, qb0, nqb, heads=None, flags=0, sr_seed=None, q=None):
    """Run the observed kernel, compare its logits with the oracle's on the
    observed blocks of `heads` ((b, h) pairs; all by default), and return the
    observed run's outputs."""
    if q is None:
        q, k, v, qd, kd, vd = _dev(w)
    else:
        q, k, v, qd, kd, vd = q
    o, lse, mask, y8, y16 = L.observe_logits(qd, kd, vd, qb0, nqb, w.causal, w.window, w.bq, w.bk, w.nk, w.delta,
                                             tau, flags=flags, sr_seed=sr_seed)
    torch.cuda.synchronize()
    N, bq, nk, bk = w.N, w.bq, w.nk, w.bk
    Nt = -(-N // (bk * nk)) * bk * nk
    r0 = qb0 * bq
    nrows = min(nqb * bq, N - r0)
    if heads is None:
        heads = [(b, h) for b in range(w.B) for h in range(w.Hq)]
    qb_bits, kb_bits = O.bf16_bits(q), O.bf16_bits(k)
    G = w.Hq // w.Hkv
    m = mask.cpu().numpy()
    for b, h in heads:
        qh = qb_bits[b:b + 1, h:h + 1]
        kh = kb_bits[b:b + 1, h // G:h // G + 1]
        g8 = y8[b, h].cpu().numpy()
        g16 = y16[b, h].cpu().numpy().view(np.uint16)
        # rows of the observed blocks beyond N are never visible
        assert np.all(g8[nrows:] == 0xFF) and np.all(g16[nrows:] == 0xFFFF)
        g8, g16 = g8[:nrows], g16[:nrows]
        assert np.all(g8[:, N:] == 0xFF) and np.all(g16[:, N:] == 0xFFFF)
        g8, g16 = g8[:, :N], g16[:, :N]
        if tau == 0.0:
            assert np.all(g8 == 0xFF), "no 8-bit logit is computed at threshold 0"
        else:
            if sr_seed is None:
                r8 = O.logits8(qh, kh, w.causal, w.window, r0, nrows)[0, 0]
            else:   # the generator's counter holds the head index b*Hq + h: all heads
                r8 = O.logits8_sr(qb_bits, kb_bits, w.causal, w.window, r0, nrows, sr_seed)[b, h]
            bad = g8 != r8
            assert not bad.any(), "(b %d, h %d): %d of %d 8-bit codes differ, first at %s" % (
                b, h, bad.sum(), bad.size, np.argwhere(bad)[0])
        r16 = O.logits16(qh, kh, w.causal, w.window, r0, nrows)[0, 0]
        # the sub-blocks recomputed in 16 bits, per row of the observed blocks
        sub = m[b, h, qb0:qb0 + nqb]                                   # [nqb, nsub]
        rec = np.repeat((sub == 1) | (sub == 2), bq, axis=0)[:nrows]  # [nrows, nsub]
        rec = np.repeat(rec, bk, axis=1)[:, :N]                        # [nrows, N]
        want16 = np.where(rec & (r16 != 0xFFFF), r16, 0xFFFF).astype(np.uint16)
        bad = g16 != want16
        assert not bad.any(), "(b %d, h %d): %d 16-bit codes differ, first at %s (got %04x want %04x)" % (
            b, h, bad.sum(), np.argwhere(bad)[0], g16[tuple(np.argwhere(bad)[0])], want16[tuple(np.argwhere(bad)[0])])
    return o, lse, mask


SMALL = [
    W.small("o_causal_d128", N=256, d=128, Hq=2, Hkv=1, bq=128, bk=16, nk=4, causal=1, seed=501),
    W.small("o_d64_bq64", N=256, d=64, Hq=2, Hkv=2, bq=64, bk=16, nk=4, causal=1, seed=502),
    W.small("o_bk64_outlier", N=256, d=64, Hq=1, Hkv=1, bq=64, bk=64, nk=4, causal=0, seed=503,
            kind="outlier", n_outlier=2, outlier_gain=16.0),
    W.small("o_window_ragged", N=333, d=128, Hq=1, Hkv=1, bq=128, bk=16, nk=4, causal=1, window=70, seed=504),
    W.small("o_d256", N=256, d=256, Hq=2, Hkv=1, bq=128, bk=16, nk=4, causal=1, seed=505),
    W.small("o_d128_bq64_gqa", N=384, d=128, Hq=4, Hkv=2, bq=64, bk=16, nk=4, causal=1, seed=506),
    W.small("o_saturate", N=256, d=128, Hq=1, Hkv=1, bq=128, bk=16, nk=4, causal=1, seed=313, extra={"gain": 8.0}),
    W.small("o_saturate_bk64", N=256, d=64, Hq=1, Hkv=1, bq=64, bk=64, nk=4, causal=0, seed=314,
            extra={"gain": 8.0}),
]


@pytest.mark.parametrize("tau", [math.inf, 0.5, 2.0 ** -5, 0.0])
@pytest.mark.parametrize("w", SMALL, ids=[w.name for w in SMALL])
def test_observables_small(L, w, tau):
    """Every query block observed: all 8-bit codes and all used 16-bit codes
    of both kernels (pipelined: 16-key sub-blocks; the other: 64-key
    sub-blocks), ragged lengths, saturating inputs."""
    nqb = -(-w.N // w.bq)
    _check_observables(L, w, tau, 0, nqb)


@pytest.mark.parametrize("tau", [math.inf, 0.5, 0.0])
@pytest.mark.parametrize("w", [SMALL[0], SMALL[2], SMALL[4], SMALL[6]], ids=[SMALL[i].name for i in (0, 2, 4, 6)])
def test_observed_instantiation_equals_timed_one(L, w, tau):
    """The instantiation writing the observables and the one without give
    bit-identical O, lse, mask and statistics words on the same inputs."""
    q, k, v, qd, kd, vd = _dev(w)
    s0 = torch.zeros(L.stats_words(w.nk), dtype=torch.int64, device="cuda")
    s1 = torch.zeros_like(s0)
    a = L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, tau, stats=s0)
    nqb = -(-w.N // w.bq)
    b = L.observe_logits(qd, kd, vd, 0, nqb, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, tau, stats=s1)
    torch.cuda.synchronize()
    for x, y in zip(a, b[:3]):   # bit patterns
        assert torch.equal(x.view(torch.int32) if x.dtype == torch.float32 else x,
                           y.view(torch.int32) if y.dtype == torch.float32 else y)
    assert torch.equal(s0, s1)


def test_observables_subrange_and_sr(L):
    """A sub-range of query blocks (the others are not written), and the
    stochastically rounded 8-bit logits."""
    w = W.small("o_sr", N=320, d=128, Hq=2, Hkv=1, bq=64, bk=16, nk=4, causal=1, seed=507)
    _check_observables(L, w, 0.5, 2, 2)
    _check_observables(L, w, 0.5, 1, 3, sr_seed=9)
    _check_observables(L, w, math.inf, 0, 5, sr_seed=2 ** 64 - 1)


@pytest.mark.parametrize("tau", [math.inf, 0.5])
def test_observables_config3_sampled(L, tau):
    """Qwen3-8B-shaped prefill at full size, in the launch configuration the
    benchmark times: the last query block (8192 keys) and block 21 of two
    heads (one per end of the head range), every 8-bit code and every used
    16-bit code."""
    w = W.CONFIGS[3]
    nqb = w.N // w.bq
    inp = _dev(w)
    _check_observables(L, w, tau, nqb - 1, 1, heads=[(0, 0), (0, 31)], q=inp)
    o, lse, mask = _check_observables(L, w, tau, 21, 1, heads=[(0, 5)], q=inp)
    _say("config 3 tau %s: observables of 3 blocks bit-exact, mask %s" % (
        tau, np.bincount(mask.cpu().numpy().ravel(), minlength=4)))


@pytest.mark.parametrize("tau", [math.inf, 0.5])
def test_observables_config5_sampled(L, tau):
    """Long-context batch (N = 32768, B = 4): block nqb/4 of (b 2, h 20) and
    block 40 of (b 3, h 31)."""
    w = W.CONFIGS[5]
    nqb = w.N // w.bq
    inp = _dev(w)
    _check_observables(L, w, tau, nqb // 4, 1, heads=[(2, 20)], q=inp)
    _check_observables(L, w, tau, 40, 1, heads=[(3, 31)], q=inp)
    _say("config 5 tau %s: observables bit-exact" % tau)


def test_observables_config4_global_d256(L):
    """d = 256 at full size (N = 16384, global causal): block 100 of head 7."""
    w = W.CONFIGS[40]
    _check_observables(L, w, 0.5, 100, 1, heads=[(0, 7)])


# ------------------------------------------------------------------ statistics
STAT_CASES = SMALL + [W.CONFIGS[1], W.CONFIGS[2]]


@pytest.mark.parametrize("tau", [math.inf, 0.5, 2.0 ** -5, 0.0])
@pytest.mark.parametrize("w", STAT_CASES, ids=[w.name for w in STAT_CASES])
def test_stats_vs_oracle(L, w, tau):
    """Words 0-5 and the histogram equal the oracle's exactly (saturation
    counts included); the schedule words are consistent with the mode."""
    q, k, v, qd, kd, vd = _dev(w)
    st = torch.zeros(L.stats_words(w.nk), dtype=torch.int64, device="cuda")
    o, lse, mask = L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, tau, stats=st)
    torch.cuda.synchronize()
    got = st.cpu().numpy().astype(np.uint64)
    ro, rlse, rmask, rst = O.fwd(O.bf16_bits(q), O.bf16_bits(k), O.bf16_bits(v), w.causal, w.window, w.bq, w.bk,
                                 w.nk, w.delta, tau, stats=True)
    assert np.array_equal(mask.cpu().numpy(), rmask)
    sel = [0, 1, 2, 3, 4, 5] + list(range(8, 8 + w.nk + 1))
    assert got[sel].tolist() == rst[sel].tolist(), (got.tolist(), rst.tolist())
    if tau == 0.0 or math.isinf(tau):
        assert got[6] == 0 and got[7] == 0


def test_stats_accumulate_and_config3_mask_words(L):
    """Config 3 at full size: the mask-derived words against the mask; two
    calls add up."""
    w = W.CONFIGS[3]
    q, k, v, qd, kd, vd = _dev(w)
    st = torch.zeros(L.stats_words(w.nk), dtype=torch.int64, device="cuda")
    o, lse, mask = L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau, stats=st)
    one = st.clone()
    L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau, stats=st)
    torch.cuda.synchronize()
    assert torch.equal(st, 2 * one)
    s = L.stats_dict(one)
    ms = L.mask_stats(mask, w.nk)
    assert s["stage1"] == ms["stage1"] and s["stage2"] == ms["stage2"] and s["inactive"] == ms["inactive"]
    assert s["hist"] == ms["tile_hist"] and s["tiles"] == sum(ms["tile_hist"])
    _say("config 3 stats: %s" % s)


# ------------------------------------------------------------------ input check, workspace
def test_check_finite(L):
    w = W.small("cf", N=256, d=128, Hq=2, Hkv=1, bq=128, bk=16, nk=4, causal=1, seed=508)
    q, k, v, qd, kd, vd = _dev(w)
    ref = L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau)
    chk = L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau, flags=L.CHECK_FINITE)
    torch.cuda.synchronize()
    for x, y in zip(ref, chk):
        assert torch.equal(x.view(torch.int32) if x.dtype == torch.float32 else x,
                           y.view(torch.int32) if y.dtype == torch.float32 else y)
    for name, t, val in (("q", qd, float("nan")), ("k", kd, float("inf")), ("v", vd, float("-inf"))):
        bad = t.clone()
        bad[0, 0, 77, 5] = val
        args = {"q": (bad, kd, vd), "k": (qd, bad, vd), "v": (qd, kd, bad)}[name]
        with pytest.raises(L.LampError) as ei:
            L.attn_fwd(*args, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau, flags=L.CHECK_FINITE)
        assert ei.value.status == L.LAMP_ERR_NONFINITE_INPUT and str(ei.value).rstrip().endswith(name)
    # a NaN beyond the first block row of the SR and all-16-bit modes as well
    bad = qd.clone()
    bad[0, 1, 255, 127] = float("nan")
    with pytest.raises(L.LampError):
        L.attn_fwd(bad, kd, vd, 1, 0, 128, 16, 4, 2.0 ** -8, 0.0, flags=L.CHECK_FINITE, sr_seed=3)


def test_caller_workspace(L):
    w = W.small("ws", N=300, d=128, Hq=2, Hkv=1, bq=128, bk=16, nk=4, causal=1, seed=509)
    q, k, v, qd, kd, vd = _dev(w)
    ref = L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau)
    n = L.fwd_workspace_size(w.B, w.Hq, w.Hkv, w.N, w.d, w.bq, w.bk, w.nk)
    assert n > 0
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    got = L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau, workspace=ws)
    torch.cuda.synchronize()
    for x, y in zip(ref, got):
        assert torch.equal(x.view(torch.int32) if x.dtype == torch.float32 else x,
                           y.view(torch.int32) if y.dtype == torch.float32 else y)
    with pytest.raises(L.LampError) as ei:
        L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau, workspace=ws[: n - 256])
    assert ei.value.status == L.LAMP_ERR_WORKSPACE
    with pytest.raises(L.LampError) as ei:
        L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau, workspace=ws[16:])
    assert ei.value.status == 1


def test_library_workspace_grows_and_reserve(L):
    """Calls of growing size on the library's workspace (old buffers retired,
    never freed under a running kernel), then lamp_reserve."""
    outs = []
    for n in (128, 512, 2048, 256):
        w = W.small("g%d" % n, N=n, d=128, Hq=2, Hkv=1, bq=128, bk=16, nk=4, causal=1, seed=510)
        q, k, v, qd, kd, vd = _dev(w)
        outs.append((w, q, k, v, L.attn_fwd(qd, kd, vd, w.causal, w.window, w.bq, w.bk, w.nk, w.delta, w.tau)))
    torch.cuda.synchronize()
    for w, q, k, v, (o, lse, mask) in outs:
        ro, rlse, rmask = O.fwd(O.bf16_bits(q), O.bf16_bits(k), O.bf16_bits(v), w.causal, w.window, w.bq, w.bk,
                                w.nk, w.delta, w.tau)
        assert np.array_equal(mask.cpu().numpy(), rmask)
        assert np.abs(o.cpu().numpy() - ro).max() <= 2e-3 * np.abs(ro).max()
    L.reserve(0, 64 << 20)
