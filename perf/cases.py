"""The workloads that the speed of this framework is measured on.

Every case is one call of a public entry point (paper_2609_39361_amd.lamp:
attn_fwd for prompts, attn_decode for new tokens against a cache) on seeded
inputs with the statistics of paper_2609_39361_amd/workloads.py: heavy-tailed
per-channel scales on Q and K, rotary embedding, V ~ N(0, 1).  A case holds
the attention shape (B, Hq, Hkv, N, d, causal, window), the method's block
sizes and thresholds (bq, bk, nk, delta, tau), the precision options (flags,
sr_seed) and the input recipe; M > 0 marks a decode case.
"""
import math

import torch

from paper_2609_39361_amd import lamp

DELTA = 2.0 ** -8
# flag of the forward pass that selects the paper's simulation numerics
SIM = lamp.SIM_PROFILE


def _case(name, **kw):
    c = dict(B=1, Hq=32, Hkv=8, N=1024, d=128, M=0, causal=1, window=0, bq=128, bk=16, nk=4, delta=DELTA, tau=0.5,
             flags=0, sr_seed=-1, kind="lognormal", sigma=0.75, rope=1e6)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    """The listed cases, small to large."""
    return [
        # the smallest call the test suite and a first user make: one head, a
        # non-causal encoder block of 256 tokens, 64-key sub-blocks (launch and
        # latency bound)
        _case("single_head_256", Hq=1, Hkv=1, N=256, d=64, causal=0, bq=64, bk=64, kind="outlier", sigma=16.0),
        # a short chat prompt on a Qwen3-8B-shaped layer, ragged length
        _case("chat_prompt_300", N=300),
        # two sequences of 1024, 8 heads, the coarse 64-key sub-blocks, with
        # attention-sink-like keys
        _case("mha8_1024_coarse", B=2, Hq=8, Hkv=8, N=1024, bk=64, kind="sink", sigma=12.0),
        # a medium prompt whose length divides no block size
        _case("prompt_1999", N=1999),
        # small heads (d = 64), the pure 8-bit baseline of the paper
        _case("d64_low_2048", B=4, Hq=16, Hkv=16, N=2048, d=64, tau=math.inf, rope=1e4),
        # the paper's own simulation numerics
        _case("simulation_2048", N=2048, flags=SIM),
        # the 16-bit FlashAttention baseline (every sub-block in 16 bits)
        _case("all16_4096", N=4096, tau=0.0),
        # Gemma-3-4B-shaped local layer: d = 256, sliding window 1024
        _case("window_16k_d256", Hq=8, Hkv=4, N=16384, d=256, window=1024, sigma=1.0, rope=1e4),
        # Qwen3-8B-shaped 8K prefill, the framework's headline configuration
        _case("prefill_8k", N=8192),
        # long context: the 32K configuration's sequence, |Student-t| channels
        _case("long_context_32k", N=32768, kind="student"),
        # one user's next token against a long cache of odd length
        _case("decode_1x20011", M=1, N=20011, bq=1, bk=64, nk=1),
        # a serving batch: the next token of 32 sequences against 8K caches
        _case("decode_32x8192", B=32, M=1, N=8192, bq=1, bk=64, nk=1),
    ]


def _pairs(c):
    """Visible (query, key) pairs of one head."""
    n, w = c["N"], c["window"]
    if c["M"] > 0:
        return sum(min(p + 1, w) if w else (p + 1 if c["causal"] else n) for p in range(n - c["M"], n))
    if not c["causal"]:
        return n * n
    return n * (n + 1) // 2 if not w or w >= n else w * (w + 1) // 2 + (n - w) * w


# drawn cases cost at most a quarter of the largest listed one (multiply-adds
# of the logits, the options' extra cost counted)
_MAX_MACS = 32 * 128 * (32768 * 32769 // 2) // 4


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: lengths from one token block to the
    long context, odd ones among them, every head dimension, head grouping,
    block size, threshold and precision option."""
    while True:
        d = rng.choice([64, 128, 128, 128, 256])
        hkv = rng.choice([1, 2, 4, 8])
        hq = hkv * rng.choice([1, 2, 4])
        tau = rng.choice([0.5, 0.5, 0.5, 1.0, 2.0 ** -5, math.inf, 0.0])
        kind, sigma = rng.choice([("lognormal", 0.75), ("lognormal", 1.0), ("student", 0.0), ("outlier", 12.0)])
        rope = rng.choice([1e4, 1e6])
        common = dict(Hq=hq, Hkv=hkv, d=d, tau=tau, kind=kind, sigma=sigma, rope=rope)
        if rng.random() < 0.35:
            n = _log_int(rng, 65, 40000)
            c = _case("", B=_log_int(rng, 1, 32), M=rng.choice([1, 1, 1, 2]), N=n, bq=1, bk=64, nk=1,
                      window=rng.choice([0, 0, 0, 1024]), **common)
            # the cache stays below 4 GB
            if 4 * c["B"] * hkv * n * d > 4 << 30:
                continue
            return c
        n = _log_int(rng, 64, 16384)
        if rng.random() < 0.4:
            n = max(64, n // 64 * 64)
        causal = 1 if rng.random() < 0.8 else 0
        bk = 16 if rng.random() < 0.75 else 64
        c = _case("", B=rng.choice([1, 1, 2, 4]), N=n, causal=causal, bq=rng.choice([64, 128, 128]), bk=bk,
                  window=rng.choice([0, 0, 0, 512, 1024]) if causal else 0, **common)
        option = rng.random()
        cost = c["B"] * hq * _pairs(c) * d
        if option < 0.15 and bk == 16 and d >= 128:
            c["flags"] = SIM
            cost *= 2
        elif option < 0.25 and tau != 0.0:
            c["sr_seed"] = rng.randrange(1 << 31)
            cost *= 4
        if cost <= _MAX_MACS:
            return c


def _rope(x, base, pos0):
    """Rotate-half rotary embedding of x [B, H, n, d], positions pos0, pos0+1, ..."""
    n, d = x.shape[-2], x.shape[-1]
    inv = base ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    ang = torch.arange(pos0, pos0 + n, device=x.device, dtype=torch.float64)[:, None] * inv[None, :]
    c, s = ang.cos().float(), ang.sin().float()
    a, b = x[..., : d // 2], x[..., d // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _inputs(case, seed):
    """(q, k, v) bf16 on the GPU, from the seed alone."""
    dev = "cuda"
    g = torch.Generator(dev)
    g.manual_seed(1000003 * (seed + 1) + 17)
    B, Hq, Hkv, N, d = (case[x] for x in ("B", "Hq", "Hkv", "N", "d"))
    nq = case["M"] or N

    def randn(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32)

    q, k, v = randn(B, Hq, nq, d), randn(B, Hkv, N, d), randn(B, Hkv, N, d)
    kind = case["kind"]
    if kind in ("outlier", "sink"):
        # a few outlier channels; "sink": some key rows much larger than the rest
        ch = torch.randperm(d, generator=g, device=dev)[:4]
        q[..., ch] *= case["sigma"]
        k[..., ch] *= case["sigma"]
        if kind == "sink":
            rows = torch.randperm(N, generator=g, device=dev)[:9]
            k[:, :, rows] *= 8.0
            k[:, :, 0] *= 8.0
    else:
        if kind == "lognormal":
            sq, sk = (case["sigma"] * randn(1, Hq, 1, d)).exp(), (case["sigma"] * randn(1, Hkv, 1, d)).exp()
        else:
            sq = (randn(1, Hq, 1, d) / (randn(1, Hq, 1, d, 3).square().mean(-1)).sqrt()).abs()
            sk = (randn(1, Hkv, 1, d) / (randn(1, Hkv, 1, d, 3).square().mean(-1)).sqrt()).abs()
        q = _rope(q * sq, case["rope"], N - nq)
        k = _rope(k * sk, case["rope"], 0)
    return tuple(t.to(torch.bfloat16).contiguous() for t in (q, k, v))


def prepare(case, seed):
    """The call's inputs, resident on the GPU."""
    q, k, v = _inputs(case, seed)
    return {"case": case, "q": q, "k": k, "v": v}


def run(state):
    """One call: (o, lse, mask)."""
    c = state["case"]
    if c["M"] > 0:
        return lamp.attn_decode(state["q"], state["k"], state["v"], causal=bool(c["causal"]), window=c["window"],
                                tk=c["bk"], delta=c["delta"], tau=c["tau"])
    return lamp.attn_fwd(state["q"], state["k"], state["v"], causal=bool(c["causal"]), window=c["window"], bq=c["bq"],
                         bk=c["bk"], nk=c["nk"], delta=c["delta"], tau=c["tau"], flags=c["flags"],
                         sr_seed=c["sr_seed"] if c["sr_seed"] >= 0 else None)


def work(case):
    """q, k, v read and o, lse, mask written once; two operations per
    multiply-add of the logits and of P.V over the visible pairs (the keys a
    window hides from every query are not read)."""
    B, Hq, Hkv, N, d, M, w = (case[x] for x in ("B", "Hq", "Hkv", "N", "d", "M", "window"))
    nq = M or N
    keys = min(N, w + M - 1) if M and w else N
    if M:
        mask = M * (-(-N // 64) * 64)
    else:
        t = case["bk"] * case["nk"]
        mask = -(-N // case["bq"]) * (-(-N // t) * case["nk"])
    nbytes = 2 * B * Hq * nq * d + 4 * B * Hkv * keys * d + B * Hq * (4 * nq * d + 4 * nq + mask)
    return {"bytes": nbytes, "flops": 4 * B * Hq * d * _pairs(case)}


def tolerance(case):
    """Masks are decisions on rounded logits that the method fixes bit for bit:
    they have to be equal.  o and lse are sums in fp32 (o accumulates up to N
    exact products per element) and one fp32 rounding."""
    return {"rel": 4e-6, "max": 4e-5}


# ---------------------------------------------------------------------------
# The method in plain torch with 64-bit arithmetic, from its definition: every
# number is rounded to the format the method names and to nothing else.

def _rnd(x, bits, emin, top=math.inf):
    """x rounded to nearest even with `bits` mantissa bits, smallest normal
    exponent emin (gradual underflow below), magnitudes limited to top."""
    e = torch.frexp(x.abs())[1].to(torch.float64) - 1
    q = torch.exp2(torch.clamp(e, min=emin) - bits)
    return torch.clamp(torch.round(x / q) * q, -top, top)


class _Formats:
    """The two profiles: the hardware formats, and the paper's simulation (3
    and 11 mantissa bits in FP32's range)."""

    def __init__(self, sim):
        if sim:
            self.y8 = self.s8 = self.e8 = lambda x: _rnd(x, 3, -126)
            self.y16 = self.s16 = self.e16 = lambda x: _rnd(x, 11, -126)
        else:
            self.y8 = lambda x: _rnd(x, 3, -6, 448.0)
            self.y16 = lambda x: _rnd(x, 11, -6, 511.875)
            self.s8, self.s16 = (lambda x: _rnd(x, 3, -14)), (lambda x: _rnd(x, 11, -14))
            self.e8, self.e16 = (lambda x: _rnd(x, 3, -30)), (lambda x: _rnd(x, 11, -30))

    def exp8(self, mu, y):
        return self.e8(torch.exp(-self.s8((mu - y).clamp(min=0.0))))

    def exp16(self, mu, y):
        return self.e16(torch.exp(-self.s16((mu - y).clamp(min=0.0))))


def _logits(q, k, d, fm):
    """8-bit and 16-bit logits of q [..., n, d] and k [..., m, d]: FP32 fused
    multiply-adds over ascending channels, the 8-bit sum rounded after every
    one, the 16-bit sum once at the end."""
    qs = (q.float() * torch.tensor(1.0 / math.sqrt(d), device=q.device).float()).double()
    ks = k.double()
    y8 = torch.zeros(torch.broadcast_shapes(q.shape[:-2], k.shape[:-2]) + (q.shape[-2], k.shape[-2]),
                     dtype=torch.float64, device=q.device)
    y16 = torch.zeros_like(y8)
    for c in range(d):
        prod = qs[..., :, c, None] * ks[..., None, :, c]
        y8 = fm.y8((prod + y8).float().double())
        y16 = (prod + y16).float().double()
    return y8, fm.y16(y16)


def _visible(pos, n, causal, window):
    i = torch.arange(n, device=pos.device)
    v = torch.ones(pos.shape[0], n, dtype=torch.bool, device=pos.device)
    if causal:
        v &= i[None, :] <= pos[:, None]
    if window:
        v &= i[None, :] > pos[:, None] - window
    return v


def _exact_fwd(case, q, k, v):
    """One (batch, head) after another; all query blocks of a head at once."""
    B, Hq, Hkv, N, d, bq, bk, nk = (case[x] for x in ("B", "Hq", "Hkv", "N", "d", "bq", "bk", "nk"))
    tau, delta, fm, T = case["tau"], case["delta"], _Formats(case["flags"] & SIM), bk * nk
    dev, inf = q.device, math.inf
    nqb, nt = -(-N // bq), -(-N // T)
    pos = torch.arange(nqb * bq, device=dev)
    vis = torch.zeros(nqb * bq, nt * T, dtype=torch.bool, device=dev)
    vis[:N, :N] = _visible(pos[:N], N, case["causal"], case["window"])
    vis = vis.view(nqb, bq, nt, nk, bk)
    o = torch.empty(B, Hq, N, d, dtype=torch.float64, device=dev)
    lse = torch.empty(B, Hq, N, dtype=torch.float64, device=dev)
    mask = torch.empty(B, Hq, nqb, nt * nk, dtype=torch.uint8, device=dev)
    subsets = sorted(range(1 << nk), key=lambda r: (bin(r).count("1"), r))
    for b in range(B):
        for h in range(Hq):
            kh, vh = k[b, h // (Hq // Hkv)], v[b, h // (Hq // Hkv)].double()
            vp = torch.zeros(nt * T, d, dtype=torch.float64, device=dev)
            vp[:N] = vh
            y8, y16 = _logits(q[b, h], kh, d, fm)
            pad = (0, nt * T - N, 0, nqb * bq - N)
            y8 = torch.nn.functional.pad(y8, pad).view(nqb, bq, nt, nk, bk)
            y16 = torch.nn.functional.pad(y16, pad).view(nqb, bq, nt, nk, bk)
            mu = torch.full((nqb, bq), -inf, dtype=torch.float64, device=dev)
            om, O = torch.zeros_like(mu), torch.zeros(nqb, bq, d, dtype=torch.float64, device=dev)
            for t in range(nt):
                vt, a8, a16 = vis[:, :, t], y8[:, :, t], y16[:, :, t]
                m8 = a8.masked_fill(~vt, -inf).amax(-1)          # [nqb, bq, nk]
                m16 = a16.masked_fill(~vt, -inf).amax(-1)
                act = vt.any(-1).any(1)                          # [nqb, nk]
                high = torch.zeros_like(act)                     # stage 1
                muh = mu.clone()
                if tau == inf:
                    muh = torch.maximum(mu, m8.amax(-1))
                elif tau == 0.0:
                    high = act.clone()
                    muh = torch.maximum(mu, m16.amax(-1))
                else:
                    # threat of a sub-block: max over rows of m8 - mu, tested in descending order
                    thr = torch.where(m8 > -inf, torch.where(mu[..., None] > -inf, m8 - mu[..., None], inf), -inf)
                    thr = thr.amax(1).masked_fill(~act, -inf)
                    order = torch.argsort(thr, dim=-1, descending=True, stable=True)
                    for r in range(nk):
                        th = order[:, r]
                        ix = th[:, None, None].expand(nqb, bq, 1)
                        c8, c16 = m8.gather(-1, ix)[..., 0], m16.gather(-1, ix)[..., 0]
                        ok = (muh > muh.abs() * delta + c8) | (c8 == -inf)
                        bad = ~ok.all(1) & act.gather(-1, th[:, None])[:, 0]
                        high[torch.arange(nqb, device=dev)[bad], th[bad]] = True
                        muh = torch.where(bad[:, None], torch.maximum(muh, c16), muh)
                mref = muh.masked_fill(muh == -inf, 0.0)[..., None, None]
                e8 = fm.exp8(mref, a8).masked_fill(~vt, 0.0)
                e16 = fm.exp16(mref, a16).masked_fill(~vt, 0.0)
                E = torch.where(high[:, None, :, None], e16, e8)
                lam = torch.where(muh == -inf, 1.0, torch.where(mu == -inf, 0.0, torch.exp(mu - muh)))
                codes = torch.where(act, high.to(torch.uint8), 3)
                if 0.0 < tau < inf:
                    omh = lam * om + E.sum((-1, -2))
                    keep = act & ~high
                    cost = (E * (omh[..., None, None] - E)).sum(-1)      # [nqb, bq, nk]
                    cost = cost * keep[:, None, :]
                    lim = tau * omh * omh
                    chosen = torch.full((nqb,), -1, device=dev)
                    free = (keep.long() << torch.arange(nk, device=dev)).sum(-1)
                    for r in subsets:
                        bits = torch.tensor([(r >> i) & 1 for i in range(nk)], device=dev, dtype=torch.bool)
                        fits = ((cost * ~bits).sum(-1) <= lim).all(1) & ((r & ~free) == 0)
                        chosen = torch.where((chosen < 0) & fits, r, chosen)
                    two = ((chosen[:, None] >> torch.arange(nk, device=dev)) & 1).bool()
                    codes = torch.where(two, 2, codes)
                    E = torch.where(two[:, None, :, None], e16, E)
                om = lam * om + E.sum((-1, -2))
                O = O * lam[..., None] + E.reshape(nqb, bq, T) @ vp[t * T:(t + 1) * T]
                mu = muh
                mask[b, h, :, t * nk:(t + 1) * nk] = codes.to(torch.uint8)
            o[b, h] = (O / om[..., None]).view(nqb * bq, d)[:N]
            lse[b, h] = (mu + om.log()).view(-1)[:N]
    return o, lse, mask


def _exact_decode(case, q, k, v):
    """All query rows at once, one tile of 64 keys after another."""
    B, Hq, Hkv, N, d, M = (case[x] for x in ("B", "Hq", "Hkv", "N", "d", "M"))
    tau, delta, fm, T = case["tau"], case["delta"], _Formats(False), 64
    dev, inf, G = q.device, math.inf, Hq // Hkv
    nt = -(-N // T)
    y8, y16 = _logits(q.view(B, Hkv, G * M, d), k, d, fm)
    pad = (0, nt * T - N)
    y8 = torch.nn.functional.pad(y8, pad).view(B * Hq, M, nt, T)
    y16 = torch.nn.functional.pad(y16, pad).view(B * Hq, M, nt, T)
    vis = torch.nn.functional.pad(_visible(torch.arange(N - M, N, device=dev), N, case["causal"], case["window"]), pad)
    vis = vis.view(1, M, nt, T).expand(B * Hq, M, nt, T)
    vp = torch.zeros(B, Hkv, nt * T, d, dtype=torch.float64, device=dev)
    vp[:, :, :N] = v.double()
    mu = torch.full((B * Hq, M), -inf, dtype=torch.float64, device=dev)
    om = torch.zeros_like(mu)
    O = torch.zeros(B, Hkv, G * M, d, dtype=torch.float64, device=dev)
    mask = torch.full((B * Hq, M, nt, T), 3, dtype=torch.uint8, device=dev)
    for t in range(nt):
        vt, a8, a16 = vis[:, :, t], y8[:, :, t], y16[:, :, t]
        live = vt.any(-1)
        c = a8.masked_fill(~vt, -inf).max(-1)
        first = (a8 == c.values[..., None]) & vt
        ci = first.to(torch.uint8).argmax(-1, keepdim=True)
        codes = torch.where(vt, 0, 3)
        high = torch.zeros_like(vt)
        if tau == inf:
            muh = torch.maximum(mu, c.values)
        elif tau == 0.0:
            muh, high = torch.maximum(mu, a16.masked_fill(~vt, -inf).amax(-1)), vt.clone()
        else:
            fails = live & ~(mu > mu.abs() * delta + c.values)
            muh = torch.where(fails, torch.maximum(mu, a16.gather(-1, ci)[..., 0]), mu)
            high = torch.zeros_like(vt).scatter(-1, ci, fails[..., None])
        codes = torch.where(high, 1, codes)
        mref = muh.masked_fill(muh == -inf, 0.0)[..., None]
        e8, e16 = fm.exp8(mref, a8).masked_fill(~vt, 0.0), fm.exp16(mref, a16).masked_fill(~vt, 0.0)
        E = torch.where(high, e16, e8)
        lam = torch.where(muh == -inf, 1.0, torch.where(mu == -inf, 0.0, torch.exp(mu - muh)))
        if 0.0 < tau < inf:
            omh = lam * om + E.sum(-1)
            cost = (E * (omh[..., None] - E)).masked_fill(~vt | high, inf)
            srt = torch.sort(cost, dim=-1, stable=True)
            over = ~(srt.values.cumsum(-1) <= (tau * omh * omh)[..., None])
            two = torch.zeros_like(vt).scatter(-1, srt.indices, over) & vt & ~high
            codes = torch.where(two, 2, codes)
            E = torch.where(two, e16, E)
        om = lam * om + E.sum(-1)
        O = O * lam.view(B, Hkv, G * M, 1) + E.view(B, Hkv, G * M, T) @ vp[:, :, t * T:(t + 1) * T]
        mu = muh
        mask[:, :, t] = codes.to(torch.uint8)
    lse = (mu + om.log()).view(B, Hq, M)
    return (O.view(B, Hq, M, d) / om.view(B, Hq, M, 1)), lse, mask.view(B, Hq, M, nt * T)


def exact(case, seed):
    """(o, lse, mask) of the method in 64-bit arithmetic.  None for
    stochastic rounding, whose random numbers only the library defines, and
    where the 64-bit pass would take too long."""
    if case["sr_seed"] >= 0:
        return None
    q, k, v = _inputs(case, seed)
    if case["M"] > 0:
        if case["B"] * case["Hq"] * case["M"] * case["N"] * case["d"] > 1 << 31:
            return None
        return _exact_decode(case, q, k, v)
    if case["B"] * case["Hq"] * case["N"] ** 2 * case["d"] > 1 << 34 or case["B"] * case["Hq"] * case["N"] > 1 << 17:
        return None
    return _exact_fwd(case, q, k, v)
