"""The calls that a decoding program makes of this library, as cases that can be timed.

A program that decodes with speculative coupling keeps a context and a state, puts the hidden rows
of the current window in front of `step` once per iteration (or its own logits in front of
`step_logits`), and reads tokens out of the state; a program with a loop of its own calls the stages
`lm_head`, `select`, `couple_draft` and `verify` instead.  One pass of a decode case is the beginning of a
decode: `reset`, then `steps` iterations on hidden rows that are resident (they come out of the
model's own kernels in earnest).  In the first iteration every window row is new; in the later
ones about half of the drafts are accepted, the mean over this repository's whole decodes.

Kinds: "step" (LM head and everything after it), "logits" (the same iteration on supplied logits),
"stages" (select, couple_draft, verify on supplied logits), "lm_head" (the projection alone).
"""
import math

import torch

from paper_2510_24211_amd import binding as B

N_TOKENS = 2304        # tokens of a decode (a 48 x 48 image); no case comes near its end


def _case(name, kind, **kw):
    c = dict(name=name, kind=kind, B=1, L=32, V=65536, d=4096, v_lo=0, v_hi=0, top_k=2000, top_p=0.0, lam=3.0,
             tau=1.0, gs=False, mix=0.0, stats=False, steps=4)
    c.update(kw)
    c["v_hi"] = c["v_hi"] or c["V"]
    return c


def listed():
    return [
        # the smallest decode: eight positions over a toy vocabulary, logits supplied by the program
        _case("toy logits", "logits", L=8, V=1024, d=0, top_k=0, lam=0.0),
        # a 24 x 24 image, one class-conditional sequence without guidance
        _case("image 24x24", "step", V=16384, d=1280, top_k=1000, lam=0.0),
        # a 48 x 48 image with guidance, the 8192 image codes of a 65536-entry vocabulary allowed
        _case("image 48x48", "step", v_lo=4, v_hi=8196),
        # the same with every id allowed: the stream over the whole projection matrix
        _case("image full vocabulary", "step"),
        # sixteen images decoded together
        _case("image batch 16", "step", B=16, v_lo=4, v_hi=8196),
        # two videos, window of 64, top-k filter
        _case("video", "step", B=2, L=64, V=64000),
        # the paper's video setting: nucleus filter in place of top-k
        _case("video nucleus", "step", B=2, L=64, V=64000, top_k=0, top_p=0.8),
        # Gumbel sharing, nucleus after top-k and the per-position statistics on the image shape
        _case("image all options", "step", v_lo=4, v_hi=8196, top_p=0.9, gs=True, stats=True),
        # a vocabulary longer than 65536 ids
        _case("long vocabulary", "step", V=131072),
        # a serving loop with a projection of its own, all ids of a 65536-entry vocabulary
        _case("full vocabulary logits", "logits", d=0, lam=0.0),
        # a loop that calls the stages itself; odd row length, window no power of two
        _case("stages odd rows", "stages", B=3, L=20, V=30001, d=0, top_k=1500, lam=0.0),
        # the projection alone on three sequences with a ragged window, id range and temperature
        _case("lm head ragged", "lm_head", B=3, L=20, V=52000, d=2048, v_lo=5, v_hi=51290, tau=0.8, steps=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Windows of 1 to 128, 1 to 16 sequences, rows of 1000 to 131072 ids, hidden sizes of 512 to 4096."""
    while True:
        kind = rng.choices(["step", "logits", "stages", "lm_head"], [6, 2, 1, 1])[0]
        n = _log_int(rng, 1000, 131072)
        v_lo = rng.choice([0, 0, 4, rng.randrange(1, 500)])
        if rng.random() < 0.4:
            n = max(1024, n // 256 * 256)
        d = 0
        if kind in ("step", "lm_head"):
            d = rng.choice([1280, 2048, 4096, 8 * rng.randrange(64, 513)])
        L = rng.choice([8, 16, 32, 32, 64, 128, rng.randrange(1, 129)])
        Bn = rng.choice([1, 1, 1, 2, 3, 4, 8, 16, rng.randrange(1, 17)])
        lam = rng.choice([0.0, 3.0, 3.0]) if d else 0.0
        c = _case("", kind, B=Bn, L=L, V=v_lo + n + rng.choice([0, 0, 100]), d=d, v_lo=v_lo, v_hi=v_lo + n, lam=lam,
                  top_k=rng.choice([0, 1000, 2000, 2000, 2000, _log_int(rng, 20, 3000)]),
                  tau=rng.choice([1.0, 1.0, 0.8]), steps=1 if kind == "lm_head" else 4)
        if kind in ("step", "logits") and n <= 65536:
            c["top_p"] = rng.choice([0.0, 0.0, 0.0, 0.8, 0.9])
            c["gs"] = rng.random() < 0.2
            c["mix"] = rng.choice([0.0, 0.0, 0.0, 0.5])
            c["stats"] = rng.random() < 0.15
        if c["top_k"] == 0 and c["top_p"] == 0.0 and n > 20000:
            c["top_k"] = 2000
        del c["name"]
        w = work(c)
        # no dearer than the listed ones: bytes of the long vocabulary, products of the two videos, and
        # as many logits as the videos hold where the kernels after the projection are what counts
        logits = Bn * L * n
        if Bn * L <= 512 and w["bytes"] <= 4.4e9 and w["flops"] <= 5.3e11 and logits <= (4.2e6 if n > 65536 else 8.2e6):
            return c


def _sizes(c):
    n = c["v_hi"] - c["v_lo"]
    C = 2 if c["lam"] else 1
    return c["B"], C, c["L"], c["d"], n


def _drift(c):
    """Size of the noise by which a row's input changes from one evaluation to the next, for a
    standard deviation of 1.35 in the logits' difference: an overlap of about one half."""
    if c["d"] == 0:
        return 1.35 / math.sqrt(2)
    raw = 0.02 * math.sqrt(c["d"]) / c["tau"]
    return 1.35 / (math.sqrt(2) * raw * math.hypot(1 + c["lam"], c["lam"]))


def _inputs(c, seed):
    """Weights and per-step inputs, from the seed alone.  The rows of a window share one prediction
    (they differ by the drift only): which position a row stands for depends on what was accepted."""
    Bn, C, L, d, n = _sizes(c)
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=g)  # noqa: E731
    steps = 2 if c["kind"] == "stages" else c["steps"]
    if d == 0:
        base = 2.0 * rand(Bn, 1, n)
        return None, [base + _drift(c) * rand(Bn, L, n) for _ in range(steps)]
    W = torch.empty(c["V"], d, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    base = rand(Bn, 1, 1, d)
    if C == 2:
        base = torch.cat([base, 0.9 * base + 0.44 * rand(Bn, 1, 1, d)], 1)
    return W, [(base + _drift(c) * rand(Bn, C, L, d)).to(torch.bfloat16) for _ in range(steps)]


def _config(c, seed):
    return B.make_config(B=c["B"], L=c["L"], N=N_TOKENS, V=c["V"], d=c["d"], v_lo=c["v_lo"], v_hi=c["v_hi"],
                         top_k=c["top_k"], temperature=c["tau"], cfg_lambda=c["lam"], seed=seed,
                         coupling=B.COUPLING_GS if c["gs"] else B.COUPLING_MC, sjd_mix=c["mix"],
                         top_p=c["top_p"], diagnostics=int(c["stats"]))


def _window(c):
    """Where the windows of a call of the stages stand, and its iteration."""
    return [7 + 100 * b for b in range(c["B"])], 5


def _drafts(c, z_prev, seed):
    """Draft tokens drawn from the previous iteration's distribution; every eighth position is new."""
    Bn, _, L, _, n = _sizes(c)
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    z = z_prev.reshape(Bn * L, n)
    if 0 < c["top_k"] < n:
        z = torch.where(z >= torch.topk(z, c["top_k"]).values[:, -1:], z, -math.inf)
    noise = -torch.log(-torch.log(torch.rand(z.shape, device="cuda", generator=g).clamp(1e-7, 1 - 1e-7)))
    x = torch.argmax(z + noise, 1).to(torch.int32).reshape(Bn, L)
    fresh = (torch.arange(L, device="cuda") % 8 == 7).to(torch.uint8).repeat(Bn, 1)
    return x, fresh


def prepare(case, seed):
    c = dict(case)
    Bn, C, L, d, n = _sizes(c)
    W, xs = _inputs(c, seed)
    s = B.Scd(_config(c, seed))
    st = dict(case=c, ctx=s, W=W, xs=xs)
    new = lambda dtype, *shape: torch.empty(*shape, dtype=dtype, device="cuda")  # noqa: E731
    if c["kind"] == "lm_head":
        st["z"] = new(torch.float32, Bn, L, n)
        return st
    if c["kind"] == "stages":
        st["x"], st["fresh"] = _drafts(c, xs[0], seed)
        pos, st["it"] = _window(c)
        st["pos"] = torch.tensor(pos, dtype=torch.int32, device="cuda")
        st.update(thr=new(torch.float32, Bn, L), lse=new(torch.float32, Bn, L), nkept=new(torch.int32, Bn, L),
                  y=new(torch.int32, Bn, L), k=new(torch.uint8, Bn, L), acc=new(torch.int32, Bn),
                  out=torch.full((Bn, N_TOKENS), -1, dtype=torch.int32, device="cuda"))
        return st
    state = st["state"] = s.alloc_state()
    view = lambda f, *shape: s.state_field(state, f).view(*shape)  # noqa: E731
    st["views"] = dict(out=view(B.F_OUT, Bn, N_TOKENS), pos=view(B.F_POS, Bn), drafts=view(B.F_X, Bn, L),
                       y=view(B.F_Y, Bn, L), k=view(B.F_K, Bn, L), px=view(B.F_PX, Bn, L), qx=view(B.F_QX, Bn, L),
                       thr=view(B.F_THR, 2, Bn, L), lse=view(B.F_LSE, 2, Bn, L), z=view(B.F_Z, 2, Bn, L, n))
    if c["gs"] or c["mix"] > 0:
        st["views"]["g"] = view(B.F_G, Bn, L)
    if c["stats"]:
        st["views"].update(stats=view(B.F_DIAG, Bn, L, 4), hamming=view(B.F_HAMM, Bn, 6))
    return st


def run(st):
    s, kind, xs = st["ctx"], st["case"]["kind"], st["xs"]
    if kind == "lm_head":
        s.lm_head(xs[0], st["W"], st["z"])
        return st["z"]
    if kind == "stages":
        s.select(xs[1], st["case"]["B"] * st["case"]["L"], st["thr"], st["lse"], st["nkept"])
        s.couple_draft(xs[1], xs[0], st["x"], st["fresh"], st["pos"], st["it"], st["y"], st["k"])
        s.verify(st["k"], st["y"], st["pos"], st["acc"], st["out"])
        return {f: st[f] for f in ("thr", "lse", "nkept", "y", "k", "acc", "out")}
    state = st["state"]
    s.reset(state)
    for x in xs:
        if kind == "step":
            s.step(x, st["W"], state)
        else:
            s.step_logits(x, state)
    return st["views"]


def work(case):
    Bn, C, L, d, n = _sizes(case)
    rows = Bn * L
    if case["kind"] == "stages":       # both logit arrays, read once
        return {"bytes": 2 * 4 * rows * n, "flops": 0}
    if d == 0:                         # the logits in, and kept for the next iteration
        return {"bytes": case["steps"] * 2 * 4 * rows * n, "flops": 0}
    # each step: the allowed rows of the matrix, the hidden rows, the logits kept for the next one
    return {"bytes": case["steps"] * (2 * d * n + 2 * rows * C * d + 4 * rows * n),
            "flops": case["steps"] * 2 * rows * C * d * n}


def tolerance(case):
    """About four times the largest error against 64 bits that was seen over these ranges."""
    if case["kind"] == "stages":       # logits given: thresholds are exact, normalisers 32-bit sums
        return {"rel": 2e-7, "max": 2e-6, "differ": 0.001}
    if case["d"] == 0:                 # p(x) = exp(z - lse): seen 2.9e-7
        return {"rel": 1.5e-6, "max": 2e-5, "differ": 0.001}
    if case["kind"] == "lm_head":      # seen 6.7e-7
        return {"rel": 3e-6, "max": 4e-5}
    # p(x) moves by the logits' absolute error: seen 8.6e-6
    return {"rel": 4e-5, "max": 4e-4, "differ": 0.005}


# ---- the same in 64 bits ---------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    c = torch.broadcast_tensors(*[torch.as_tensor(v, dtype=torch.int64, device="cuda") for v in (c0, c1, c2, c3)])
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = (((p1 >> 32) & _M32) ^ c[1] ^ k0, p1 & _M32, ((p0 >> 32) & _M32) ^ c[3] ^ k1, p0 & _M32)
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c


def _u01(bits):
    return ((bits >> 9).double() + 0.5) * 2.0 ** -23


def _noise(seq, stream, pos, it, n, seed):
    """-ln U of every id: [rows, n]."""
    ids = torch.arange((n + 3) // 4, device="cuda")
    lanes = _philox(ids[None], pos[:, None], it, (seq[:, None] << 8) | stream, seed)
    return -torch.log(_u01(torch.stack(lanes, 2).reshape(len(pos), -1)[:, :n]))


def _initial(seq, pos, n, seed):
    r = _philox(0, pos, 0, seq << 8, seed)
    return (r[0] * n + ((r[1] * n) >> 32)) >> 32


def _distribution(c, z):
    """Threshold, log normaliser, size of the kept set and probabilities of rows of logits."""
    n = z.shape[-1]
    thr = torch.full_like(z[..., :1], -math.inf)
    if 0 < c["top_k"] < n:
        thr = torch.topk(z, c["top_k"], dim=-1).values[..., -1:]
    if 0 < c["top_p"] < 1:
        s = torch.sort(torch.where(z >= thr, z, -math.inf), dim=-1, descending=True).values
        w = torch.exp(s - s[..., :1])
        above = torch.cumsum(w, -1) - w
        last = (above < c["top_p"] * w.sum(-1, keepdim=True)).sum(-1, keepdim=True) - 1
        thr = torch.gather(s, -1, last)
    kept = z >= thr
    lse = torch.logsumexp(torch.where(kept, z, -math.inf), -1, keepdim=True)
    return thr[..., 0], lse[..., 0], kept.sum(-1), torch.where(kept, torch.exp(z - lse), 0.0)


def _logits(c, W64, x):
    if W64 is None:
        return x.double()
    a = torch.matmul(x.double().reshape(-1, c["d"]), W64.t()).reshape(x.shape[:3] + (W64.shape[0],))
    z = a[:, 0] if a.shape[1] == 1 else (1 + c["lam"]) * a[:, 0] - c["lam"] * a[:, 1]
    return z / c["tau"]


def _residual(p, q, seq, pos, it, x, seed):
    """One rejection-sampling call per row of [rows, n]: accepted, next token, p(x), q(x)."""
    px, qx = (torch.gather(v, 1, x[:, None])[:, 0] for v in (p, q))
    u = _u01(_philox(0, pos, it, (seq << 8) | 1, seed)[0])
    r = torch.clamp(p - q, min=0.0)
    y = torch.argmin(torch.where(r > 0, _noise(seq, 2, pos, it, p.shape[1], seed) / r, math.inf), 1)
    accept = (u * qx <= px) | ~(r > 0).any(1)
    return accept, torch.where(accept, x, y), px, qx


def exact(case, seed):
    c = dict(case)
    Bn, C, L, d, n = _sizes(c)
    W, xs = _inputs(c, seed)
    W64 = None if W is None else W[c["v_lo"]:c["v_hi"]].double()
    if c["kind"] == "lm_head":
        return _logits(c, W64, xs[0])
    if c["kind"] == "stages":
        thr, lse, _, _ = _distribution(c, xs[1].double())
        return dict(thr=thr, lse=lse, nkept=None, y=None, k=None, acc=None, out=None)
    s = torch.arange(L, device="cuda")
    seqs = torch.arange(Bn, device="cuda")
    seed64 = seed & 0xFFFFFFFFFFFFFFFF
    pos = torch.zeros(Bn, dtype=torch.int64, device="cuda")
    X = _initial(seqs[:, None], s[None].repeat(Bn, 1), n, seed64)        # window order
    seen = torch.zeros(Bn, L, dtype=torch.bool, device="cuda")
    p_old = torch.zeros(Bn, L, n, dtype=torch.float64, device="cuda")
    ring = {f: torch.zeros(2, Bn, L, dtype=torch.float64, device="cuda") for f in ("thr", "lse")}
    z_ring = torch.zeros(2, Bn, L, n, dtype=torch.float64, device="cuda")
    stats = torch.zeros(Bn, L, 4, dtype=torch.float64, device="cuda")
    px, qx = (torch.zeros(Bn, L, dtype=torch.float64, device="cuda") for _ in range(2))
    for t, x in enumerate(xs):
        z = _logits(c, W64, x)
        for b in range(Bn):
            j = pos[b] + s
            thr, lse, _, p = _distribution(c, z[b])
            q = torch.where(seen[b][:, None], p_old[b], 1.0 / n)
            seq = seqs[b].expand(L)
            accept, y, px[b], qx[b] = _residual(p, q, seq, j, t, X[b], seed64)
            stats[b] = torch.stack([torch.minimum(p, q).sum(1), (p * q).sum(1), (p * p).sum(1), (q * q).sum(1)], 1)
            ring["thr"][t & 1, b, j % L], ring["lse"][t & 1, b, j % L] = thr, lse
            z_ring[t & 1, b, j % L] = z[b]
            nxt = y
            if c["gs"]:
                nxt = torch.argmin(_noise(seq, 3, j, 0, n, seed64) / p, 1)
            if c["mix"] > 0:
                alone = _u01(_philox(0, j, t, (seq << 8) | 4, seed64)[0]) > 1.0 - c["mix"]
                nxt = torch.where(alone, torch.argmin(_noise(seq, 5, j, t, n, seed64) / p, 1), nxt)
            rejected = torch.nonzero(~accept)
            a = int(rejected[0]) + 1 if len(rejected) else L
            enter = pos[b] + L + torch.arange(a, device="cuda")
            X[b] = torch.cat([nxt[a:], _initial(seqs[b].expand(a), enter, n, seed64)])
            seen[b] = s < L - a
            p_old[b] = torch.cat([p[a:], p[:a]])
            pos[b] += a
    out = dict(out=None, pos=None, drafts=None, y=None, k=None, px=px, qx=qx, thr=ring["thr"], lse=ring["lse"], z=z_ring)
    if c["gs"] or c["mix"] > 0:
        out["g"] = None
    if c["stats"]:
        out.update(stats=stats, hamming=None)
    return out
