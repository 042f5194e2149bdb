"""What is timed: the calls that a decoding program makes on this library.

A program built on the library decodes candidate trajectories: every step it
calls the base attention (append, attend, window score) over an evicted cache,
the helper attention over a long context, and the entropy and token draw over
the logits; when a cache overflows it evicts; when a step is accepted it
commits it (bulk append, window scores) or forks the candidates again; a
prompt is compressed in one shot. Shapes are those of the workloads of
paper_2608_15797_amd/workloads.py and of movebench.py (7B: 28 layers, 28 query
and 4 KV heads; 72B: 80 layers, 64 and 8; 1.5B helper: 28 layers, 12 and 2;
head_dim 128), inputs N(0, 1) keys, values and queries and logits of standard
deviation 3 with five raised entries, as there.

Every case has a "kind" (the call) and its sizes. Live lengths run evenly from
a lowest to a highest value over the sequences, in an order drawn from the
seed, so the work does not depend on the seed.
"""
import math
import random

import torch

from paper_2608_15797_amd import kvr

DEV = "cuda"
M7B = dict(L=28, Hq=28, Hkv=4, D=128)
M72B = dict(L=80, Hq=64, Hkv=8, D=128)
M15B = dict(L=28, Hq=12, Hkv=2, D=128)
V_BASE, V_HELPER = 152064, 151936
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
ESZ = {"bf16": 2, "f32": 4}


def listed():
    return [
        # One layer of a model that decodes layer by layer: 16 problems x 8
        # candidates of the 7B base at B = 64, inside the window. The smallest
        # call: launch and host time count.
        dict(name="decode_7b_one_layer", kind="decode", dtype="bf16", S=128, **{**M7B, "L": 1}, B=64, W=32,
             buffer=64, n_lo=98, n_hi=129, cap=144, R=0, V=0, ldt="bf16", sample=False),
        # A whole step of the 7B base, 16 problems x 4 candidates at B = 128 at
        # every point of the eviction cycle, with the entropies, the detector
        # and the token draw of its logit rows in the same call.
        dict(name="decode_7b_sample", kind="decode", dtype="bf16", S=64, **M7B, B=128, W=32, buffer=128, n_lo=129,
             n_hi=257, cap=272, R=64, V=V_BASE, ldt="bf16", sample=True),
        # A whole step of the 72B base in lockstep inside the observation
        # window, with the entropies of its logit rows.
        dict(name="decode_72b_window", kind="decode", dtype="bf16", S=32, **M72B, B=64, W=32, buffer=64, n_lo=119,
             n_hi=119, cap=144, R=32, V=V_BASE, ldt="bf16", sample=False),
        # A float32 cache (the type of the small validation workload) at the
        # 7B shape with few candidates.
        dict(name="decode_7b_f32", kind="decode", dtype="f32", S=8, **M7B, B=128, W=32, buffer=128, n_lo=129,
             n_hi=257, cap=257, R=0, V=0, ldt="f32", sample=False),
        # Helper-only decode: 8 private contexts of 4096 tokens, the entropy
        # rows in the context launch.
        dict(name="helper_4k", kind="context", S=8, P=8, **M15B, plen=4096, scap=512, u_lo=1, u_hi=512, R=8,
             V=V_HELPER, sample=False),
        # Helper beside the 7B base: 16 contexts of 8192 tokens, each shared by
        # 8 candidates, ragged suffixes.
        dict(name="helper_8k_shared", kind="context", S=128, P=16, **M15B, plen=8192, scap=512, u_lo=1, u_hi=512,
             R=0, V=0, sample=False),
        # Helper beside the 72B base: 32 private contexts of 16384 tokens. The
        # largest call by bytes.
        dict(name="helper_16k_private", kind="context", S=32, P=32, **M15B, plen=16384, scap=512, u_lo=1, u_hi=512,
             R=0, V=0, sample=False),
        # Committing an accepted step to 16 states: append of 128 tokens and
        # the window scores of their queries, ragged live lengths.
        dict(name="commit_7b", kind="score", dtype="bf16", S=16, **M7B, n_lo=513, n_hi=640, T=128, nq=128, cap=769),
        # One-shot compression of a 4096-token prompt: append and window scores.
        dict(name="prompt_7b", kind="score", dtype="bf16", S=16, **M7B, n_lo=0, n_hi=0, T=4096, nq=128, cap=4096),
        # The eviction of a 72B step in lockstep.
        dict(name="evict_72b", kind="evict", dtype="bf16", S=32, L=80, Hkv=8, D=128, B=64, W=32, buffer=64,
             n_lo=129, n_hi=129, cap=144),
        # Fork of 16 trajectory states to 8 candidates each.
        dict(name="fork_7b", kind="fork", dtype="bf16", P=16, N=8, L=28, Hkv=4, D=128, n_lo=513, n_hi=640, cap=641),
        # Entropy, detector and token draw of a step's logits on their own (a
        # model that decodes layer by layer has them after its last layer).
        dict(name="sample_128_rows", kind="sample", ldt="bf16", R=128, V=V_BASE, top_k=20),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "context", "context", "score", "score", "evict", "fork", "sample"))
    if kind == "decode":
        f32 = rng.random() < 0.25
        m = dict(rng.choice((M7B, M7B, M72B)))
        m["L"] = _log(rng, 1, m["L"])
        if rng.random() < 0.2:
            m["D"] = 64
        W = rng.choice((8, 16, 32))
        B, buffer = rng.randint(W + 16, 160), rng.randint(W, 128)
        S = rng.randint(1, 8) if f32 else _log(rng, 4, 128)
        while S > 1 and S * m["L"] * m["Hkv"] > (900 if f32 else 20480):
            S //= 2
        cap = B + buffer + 1 + rng.choice((0, 0, -(B + buffer + 1) % 16))
        rows = rng.choice((0, S)) if not f32 else 0
        return dict(kind="decode", dtype="f32" if f32 else "bf16", S=S, **m, B=B, W=W, buffer=buffer, n_lo=B + 1,
                    n_hi=B + buffer + 1, cap=cap, R=rows, V=rng.choice((V_BASE, V_HELPER)) if rows else 0,
                    ldt="bf16", sample=bool(rows and rng.random() < 0.5))
    if kind == "context":
        C = rng.choice((1, 1, 2, 4, 5, 8))
        m = dict(M15B)
        m["L"] = _log(rng, 2, 28)
        plen = _log(rng, 1000, 16384)
        P = _log(rng, 1, 32)
        rows = rng.choice((0, 0, P * C))
        return dict(kind="context", S=P * C, P=P, **m, plen=plen, scap=512, u_lo=1, u_hi=rng.randint(2, 512), R=rows,
                    V=V_HELPER if rows else 0, sample=bool(rows and rng.random() < 0.5))
    if kind == "score":
        m = dict(M7B)
        m["L"] = _log(rng, 1, 28)
        T = _log(rng, 16, 3000)
        n_hi = rng.randint(1, 640)
        n_lo = max(0, n_hi - rng.randint(0, 127))
        return dict(kind="score", dtype="bf16", S=_log(rng, 1, 16), **m, n_lo=n_lo, n_hi=n_hi, T=T,
                    nq=min(T, rng.randint(8, 128)), cap=n_hi + T + rng.randint(0, 128))
    if kind == "evict":
        W = rng.choice((8, 32, 64))
        B, buffer = rng.randint(W + 16, 512), rng.randint(W, 160)
        return dict(kind="evict", dtype="bf16", S=_log(rng, 1, 32), L=rng.choice((1, 28, 28, 80)), Hkv=4, D=128, B=B,
                    W=W, buffer=buffer, n_lo=B + buffer - rng.randint(0, 3), n_hi=B + buffer + 1, cap=B + buffer + 1)
    if kind == "fork":
        n_hi = rng.randint(65, 640)
        return dict(kind="fork", dtype="bf16", P=_log(rng, 1, 16), N=rng.randint(2, 8), L=rng.choice((1, 28, 28)),
                    Hkv=4, D=128, n_lo=max(1, n_hi - rng.randint(0, 128)), n_hi=n_hi, cap=n_hi + rng.randint(0, 31))
    return dict(kind="sample", ldt=rng.choice(("bf16", "bf16", "f32")), R=_log(rng, 1, 256),
                V=rng.choice((V_BASE, V_HELPER, rng.randint(30000, 152000))), top_k=rng.choice((1, 20, 20, 50)))


# ---------------------------------------------------------------------------
def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + tag * 7919 + 12345) & ((1 << 62) - 1))
    return g


def _normal(shape, g, dtype):
    """N(0, 1) in dtype, drawn in pieces so that a large array needs no float32 copy."""
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        part = flat[i:i + (1 << 28)]
        part.copy_(torch.randn(part.shape, generator=g, device=DEV, dtype=torch.float32))
    return out


def _spread(lo, hi, S):
    return [lo + (i * (hi - lo)) // max(1, S - 1) for i in range(S)]


def _lens(lo, hi, S, seed):
    n = _spread(lo, hi, S)
    random.Random(seed).shuffle(n)
    return torch.tensor(n, dtype=torch.int32, device=DEV)


def _logits(R, V, g, dtype):
    x = torch.randn((R, V), generator=g, device=DEV, dtype=torch.float32).mul_(3.0)
    idx = torch.randint(0, V, (R, 5), generator=g, device=DEV)
    x.scatter_add_(1, idx, torch.full(idx.shape, 10.0, device=DEV))
    return x.to(dtype)


def _detector(R, g):
    """A detector past its guard, its window full."""
    det = kvr.Detector.zeros(R, device=DEV)
    det.hist.copy_(torch.rand((R, det.window), generator=g, device=DEV) * 9.0)
    det.cnt.fill_(30)
    return det


def _rows(case, g, dtype):
    """Logit rows of a step with their outputs: a LogitSet and, to draw tokens, the sampler and their array."""
    det = _detector(case["R"], g)
    lg = _logits(case["R"], case["V"], g, dtype)
    H = torch.zeros(case["R"], dtype=torch.float32, device=DEV)
    tok = torch.full((case["R"],), -1, dtype=torch.int32, device=DEV)
    return kvr.LogitSet(lg, H, case["V"], detector=det), kvr.Sampler(seed=11, step=7), tok


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return _RUN[state["kind"]](state)


def work(case):
    b, f = _WORK[case["kind"]](case)
    return {"bytes": b, "flops": f}


def tolerance(case):
    # Copies and selections are exact. bfloat16 outputs: half a unit in the
    # last place (2^-9) on the output and on the probabilities, about 3e-3 in
    # the 2-norm against the exact value. The largest single difference is a
    # few units of the output's rms. float32 sums: measured 1e-7 to 6e-7.
    if case["kind"] in ("evict", "fork"):
        return "exact"
    if case["kind"] in ("score", "sample") or case.get("dtype") == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2, "max": 0.1}


def exact(case, seed):
    f = _EXACT.get(case["kind"])
    return f(case, seed) if f else None


# Base decode: append, attend, window score, with the logit rows of the step.
def _prepare_decode(c, seed):
    g = _gen(seed, 1)
    dt = DT[c["dtype"]]
    S, L, Hq, Hkv, D, cap = (c[k] for k in ("S", "L", "Hq", "Hkv", "D", "cap"))
    k, v = _normal((S, L, Hkv, cap, D), g, dt), _normal((S, L, Hkv, cap, D), g, dt)
    pos = torch.arange(cap, dtype=torch.int32, device=DEV).repeat(S, L, Hkv, 1).contiguous()
    st = dict(kind="decode", cache=kvr.Cache(k, v, pos), scale=1.0 / math.sqrt(D),
              q=_normal((S, L, Hq, D), g, dt), kn=_normal((S, L, Hkv, D), g, dt), vn=_normal((S, L, Hkv, D), g, dt),
              len=_lens(c["n_lo"], c["n_hi"], S, seed), policy=kvr.Policy(c["B"], c["W"], c["buffer"]),
              pos=torch.full((S,), 5000, dtype=torch.int32, device=DEV),
              scores=torch.rand((S, L, Hkv, cap), generator=g, device=DEV) * 2.0,
              out=torch.zeros((S, L, Hq, D), dtype=dt, device=DEV), sets=None)
    if c["R"]:
        ls, smp, tok = _rows(c, g, DT[c["ldt"]])
        st.update(sets=[ls], sampler=smp if c["sample"] else None, tokens=[tok])
    return st


def _run_decode(s):
    kw = dict(k_new=s["kn"], v_new=s["vn"], new_pos=s["pos"], policy=s["policy"], scores=s["scores"])
    got = {"out": s["out"], "scores": s["scores"], "k": s["cache"].k, "v": s["cache"].v, "pos": s["cache"].pos}
    if s["sets"] is None:
        kvr.decode_attn(s["cache"], s["len"], s["q"], s["out"], s["scale"], **kw)
        return got
    ls = s["sets"][0]
    got.update(H=ls.H, hist=ls.detector.hist, cnt=ls.detector.cnt, flag=ls.detector.flag)
    if s["sampler"] is not None:
        kvr.decode_attn_entropy_sample(s["cache"], s["len"], s["q"], s["out"], s["scale"], s["sets"], s["sampler"],
                                       s["tokens"], **kw)
        got["tokens"] = s["tokens"][0]
    else:
        kvr.decode_attn_entropy(s["cache"], s["len"], s["q"], s["out"], s["scale"], s["sets"], **kw)
    return got


def _work_decode(c):
    e = ESZ[c["dtype"]]
    S, L, Hq, Hkv, D = (c[k] for k in ("S", "L", "Hq", "Hkv", "D"))
    n = _spread(c["n_lo"], c["n_hi"], S)
    wstart = c["B"] + c["buffer"] + 2 - c["W"]
    b = sum(n) * L * Hkv * D * 2 * e + S * L * Hkv * (2 * D * e + 4) + 2 * S * L * Hq * D * e
    b += sum((1 if x == wstart else 2) * 4 * x for x in n if x >= wstart) * L * Hkv
    f = 4 * sum(n) * L * Hq * D
    return b + c["R"] * (c["V"] * ESZ[c["ldt"]] + 8), f


def _entropy64(lg, inv_temp=1.0):
    out = []
    for r in range(lg.shape[0]):
        p = torch.log_softmax(lg[r].double() * inv_temp, 0)
        out.append(-(p.exp() * p).nan_to_num(0.0).sum())
    return torch.stack(out)


def _exact_decode(c, seed):
    s = _prepare_decode(c, seed)
    S, L, Hq, Hkv, D = (c[k] for k in ("S", "L", "Hq", "Hkv", "D"))
    G, wstart = Hq // Hkv, c["B"] + c["buffer"] + 2 - c["W"]
    out = torch.zeros((S, L, Hq, D), dtype=torch.float64, device=DEV)
    scores = s["scores"].double()
    for i, n in enumerate(s["len"].tolist()):
        k, v = s["cache"].k[i, :, :, :n].double(), s["cache"].v[i, :, :, :n].double()
        k[:, :, n - 1], v[:, :, n - 1] = s["kn"][i].double(), s["vn"][i].double()
        q = s["q"][i].double().view(L, Hkv, G, D)
        p = torch.softmax(torch.matmul(q, k.transpose(-1, -2).contiguous()) * s["scale"], -1)
        out[i] = torch.matmul(p, v).view(L, Hq, D)
        if n >= wstart:
            r = p.sum(2)
            old = scores[i, :, :, :n] if n > wstart else torch.zeros_like(r)
            old[:, :, n - 1] = 0.0
            scores[i, :, :, :n] = old + r
    got = {"out": out, "scores": scores, "k": None, "v": None, "pos": None}
    if c["R"]:
        got.update(H=_entropy64(s["sets"][0].logits), hist=None, cnt=None, flag=None)
        if c["sample"]:
            got["tokens"] = None
    return got


# Helper decode: context (shared or private) then the candidate's suffix.
def _prepare_context(c, seed):
    g = _gen(seed, 2)
    dt = torch.bfloat16
    S, P, L, Hq, Hkv, D = (c[k] for k in ("S", "P", "L", "Hq", "Hkv", "D"))
    pk, pv = _normal((P, L, Hkv, c["plen"], D), g, dt), _normal((P, L, Hkv, c["plen"], D), g, dt)
    k, v = _normal((S, L, Hkv, c["scap"], D), g, dt), _normal((S, L, Hkv, c["scap"], D), g, dt)
    cache, prefix = kvr.Cache(k, v, None), kvr.Prefix(pk, pv)
    ws = torch.empty(max(kvr.decode_attn_workspace_size(cache, prefix, Hq), 16) // 4 + 4, dtype=torch.float32, device=DEV)
    st = dict(kind="context", cache=cache, prefix=prefix, ws=ws, scale=1.0 / math.sqrt(D),
              q=_normal((S, L, Hq, D), g, dt), kn=_normal((S, L, Hkv, D), g, dt), vn=_normal((S, L, Hkv, D), g, dt),
              len=_lens(c["u_lo"], c["u_hi"], S, seed), out=torch.zeros((S, L, Hq, D), dtype=dt, device=DEV), sets=None)
    if c["R"]:
        ls, smp, tok = _rows(c, g, torch.bfloat16)
        st.update(sets=[ls], sampler=smp if c["sample"] else None, tokens=[tok])
    return st


def _run_context(s):
    kw = dict(k_new=s["kn"], v_new=s["vn"], prefix=s["prefix"], workspace=s["ws"])
    got = {"out": s["out"], "k": s["cache"].k, "v": s["cache"].v}
    if s["sets"] is None:
        kvr.decode_attn(s["cache"], s["len"], s["q"], s["out"], s["scale"], **kw)
        return got
    ls = s["sets"][0]
    got.update(H=ls.H, hist=ls.detector.hist, cnt=ls.detector.cnt, flag=ls.detector.flag)
    if s["sampler"] is not None:
        kvr.decode_attn_entropy_sample(s["cache"], s["len"], s["q"], s["out"], s["scale"], s["sets"], s["sampler"],
                                       s["tokens"], **kw)
        got["tokens"] = s["tokens"][0]
    else:
        kvr.decode_attn_entropy(s["cache"], s["len"], s["q"], s["out"], s["scale"], s["sets"], **kw)
    return got


def _work_context(c):
    S, P, L, Hq, Hkv, D = (c[k] for k in ("S", "P", "L", "Hq", "Hkv", "D"))
    u = sum(_spread(c["u_lo"], c["u_hi"], S))
    b = (P * c["plen"] + u + S) * L * Hkv * D * 4 + 2 * S * L * Hq * D * 2
    f = 4 * (S * c["plen"] + u) * L * Hq * D
    return b + c["R"] * (c["V"] * 2 + 8), f


def _exact_context(c, seed):
    s = _prepare_context(c, seed)
    S, P, L, Hq, Hkv, D = (c[k] for k in ("S", "P", "L", "Hq", "Hkv", "D"))
    G, C = Hq // Hkv, S // P
    out = torch.zeros((S, L, Hq, D), dtype=torch.float64, device=DEV)
    lens = s["len"].tolist()
    for p in range(P):
        for l in range(L):
            pk, pv = s["prefix"].k[p, l].double(), s["prefix"].v[p, l].double()
            pkt = pk.transpose(-1, -2).contiguous()
            for i in range(p * C, p * C + C):
                n = lens[i]
                k, v = s["cache"].k[i, l, :, :n].double(), s["cache"].v[i, l, :, :n].double()
                k[:, n - 1], v[:, n - 1] = s["kn"][i, l].double(), s["vn"][i, l].double()
                q = s["q"][i, l].double().view(Hkv, G, D)
                x = torch.cat([torch.matmul(q, pkt), torch.matmul(q, k.transpose(-1, -2).contiguous())], -1)
                w = torch.softmax(x * s["scale"], -1)
                o = torch.matmul(w[..., : c["plen"]].contiguous(), pv) + torch.matmul(w[..., c["plen"]:].contiguous(), v)
                out[i, l] = o.view(Hq, D)
    got = {"out": out, "k": None, "v": None}
    if c["R"]:
        got.update(H=_entropy64(s["sets"][0].logits), hist=None, cnt=None, flag=None)
        if c["sample"]:
            got["tokens"] = None
    return got


# Commit and prompt compression: bulk append, then the window scores.
def _prepare_score(c, seed):
    g = _gen(seed, 3)
    dt = DT[c["dtype"]]
    S, L, Hq, Hkv, D, cap, T = (c[k] for k in ("S", "L", "Hq", "Hkv", "D", "cap", "T"))
    k, v = _normal((S, L, Hkv, cap, D), g, dt), _normal((S, L, Hkv, cap, D), g, dt)
    pos = torch.arange(cap, dtype=torch.int32, device=DEV).repeat(S, L, Hkv, 1).contiguous()
    ln = _lens(c["n_lo"], c["n_hi"], S, seed)
    return dict(kind="score", cache=kvr.Cache(k, v, pos), scale=1.0 / math.sqrt(D), len0=ln, len1=ln + T,
                kn=_normal((S, L, Hkv, T, D), g, dt), vn=_normal((S, L, Hkv, T, D), g, dt),
                pn=(torch.arange(T, dtype=torch.int32, device=DEV) + 7000).repeat(S, 1).contiguous(),
                qw=_normal((S, L, Hq, c["nq"], D), g, dt),
                scores=torch.zeros((S, L, Hkv, cap), dtype=torch.float32, device=DEV))


def _run_score(s):
    kvr.append(s["cache"], s["len0"], s["kn"], s["vn"], s["pn"])
    kvr.accumulate_scores(s["cache"], s["len1"], s["qw"], s["scale"], s["scores"])
    return {"scores": s["scores"], "k": s["cache"].k, "v": s["cache"].v, "pos": s["cache"].pos}


def _work_score(c):
    e = ESZ[c["dtype"]]
    S, L, Hq, Hkv, D, T, nq = (c[k] for k in ("S", "L", "Hq", "Hkv", "D", "T", "nq"))
    n = sum(x + T for x in _spread(c["n_lo"], c["n_hi"], S))
    b = 2 * S * L * Hkv * T * (2 * D * e + 4) + (n - S * T) * L * Hkv * D * e + S * L * Hq * nq * D * e + 4 * n * L * Hkv
    return b, 2 * n * L * Hq * nq * D


def _exact_score(c, seed):
    s = _prepare_score(c, seed)
    S, L, Hq, Hkv, D, T, nq = (c[k] for k in ("S", "L", "Hq", "Hkv", "D", "T", "nq"))
    G = Hq // Hkv
    scores = torch.zeros(s["scores"].shape, dtype=torch.float64, device=DEV)
    for i, n0 in enumerate(s["len0"].tolist()):
        n = n0 + T
        late = torch.arange(n, device=DEV)[None, :] >= n - (nq - 1 - torch.arange(nq, device=DEV))[:, None]
        for l in range(L):
            k = torch.cat([s["cache"].k[i, l, :, :n0], s["kn"][i, l]], 1).double()
            x = torch.matmul(s["qw"][i, l].double().view(Hkv, G * nq, D), k.transpose(-1, -2).contiguous())
            x = (x * s["scale"]).view(Hkv, G, nq, n).masked_fill(late, -math.inf)
            scores[i, l, :, :n] = torch.softmax(x, -1).sum((1, 2))
    return {"scores": scores, "k": None, "v": None, "pos": None}


# Eviction of every overflowing sequence.
def _prepare_evict(c, seed):
    g = _gen(seed, 4)
    dt = DT[c["dtype"]]
    S, L, Hkv, D, cap = (c[k] for k in ("S", "L", "Hkv", "D", "cap"))
    pos = torch.arange(cap, dtype=torch.int32, device=DEV).repeat(S, L, Hkv, 1).contiguous()
    scores = -torch.log1p(-torch.rand((S, L, Hkv, cap), generator=g, device=DEV))
    return dict(kind="evict", cache=kvr.Cache(_normal((S, L, Hkv, cap, D), g, dt), _normal((S, L, Hkv, cap, D), g, dt), pos),
                len=_lens(c["n_lo"], c["n_hi"], S, seed), policy=kvr.Policy(c["B"], c["W"], c["buffer"]), scores=scores,
                kept=torch.zeros((S, L, Hkv, c["B"]), dtype=torch.int32, device=DEV),
                len_out=torch.zeros(S, dtype=torch.int32, device=DEV))


def _run_evict(s):
    kvr.evict_topb(s["cache"], s["len"], s["scores"], s["policy"], kept=s["kept"], len_out=s["len_out"])
    return {"k": s["cache"].k, "v": s["cache"].v, "pos": s["cache"].pos, "kept": s["kept"], "len": s["len_out"]}


def _work_evict(c):
    # Every kept slot past the first few moves.
    S, L, Hkv, D, B, W = (c[k] for k in ("S", "L", "Hkv", "D", "B", "W"))
    n = [x for x in _spread(c["n_lo"], c["n_hi"], S) if x > B + c["buffer"]]
    b = sum(4 * (x - W) + 4 * B + 2 * B * (2 * D * ESZ[c["dtype"]] + 4) for x in n) * L * Hkv
    return b + 8 * S, 0


# Fork of the trajectory states to their candidates.
def _prepare_fork(c, seed):
    g = _gen(seed, 5)
    dt = DT[c["dtype"]]
    P, N, L, Hkv, D, cap = (c[k] for k in ("P", "N", "L", "Hkv", "D", "cap"))
    pos = torch.arange(cap, dtype=torch.int32, device=DEV).repeat(P, L, Hkv, 1).contiguous()
    src = kvr.Cache(_normal((P, L, Hkv, cap, D), g, dt), _normal((P, L, Hkv, cap, D), g, dt), pos)
    dst = kvr.Cache.empty(P * N, L, Hkv, cap, D, dt, DEV)
    dst.k.zero_()
    dst.v.zero_()
    return dict(kind="fork", src=src, dst=dst, ssc=torch.rand((P, L, Hkv, cap), generator=g, device=DEV),
                dsc=torch.zeros((P * N, L, Hkv, cap), device=DEV),
                idx=(torch.arange(P * N, dtype=torch.int32, device=DEV) // N).contiguous(),
                len=_lens(c["n_lo"], c["n_hi"], P, seed).repeat_interleave(N).contiguous())


def _run_fork(s):
    kvr.fork(s["src"], s["dst"], s["idx"], s["len"], s["ssc"], s["dsc"])
    return {"k": s["dst"].k, "v": s["dst"].v, "pos": s["dst"].pos, "scores": s["dsc"]}


def _work_fork(c):
    n = sum(_spread(c["n_lo"], c["n_hi"], c["P"]))
    return (1 + c["N"]) * n * c["L"] * c["Hkv"] * (2 * c["D"] * ESZ[c["dtype"]] + 8), 0


# Entropy, detector and token draw of logit rows.
def _prepare_sample(c, seed):
    g = _gen(seed, 6)
    ls, smp, tok = _rows(c, g, DT[c["ldt"]])
    smp = kvr.Sampler(top_k=c["top_k"], seed=11, step=7)
    ws = torch.empty(max(kvr.logit_entropy_sample_workspace_size(c["R"], c["V"], c["top_k"]), 16) // 4 + 4,
                     dtype=torch.float32, device=DEV)
    return dict(kind="sample", ls=ls, sampler=smp, tokens=tok, ws=ws)


def _run_sample(s):
    ls = s["ls"]
    kvr.logit_entropy_sample(ls.logits, ls.H, s["tokens"], s["sampler"], V=ls.V, detector=ls.detector, workspace=s["ws"])
    return {"H": ls.H, "tokens": s["tokens"], "hist": ls.detector.hist, "cnt": ls.detector.cnt, "flag": ls.detector.flag}


def _work_sample(c):
    return c["R"] * (c["V"] * ESZ[c["ldt"]] + 12), 0


def _exact_sample(c, seed):
    s = _prepare_sample(c, seed)
    return {"H": _entropy64(s["ls"].logits), "tokens": None, "hist": None, "cnt": None, "flag": None}


_PREPARE = dict(decode=_prepare_decode, context=_prepare_context, score=_prepare_score, evict=_prepare_evict,
                fork=_prepare_fork, sample=_prepare_sample)
_RUN = dict(decode=_run_decode, context=_run_context, score=_run_score, evict=_run_evict, fork=_run_fork,
            sample=_run_sample)
_WORK = dict(decode=_work_decode, context=_work_context, score=_work_score, evict=_work_evict, fork=_work_fork,
             sample=_work_sample)
_EXACT = dict(decode=_exact_decode, context=_exact_context, score=_exact_score, sample=_exact_sample)
