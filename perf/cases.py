"""The work a user of this library has it do, as timed cases.

A case is one call (or, for a whole stream, one pass of calls) of the step entry points on one layer:
decoding one token, encoding a chunk, the options of both, and a short document from its first token to
its last.  `prepare` brings the layer to the step's past length through the same entry points a program
uses (append and unit construction, chunk by chunk), so that the step meets a real memory.

Shapes are the layer shapes of the repository's workloads (32 query and 8 kv heads of 128 dims, 128
initial tokens, a 4K window, 128-token units) and smaller or odd ones of the same kinds.
"""
from __future__ import annotations

import math

import torch

from paper_2402_04617_amd import infllm as F

_LAYER = dict(kind="step", dtype="bf16", hq=32, hkv=8, d=128, init=128, local=4096, block=128, repr=4, topk=32,
              batch=1, spread=0, repr_mode="tokens", remap=False, mass=False, prefill=512)
_DECAY = 0.1         # of the frequency scores
_ROPE_BASE = 500000.0


def _case(**kw):
    c = dict(_LAYER)
    c.update(kw)
    return c


def listed():
    return [
        # one user's generation over a 32K document: the smallest call, a token through one layer
        _case(name="decode_1x32k", past=31999, n=1, topk=16),
        # serving: a full batch of long documents, one token each
        _case(name="decode_16x128k", batch=16, past=131100, n=1),
        # serving, sequences at their own depths, down to one whose context fits the window
        _case(name="decode_varlen_8", kind="varlen", batch=8, past=120007, spread=118000, n=1),
        # a prompt that fits the window: nothing has been evicted yet, and no chunk precedes it
        _case(name="prompt_300", past=0, n=300),
        # the flagship: a chunk near the end of a 128K document
        _case(name="chunk_128k", past=130048, n=512),
        # the same with the rotary encoding applied by the library (memory at distance l_L)
        _case(name="chunk_128k_remap", past=130048, n=512, remap=True),
        # the same with the attention mass and frequency score of the cache policy
        _case(name="chunk_128k_mass", past=130048, n=512, mass=True),
        # the ragged last chunk of a 32K document, units scored by their mean key
        _case(name="chunk_32k_mean_ragged", past=30720, n=389, topk=16, repr_mode="mean"),
        # a chunk near the end of a 1M document at the long-context settings
        _case(name="chunk_1m", past=1046528, n=2048, repr=1, prefill=2048),
        # chunked prefill of several users at their own depths, a few tokens each (also what a
        # speculative verification step looks like)
        _case(name="extend_varlen_4", kind="varlen", batch=4, past=65001, spread=50000, n=24),
        # float32 throughout: the accuracy path, a chunk of a smaller layer
        _case(name="chunk_f32", dtype="f32", hq=8, hkv=2, d=64, past=16000, n=256, init=64, local=1024, block=64,
              topk=16, prefill=256),
        # a whole 32K document from its first token, chunk by chunk
        _case(name="document_32k", kind="stream", past=0, n=32768, topk=16),
    ]


def draw(rng):
    """One more case of these ranges."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def group():
        return rng.choice((1, 2, 4, 4, 8))

    block = rng.choice((64, 128, 128, 256))
    topk = rng.choice((8, 16, 32, 48))
    common = dict(block=block, topk=min(topk, 8192 // block), repr=rng.choice((1, 2, 4, 8)), d=rng.choice((64, 128, 128)))
    what = rng.choice(("decode", "decode", "varlen", "chunk", "chunk", "chunk", "option", "option", "f32"))
    if what == "decode":
        hkv = rng.choice((2, 4, 8))
        return _case(hkv=hkv, hq=hkv * group(), batch=log_int(1, 16), past=log_int(1500, 131000), n=1, **common)
    if what == "varlen":
        past = log_int(12000, 120000)
        return _case(kind="varlen", hq=8 * group(), batch=rng.randint(2, 8), past=past, n=rng.choice((1, 1, log_int(2, 400))),
                     spread=rng.randint(past // 2, past - 1), **common)
    if what == "f32":
        g = rng.choice((1, 2, 4))
        common.update(d=64, block=64)
        return _case(dtype="f32", hkv=2, hq=2 * g, past=log_int(1000, 30000), n=log_int(16, 300), init=64, local=1024,
                     prefill=256, **common)
    n = log_int(16, 1500)
    if what == "option":
        mode = rng.choice(("remap", "mass", "mean"))
        return _case(hq=8 * group(), past=log_int(6000, 131000), n=n, remap=mode == "remap", mass=mode == "mass",
                     repr_mode="mean" if mode == "mean" else "tokens", **common)
    return _case(hq=8 * group(), past=log_int(1000, 400000), n=n, **common)


# ------------------------------------------------------------------ geometry of a case
def _pasts(c):
    """Past length of each sequence."""
    if c["kind"] != "varlen":
        return [c["past"]] * c["batch"]
    return [c["past"] - (c["spread"] * b) // max(1, c["batch"] - 1) for b in range(c["batch"])]


def _units(c, past):
    return max(0, (past - c["init"] - c["local"]) // c["block"])


def _steps(c):
    """(past, n, units already built) of the calls of one pass (the first sequence's, for a batch)."""
    if c["kind"] != "stream":
        return [(c["past"], c["n"], 0)]
    steps, built = [], 0
    for p in range(0, c["n"], c["prefill"]):
        steps.append((p, min(c["prefill"], c["n"] - p), built))
        built = _units(c, p)
    return steps


def _params(c):
    return F.params(c["hq"], c["hkv"], c["d"], c["init"], c["local"], c["block"], c["repr"], c["topk"],
                    dtype=c["dtype"], sm_scale=c["d"] ** -0.5,
                    rope_inv_freq=F.rope_frequencies(c["d"], _ROPE_BASE) if c["remap"] else None,
                    repr_mode=c["repr_mode"])


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


# ------------------------------------------------------------------ inputs
def _sequence(c, seed, b, length):
    """q [Hq][length][D], k, v [Hkv][length][D] of one sequence: unit-variance queries and keys (logits of
    unit variance), and a few units whose keys lean along a direction that every 8th query shares (logits
    about 4 higher), as a passage that the text refers to again and again has."""
    g = torch.Generator(device="cuda").manual_seed((seed * 1000003 + b * 7919 + 17) % (1 << 62))
    dt, d, hkv = _dtype(c), c["d"], c["hkv"]
    q = torch.randn((c["hq"], length, d), generator=g, device="cuda", dtype=dt)
    k = torch.randn((hkv, length, d), generator=g, device="cuda", dtype=dt)
    v = torch.randn((hkv, length, d), generator=g, device="cuda", dtype=dt)
    lean = torch.randn((hkv, 1, d), generator=g, device="cuda", dtype=torch.float32)
    lean = (lean / lean.norm(dim=-1, keepdim=True) * (4.0 * d ** 0.5) ** 0.5).to(dt)
    n_units = _units(c, length)
    if n_units:
        for u in torch.randint(0, n_units, (4,), generator=g, device="cuda").tolist():
            t0 = c["init"] + u * c["block"]
            k[:, t0:t0 + c["block"]] += lean
    q.view(hkv, c["hq"] // hkv, length, d)[:, :, ::8] += lean[:, None]
    return q, k, v


def _one_sequence(p, mem, b):
    """A one-sequence view of a layer's memory."""
    s = mem.struct
    row = lambda t: t[b].data_ptr() if t is not None else None  # noqa: E731
    return F.Memory(1, s.capacity, row(mem.k), row(mem.v), s.max_units, row(mem.repr_idx), row(mem.unit_ksum),
                    row(mem.qprefix), row(mem.rpart), s.ring, row(mem.k_rot))


def prepare(case, seed):
    c = case
    p = _params(c)
    B, n, d, dt = c["batch"], c["n"], c["d"], _dtype(c)
    pasts = _pasts(c)
    stream = c["kind"] == "stream"
    chunk = c["prefill"] if stream else n
    capacity = (max(pasts) + n + 255) // 256 * 256
    max_units = max(1, (_units(c, capacity) + 7) // 8 * 8)
    ring = F.recommended_ring(p, max(chunk, c["prefill"]))
    mem = F.alloc_memory(p, B, capacity, max_units, ring)
    q = torch.empty((B, c["hq"], n, d), dtype=dt, device="cuda")
    k = torch.empty((B, c["hkv"], n, d), dtype=dt, device="cuda")
    v = torch.empty_like(k)
    built = []
    for b, past in enumerate(pasts):
        qs, ks, vs = _sequence(c, seed, b, past + n)
        q[b], k[b], v[b] = qs[:, past:], ks[:, past:], vs[:, past:]
        one, stride, es, done = _one_sequence(p, mem, b), (past + n) * d, qs.element_size(), 0
        for t in range(0, past, c["prefill"]):
            m = min(c["prefill"], past - t)
            now = _units(c, t)
            if now > done:
                F.infllm_build_units(p, one, done, now - done, t)
                done = now
            F.infllm_append(p, one, qs.data_ptr() + t * d * es, stride, ks.data_ptr() + t * d * es,
                            vs.data_ptr() + t * d * es, stride, m, t)
        # the units of an earlier step are built; those that a decoding step finds evicted mostly are none
        if n == 1 and past > 0 and _units(c, past - 1) > done:
            F.infllm_build_units(p, one, done, _units(c, past - 1) - done, past)
            done = _units(c, past - 1)
        built.append(done)
        torch.cuda.synchronize()
        del qs, ks, vs
    st = {"case": dict(c), "p": p, "mem": mem, "q": q, "k": k, "v": v, "pasts": pasts, "built": built}
    st["out"] = torch.zeros((B, c["hq"], n, d), dtype=dt, device="cuda")
    st["lse"] = torch.zeros((B * c["hq"] * n,), dtype=torch.float32, device="cuda")
    nu = _units(c, pasts[0])
    st["scores"] = torch.zeros((B, c["hkv"], max_units if c["kind"] == "varlen" or stream else max(1, nu)),
                               dtype=torch.float32, device="cuda")
    st["idx"] = torch.zeros((B, c["hkv"], c["topk"]), dtype=torch.int32, device="cuda")
    st["ws"] = torch.zeros(F.infllm_workspace_bytes(p, B, chunk), dtype=torch.uint8, device="cuda")
    if c["mass"]:
        st["mass"] = torch.zeros((B, c["hkv"], c["topk"]), dtype=torch.float32, device="cuda")
        st["freq"] = torch.ones((B, c["hkv"], max_units), dtype=torch.float32, device="cuda")
    st["outputs"] = _outputs(st)
    return st


def _ring_views(t, dim, ring, first, count):
    """The slots of positions [first, first + count) in a ring, as one or two views."""
    if count <= 0:
        return []
    s = first % ring
    m = min(count, ring - s)
    views = [t.narrow(dim, s, m)]
    if m < count:
        views.append(t.narrow(dim, 0, count - m))
    return views


def _outputs(st):
    """What the calls write: the attention's rows, the lookup, and the memory they extend."""
    c, mem = st["case"], st["mem"]
    o = {"out": st["out"], "lse": st["lse"], "idx": st["idx"], "ksum": mem.unit_ksum}
    if c["repr_mode"] == "tokens":
        o["repr_idx"] = mem.repr_idx
    if c["mass"]:
        o["mass"], o["freq"] = st["mass"], st["freq"]
    if c["kind"] == "stream":
        o["k"], o["v"] = mem.k[:, :, :c["n"]], mem.v[:, :, :c["n"]]
        return o
    if c["kind"] == "varlen":
        o["scores"] = [st["scores"][b, :, :_units(c, past)] for b, past in enumerate(st["pasts"])]
    elif _units(c, c["past"]):
        o["scores"] = st["scores"]
    n, ring = c["n"], mem.struct.ring
    rows = []
    for b, past in enumerate(st["pasts"] if c["kind"] == "varlen" else st["pasts"][:1]):
        at = slice(b, b + 1) if c["kind"] == "varlen" else slice(None)
        r = {"k": mem.k[at, :, past:past + n], "v": mem.v[at, :, past:past + n]}
        if c["remap"]:
            r["k_rot"] = mem.k_rot[at, :, past:past + n]
        if c["repr_mode"] == "tokens":
            r["qsum"] = _ring_views(mem.qprefix[at], 2, ring, past, n)
            t0 = max(c["init"], past - c["local"])
            r["rpart"] = _ring_views(mem.rpart[at], 3, ring, t0, past + n - c["local"] - t0)
        rows.append(r)
    o["rows"] = rows
    return o


def run(state):
    s = state
    c, p, m, d = s["case"], s["p"], s["mem"].struct, s["case"]["d"]
    n = c["n"]
    if c["kind"] == "varlen":
        F.infllm_step_varlen(p, m, s["q"], n * d, s["k"], s["v"], n * d, n, s["pasts"], s["built"], s["scores"],
                             s["idx"], s["out"], n * d, s["lse"], s["ws"])
    elif c["kind"] == "stream":
        es = s["q"].element_size()
        q0, k0, v0, o0, l0 = (s[x].data_ptr() for x in ("q", "k", "v", "out", "lse"))
        for past, nq, built in _steps(c):
            off = past * d * es
            F.infllm_step(p, m, q0 + off, n * d, k0 + off, v0 + off, n * d, nq, past, built, s["scores"], s["idx"],
                          o0 + off, n * d, l0 + past * c["hq"] * 4, s["ws"])
    elif c["mass"]:
        F.infllm_step_mass(p, m, s["q"], n * d, s["k"], s["v"], n * d, n, c["past"], s["built"][0], s["scores"],
                           s["idx"], s["out"], n * d, s["lse"], _DECAY, s["mass"], s["freq"], s["ws"])
    else:
        F.infllm_step(p, m, s["q"], n * d, s["k"], s["v"], n * d, n, c["past"], s["built"][0], s["scores"],
                      s["idx"], s["out"], n * d, s["lse"], s["ws"])
    return s["outputs"]


# ------------------------------------------------------------------ work, tolerance
def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    total = {"bytes": 0.0, "flops": 0.0}
    steps = [(past, n) for past, n, _ in _steps(c)] if c["kind"] == "stream" else [(past, c["n"]) for past in _pasts(c)]
    for past, n in steps:
        nu = _units(c, past)
        ctx = min(past, c["init"]) + min(c["topk"], nu) * c["block"] + max(0, past - min(past, c["init"]) - nu * c["block"])
        b = 2 * hq * n * d * e + hq * n * 4                      # queries in, rows out, lse
        b += 2 * 2 * hkv * n * d * e                             # the chunk's keys and values, in and into the store
        b += 2 * hkv * ctx * d * e                               # the attended keys and values
        b += hkv * nu * (d + 1) * 4 + hkv * c["topk"] * 4        # unit vectors, scores, the lookup
        if c["repr_mode"] == "tokens":
            b += 2 * hkv * n * d * 8                             # running query sums: written, and those that leave the window
        if c["remap"]:
            b += hkv * n * d * e                                 # rotated keys
        if c["mass"]:
            b += hkv * (2 * nu + c["topk"]) * 4                  # frequency scores, masses
        total["bytes"] += b
        total["flops"] += 4.0 * d * hq * (n * ctx + n * (n + 1) / 2) + 2.0 * hkv * nu * d
    return total


def tolerance(case):
    # Correct forms differ in the order of the sums and in the running maximum that a probability is
    # rounded to bf16 against: rows of bf16 differ by 2.6e-3 of their norm and by up to 0.03 of their root
    # mean square (a bf16 step of the larger values); float32 rows by 4e-7 and 4e-6.  The masses and float32
    # state agree far closer.
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.12, "differ": 0.002}
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.002}


# ------------------------------------------------------------------ 64-bit values
def _rotate(x, pos, freqs):
    """x [..., n, d] turned to positions pos [n] (interleaved pairs)."""
    a = pos.to(torch.float64)[:, None] * freqs
    c, s = a.cos(), a.sin()
    e, o = x[..., 0::2], x[..., 1::2]
    return torch.stack((e * c - o * s, e * s + o * c), dim=-1).flatten(-2)


def _exact_head(c, q, k, v, steps, freqs):
    """One (sequence, kv head) in 64 bits: q [G][S][D], k, v [S][D].  Per step (past, n): rows, lse, scores,
    lookup, mass; and for the whole sequence the unit vectors and representative parts."""
    f64 = torch.float64
    dev = k.device
    S, d = k.shape
    G = q.shape[0]
    k, v = k.to(f64), v.to(f64)
    pos = torch.arange(S, device=dev)
    krot = _rotate(k, pos, freqs) if c["remap"] else k
    qsum = q.to(f64).sum(0)
    r = {"steps": [], "krot": krot}
    nu_all = _units(c, steps[-1][0])
    lo, hi = c["init"], c["init"] + nu_all * c["block"]
    ksum = None
    if c["repr_mode"] == "tokens":
        run = (_rotate(qsum, pos, freqs) if c["remap"] else qsum).cumsum(0)
        r["run"] = run
        t_hi = S - c["local"]
        if t_hi > lo:
            r["t0"] = lo
            part = krot[lo:t_hi] * (run[lo + c["local"]:t_hi + c["local"]] - run[lo:t_hi])
            r["rpart"] = part.view(t_hi - lo, d // 8, 8).sum(-1).T.contiguous()
            del part
        if nu_all:
            score = r["rpart"].sum(0)[:hi - lo].view(nu_all, c["block"])
            rep = score.topk(c["repr"], dim=1).indices.sort(dim=1).values
            ksum = k[lo:hi].view(nu_all, c["block"], d).gather(1, rep[..., None].expand(-1, -1, d)).sum(1)
    elif nu_all:
        ksum = k[lo:hi].view(nu_all, c["block"], d).mean(1)
    r["ksum"] = ksum
    for past, n in steps:
        nu = _units(c, past)
        x = q[:, past:past + n].to(f64)
        scores, sel = torch.zeros(0, dtype=f64, device=dev), torch.zeros(0, dtype=torch.int64, device=dev)
        far = torch.full((1,), c["local"], device=dev)
        if nu:
            qbar = qsum[past:past + n].sum(0)[None]
            if c["remap"]:
                qbar = _rotate(qbar, far, freqs)
            scores = ksum[:nu] @ qbar[0]
            sel = scores.topk(min(c["topk"], nu)).indices.sort().values
        i0 = min(past, c["init"])
        mem = torch.cat((pos[:i0], (c["init"] + sel[:, None] * c["block"] + pos[:c["block"]][None] if sel.numel()
                                    else pos[:0]).reshape(-1)))
        loc = pos[i0 + nu * c["block"]:past + n]
        xm, xl = x, x
        if c["remap"]:
            xm = _rotate(x, far.expand(n), freqs)
            xl = _rotate(x, pos[past:past + n], freqs)
        z = torch.cat((xm.reshape(G * n, d) @ k[mem].T, xl.reshape(G * n, d) @ krot[loc].T), dim=1) * d ** -0.5
        z = z.view(G, n, -1)
        z[:, :, mem.numel():].masked_fill_(loc[None, :] > pos[past:past + n, None], -math.inf)
        lse = z.logsumexp(-1)
        pr = (z - lse[..., None]).exp_()
        o = pr.view(G * n, -1) @ torch.cat((v[mem], v[loc]))
        mass = None
        if c["mass"]:
            mass = torch.zeros(c["topk"], dtype=f64, device=dev)
            mass[:sel.numel()] = pr[:, :, i0:mem.numel()].sum((0, 1)).view(-1, c["block"]).sum(-1)
        r["steps"].append((o.view(G, n, d), lse, scores, sel, mass))
        del z, pr
    return r


def exact(case, seed):
    c = case
    f64, dev = torch.float64, "cuda"
    B, n, d, hkv, G = c["batch"], c["n"], c["d"], c["hkv"], c["hq"] // c["hkv"]
    pasts = _pasts(c)
    stream, varlen = c["kind"] == "stream", c["kind"] == "varlen"
    freqs = torch.tensor([_ROPE_BASE ** (-2.0 * i / d) for i in range(d // 2)], dtype=f64, device=dev)
    capacity = (max(pasts) + n + 255) // 256 * 256
    max_units = max(1, (_units(c, capacity) + 7) // 8 * 8)
    ring = c["local"] + c["block"] + 2 * max(c["prefill"], c["prefill"] if stream else n) + 1
    out = torch.zeros((B, c["hq"], n, d), dtype=f64, device=dev)
    lse = torch.zeros((B, c["hq"], n), dtype=f64, device=dev)
    lse_steps = []
    ksum = torch.zeros((B, hkv, d // 4, max_units, 4), dtype=f64, device=dev)
    mass = torch.zeros((B, hkv, c["topk"]), dtype=f64, device=dev)
    freq = torch.ones((B, hkv, max_units), dtype=f64, device=dev)
    scores, rows = [], []
    for b, past in enumerate(pasts):
        q, k, v = _sequence(c, seed, b, past + n)
        steps = [(s, m) for s, m, _ in _steps(c)] if stream else [(past, n)]
        nu = _units(c, steps[-1][0])
        sc = torch.zeros((hkv, nu), dtype=f64, device=dev)
        qrows, prow, krot = [], [], []
        for g in range(hkv):
            r = _exact_head(c, q[g * G:(g + 1) * G], k[g], v[g], steps, freqs)
            for i, (s, m) in enumerate(steps):
                at = s if stream else 0
                out[b, g * G:(g + 1) * G, at:at + m] = r["steps"][i][0]
                lse[b, g * G:(g + 1) * G, at:at + m] = r["steps"][i][1]
            if nu:
                sc[g] = r["steps"][-1][2]
                ksum[b, g, :, :nu] = r["ksum"].view(nu, d // 4, 4).permute(1, 0, 2)
            if c["mass"]:
                sel = r["steps"][-1][3]
                mass[b, g] = r["steps"][-1][4]
                freq[b, g, :nu] *= _DECAY
                freq[b, g, sel] += mass[b, g, :sel.numel()]
            if stream:
                continue
            if c["remap"]:
                krot.append(r["krot"][past:])
            if c["repr_mode"] == "tokens":
                qrows.append(r["run"][past:])
                t0 = max(c["init"], past - c["local"])
                if past + n - c["local"] > t0:
                    prow.append(r["rpart"][:, t0 - r["t0"]:])
            del r
        scores.append(sc)
        if not stream:
            x = {"k": k[None, :, past:], "v": v[None, :, past:]}
            if c["remap"]:
                x["k_rot"] = torch.stack(krot)[None]
            if c["repr_mode"] == "tokens":
                m = min(n, ring - past % ring)
                t = torch.stack(qrows)[None]
                x["qsum"] = [t[:, :, :m]] + ([t[:, :, m:]] if m < n else [])
                x["rpart"] = []
                if prow:
                    t = torch.stack(prow)[None]
                    t0 = max(c["init"], past - c["local"])
                    m = min(t.shape[3], ring - t0 % ring)
                    x["rpart"] = [t[..., :m]] + ([t[..., m:]] if m < t.shape[3] else [])
            rows.append(x)
        del q, k, v
    if stream:  # lse rows lie chunk by chunk, [Hq][chunk]
        for s, m, _ in _steps(c):
            lse_steps.append(lse[0, :, s:s + m].reshape(-1))
        lse = torch.cat(lse_steps)
    o = {"out": out, "lse": lse.reshape(-1), "idx": None, "ksum": ksum}
    if c["repr_mode"] == "tokens":
        o["repr_idx"] = None
    if c["mass"]:
        o["mass"], o["freq"] = mass, freq
    if stream:
        o["k"] = o["v"] = None
        return o
    if varlen:
        o["scores"], o["rows"] = scores, rows
        return o
    if _units(c, c["past"]):
        o["scores"] = torch.stack(scores)
    first = rows[0]
    o["rows"] = [{name: ([torch.cat([r[name][i] for r in rows]) for i in range(len(first[name]))]
                         if isinstance(first[name], list) else torch.cat([r[name] for r in rows])) for name in first}]
    return o
