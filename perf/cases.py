"""The workloads that users of this library run, as cases to time and to check.

A case is one call of the library's public entry points on inputs resident in
device memory, through the prepared calls that a decode loop keeps:

* ``step``   one fused decode step (scan, selection, sparse attention), where
  ``grow`` is set with the new token's KV write and the builds of the pages that
  it fills, as a batched generation loop runs it;
* ``build``  every page summary of a prefilled context, at each page size;
* ``dense``  paged decode attention over every token, for the layers and the short
  contexts that are kept dense;
* ``kivi``   the fake quantisation of every finalised page.

Keys, queries and values are seeded synthetic draws with the structure that page
summaries are meant for: a mean per KV head with a few outlier channels, pages that
drift along a few directions shared by the sequence, and an eight-dimensional
spread inside each page.  The records that a step scans are encoded here from the
factors that the keys are drawn from, so a step's inputs do not depend on the
library's own build.
"""
import math
import random

import numpy as np
import torch

from paper_2607_24555_amd import locks as B

D = 128
SUB = 8            # directions inside a page, and shared drift directions
TORCH_OF = {"bf16": torch.bfloat16, "fp32": torch.float32}
LOCKS_OF = {"bf16": B.LOCKS_BF16, "fp32": B.LOCKS_FP32}


def _step(name, seqs, lo, hi, q_heads, kv_heads, rank, budget, page=16, basis="int4",
          dtype="bf16", grow=False):
    c = {"op": "step", "seqs": seqs, "lo": lo, "hi": hi, "q_heads": q_heads,
         "kv_heads": kv_heads, "rank": rank, "budget": budget, "page": page, "basis": basis,
         "dtype": dtype, "grow": grow}
    return dict(c, name=name) if name else c


def _build(name, seqs, lo, hi, kv_heads, rank, page, dtype="bf16"):
    c = {"op": "build", "seqs": seqs, "lo": lo, "hi": hi, "q_heads": 4 * kv_heads,
         "kv_heads": kv_heads, "rank": rank, "budget": 2048, "page": page, "basis": "int4",
         "dtype": dtype, "grow": False}
    return dict(c, name=name) if name else c


def _dense(name, seqs, lo, hi, q_heads, kv_heads, dtype="bf16"):
    c = {"op": "dense", "seqs": seqs, "lo": lo, "hi": hi, "q_heads": q_heads,
         "kv_heads": kv_heads, "rank": 8, "budget": 2048, "page": 16, "basis": "int4",
         "dtype": dtype, "grow": False}
    return dict(c, name=name) if name else c


def _kivi(name, seqs, lo, hi, kv_heads, bits):
    c = {"op": "kivi", "seqs": seqs, "lo": lo, "hi": hi, "q_heads": 4 * kv_heads,
         "kv_heads": kv_heads, "rank": 8, "budget": 2048, "page": 16, "basis": "int4",
         "dtype": "bf16", "grow": False, "bits": bits}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one head, 4K tokens, fp32 (the workload "tiny-1h-4k")
        _step("step-4k-fp32", 1, 4096, 4096, 1, 1, 8, 256, dtype="fp32"),
        # one user's 32K chat: latency and launches count ("llama8b-32k")
        _step("step-32k", 1, 32768, 32768, 32, 8, 8, 2048),
        # long documents, a batch of eight at 128K ("llama8b-8x128k")
        _step("step-8x128k", 8, 131072, 131072, 32, 8, 8, 2048),
        # the same in the largest pages that the store takes
        _step("step-8x128k-page64", 8, 131072, 131072, 32, 8, 8, 2048, page=64),
        # the longest context, sixteen heads a group ("glm4-9b-1m")
        _step("step-1m", 1, 1048576, 1048576, 32, 2, 8, 2048),
        # a ragged batch with eight heads a group (the paper's four KV heads)
        _step("step-ragged-g8", 6, 20000, 262143, 32, 4, 8, 2048),
        # long-form reasoning: a large ragged batch, rank 2, a small budget, the token's
        # KV write and the builds of the pages that it fills ("qwen3-4b-reasoning")
        _step("step-reasoning", 64, 8192, 65536, 32, 8, 2, 256, grow=True),
        # summaries of freshly prefilled contexts, at the three page sizes
        _build("build-4x64k", 4, 65536, 65536, 8, 8, 16),
        _build("build-2x128k-page32", 2, 131072, 131072, 8, 8, 32),
        _build("build-2x128k-page64", 2, 131072, 131072, 8, 8, 64),
        # a ragged batch attended in full
        _dense("dense-ragged", 8, 3000, 65535, 32, 8),
        # a 128K context's pages finalised at four bits
        _kivi("kivi-128k", 1, 131072, 131072, 8, 4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges; a step, build or pass over at most 2^20 tokens
    of at most 8 KV heads, contexts of 1K to 1M tokens with ragged ends."""
    op = rng.choice(["step"] * 7 + ["build"] * 3 + ["dense", "kivi"])
    if op == "kivi":
        hi = _log(rng, 2048, 131072)
        return _kivi(None, rng.choice([1, 2, 3]), max(1024, hi // 2), hi, rng.choice([2, 4, 8]),
                     rng.choice([2, 4]))
    if op == "dense":
        hi = _log(rng, 1024, 65536)
        g = rng.choice([1, 4, 7, 8, 16])
        kv = rng.choice([2, 4, 8])
        return _dense(None, _log(rng, 1, 8), max(64, hi // 8), hi, g * kv, kv)
    if op == "build":
        page = rng.choice([16, 16, 32, 64])
        seqs = _log(rng, 1, 6)
        hi = _log(rng, 2048, 262144 // seqs)
        return _build(None, seqs, max(1024, hi // 3), hi, rng.choice([2, 4, 8]),
                      rng.choice([2, 4, 8, 8]), page, rng.choice(["bf16"] * 5 + ["fp32"]))
    kind = rng.choice(["long", "batch", "batch", "grow", "fp32"])
    if kind == "fp32":
        hi = _log(rng, 1024, 32768)
        kv = rng.choice([1, 2])
        return _step(None, rng.choice([1, 2]), max(512, hi // 2), hi, rng.choice([1, 4]) * kv, kv,
                     rng.choice([4, 8]), rng.choice([256, 512]), dtype="fp32")
    if kind == "long":
        hi = _log(rng, 65536, 1048576)
        kv = rng.choice([2, 4])
        return _step(None, 1, hi - rng.randrange(17), hi, rng.choice([4, 8, 16]) * kv, kv,
                     rng.choice([4, 8, 8]), rng.choice([1024, 2048]),
                     page=rng.choice([16, 16, 32, 64]))
    if kind == "grow":
        seqs = _log(rng, 4, 64)
        hi = _log(rng, 2048, 65536)
        return _step(None, seqs, max(1024, hi // 8), hi, 32, 8, rng.choice([2, 4, 8]),
                     rng.choice([256, 512, 1024]), grow=True)
    seqs = _log(rng, 1, 16)
    hi = _log(rng, 4096, 1048576 // seqs)
    kv = rng.choice([4, 8])
    page, basis = rng.choice([(16, "int4")] * 4 + [(32, "int4"), (64, "int4"), (16, "int8")])
    return _step(None, seqs, max(1024, hi // 4), hi, rng.choice([4, 4, 7, 8]) * kv, kv,
                 rng.choice([2, 4, 8, 8]) if basis == "int4" else 8, rng.choice([512, 1024, 2048]),
                 page=page, basis=basis)


# ---------------------------------------------------------------- inputs

def _lens(case):
    """Tokens per sequence: fixed by the case, spread over [lo, hi], odd ones among them."""
    r = random.Random(1000003 * case["hi"] + 7919 * case["lo"] + case["seqs"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["seqs"])]


def _config(case, lens):
    P = case["page"]
    spare = 8 if case["grow"] else 0
    pages = [-(-L // P) + spare for L in lens]
    basis = {"int4": B.LOCKS_BASIS_INT4, "int8": B.LOCKS_BASIS_INT8}[case["basis"]]
    dt = LOCKS_OF[case["dtype"]]
    return B.Config(case["seqs"], case["q_heads"], case["kv_heads"], case["rank"], case["budget"],
                    max(pages), sum(pages), dt, dt, page_size=P, basis=basis), pages


def _encode(V, C, mu, out, basis):
    """Records of [n] pages: V [n][r][128], C [n][P][r], mu [n][128] into out [n][stride]."""
    def scale(x, qmax):
        return (x.abs().amax(-1) / qmax).clamp(max=65504.0).half()

    def codes(x, s, qmax):
        s = s.float().unsqueeze(-1)
        return torch.where(s > 0, (x / s).round().clamp(-qmax, qmax), torch.zeros_like(x)).int()

    n, r, _ = V.shape
    P = C.shape[1]
    if basis == "int4":
        vs = scale(V, 7)
        v = codes(V, vs, 7) + 8
        v = (v[..., 0::2] | (v[..., 1::2] << 4)).to(torch.uint8)
    else:
        vs = scale(V, 127)
        v = (codes(V, vs, 127) + 128).to(torch.uint8)
    cs, ms = scale(C, 127), scale(mu, 127)
    c = (codes(C, cs, 127) + 128).to(torch.uint8)
    m = (codes(mu, ms, 127) + 128).to(torch.uint8)
    sc = torch.cat([vs, cs, ms.unsqueeze(-1)], -1).contiguous().view(torch.uint8)
    rec = torch.cat([v.reshape(n, -1), c.reshape(n, -1), m, sc], -1)
    out[:, :rec.shape[1]] = rec


def prepare(case, seed):
    dev = torch.device("cuda")
    lens = _lens(case)
    cfg, pages = _config(case, lens)
    S, H, P, r = cfg.num_seqs, cfg.num_kv_heads, cfg.page_size, cfg.rank
    dt = TORCH_OF[case["dtype"]]
    op = case["op"]
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 1000003 + 17)

    def randn(*shape):
        return torch.randn(*shape, generator=g, device=dev)

    perm = torch.randperm(cfg.num_blocks, generator=g, device=dev).int()
    table = torch.full((S, cfg.max_pages_per_seq), -1, dtype=torch.int32, device=dev)
    owner = torch.zeros(cfg.num_blocks, dtype=torch.long, device=dev)
    off = 0
    for s in range(S):
        b = perm[off:off + pages[s]]
        table[s, :pages[s]] = b
        owner[b.long()] = s
        off += pages[s]
    # per (sequence, KV head): a mean with outlier channels, shared drift directions
    mean = randn(S, H, D)
    outl = torch.randperm(D, generator=g, device=dev)[:4]
    mean[:, :, outl] = 8.0 * torch.sign(randn(S, H, 4))
    drift = torch.nn.functional.normalize(randn(S, H, SUB, D), dim=-1)
    G = cfg.group
    q = randn(S, H, G, D)
    w = 2.0 * randn(S, H, G, SUB)
    for l in range(SUB):
        q += w[..., l, None] * drift[:, :, None, l]
    q[..., outl] = mean[:, :, None, outl]
    q = q.reshape(S, H * G, D).to(dt)

    keys = torch.empty(cfg.num_blocks, H, P, D, dtype=dt, device=dev)
    summ = B.alloc_summaries(cfg, dev) if op in ("step", "build") else None
    spread = 4.0 * 0.7 ** torch.arange(SUB, device=dev, dtype=torch.float32)
    chunk = max(1, (1 << 17) // (H * (P // 16)))
    for b0 in range(0, cfg.num_blocks, chunk):
        own = owner[b0:b0 + chunk]
        n = own.shape[0]
        mu = mean[own].clone()
        t = 4.0 * randn(n, H, SUB)
        for l in range(SUB):
            mu += t[..., l, None] * drift[own, :, l]
        U = torch.nn.functional.normalize(randn(n, H, SUB, D), dim=-1)
        c = randn(n, H, P, SUB) * spread
        c -= c.mean(2, keepdim=True)
        k = randn(n, H, P, D).mul_(0.05).add_(mu[:, :, None])
        for l in range(SUB):
            k.addcmul_(c[..., l, None], U[:, :, None, l])
        keys[b0:b0 + n] = k.to(dt)
        if op == "step":
            _encode(U[:, :, :r].reshape(n * H, r, D), c[..., :r].reshape(n * H, P, r),
                    mu.reshape(n * H, D), summ[b0:b0 + n].view(n * H, -1), case["basis"])
    vals = None
    if op != "build":
        vals = torch.empty(cfg.num_blocks, H, P, D, dtype=dt, device=dev)
        for b0 in range(0, cfg.num_blocks, chunk):
            vals[b0:b0 + chunk] = randn(min(chunk, cfg.num_blocks - b0), H, P, D).to(dt)
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    st = {"case": case, "cfg": cfg, "lens": lens, "q": q, "k": keys, "v": vals, "pt": table,
          "sl": sl, "summ": summ}
    if op == "step":
        ws = B.alloc_workspace(cfg, dev)
        kn = vn = lst = None
        if case["grow"]:
            kn = (mean + 3.0 * randn(S, H, D) * 0.35).to(dt)
            vn = randn(S, H, D).to(dt)
            full = [[s, L // P - 1] for s, L in enumerate(lens) if L % P == 0]
            lst = torch.tensor(full, dtype=torch.int32, device=dev) if full else None
            B.init()
        st["new"] = (kn, vn, lst)
        st["call"] = B.prepare_decode_step(cfg, q, keys, vals, table, sl, summ, ws, lst,
                                           k_new=kn, v_new=vn)
        st["ws"] = ws
    elif op == "dense":
        ws = B.alloc_workspace(cfg, dev)
        st["call"] = B.prepare_dense_attend(cfg, q, keys, vals, table, sl, ws)
        st["ws"] = ws
    return st


def run(st):
    op, cfg = st["case"]["op"], st["cfg"]
    if op == "step":
        st["call"]()
        ids, sel, out, lse = st["call"].outputs
        r = {"ids": ids, "sel_lse": sel, "out": out, "lse": lse}
        if st["case"]["grow"]:
            r.update(summaries=st["summ"], k_cache=st["k"], v_cache=st["v"])
        return r
    if op == "dense":
        st["call"]()
        out, lse = st["call"].outputs
        return {"out": out, "lse": lse}
    if op == "build":
        B.build_summaries(cfg, st["k"], st["pt"], st["sl"], st["summ"])
        return {"summaries": st["summ"]}
    B.kivi_quantize(cfg, B.Kivi(st["case"]["bits"], 32, B.LOCKS_KIVI_POST), st["k"], st["v"],
                    st["pt"], st["sl"])
    return {"k_cache": st["k"], "v_cache": st["v"]}


# ---------------------------------------------------------------- work and tolerances

def work(case):
    lens = _lens(case)
    P, H, Hq, r = case["page"], case["kv_heads"], case["q_heads"], case["rank"]
    eb = 2 if case["dtype"] == "bf16" else 4
    col = 64 if case["basis"] == "int4" else 128
    rec = col * r + P * r + D + 2 * (r + P + 1)
    complete = sum(L // P for L in lens)
    tokens = sum(lens)
    S = case["seqs"]
    if case["op"] == "build":
        per = P * D + 2 * P * P * D + 9 * P ** 3 + 2 * D * P * r
        return {"bytes": complete * H * (P * D * eb + rec) + 4 * complete, "flops": complete * H * per}
    if case["op"] == "kivi":
        return {"bytes": complete * H * P * D * 2 * 2 * 2 + 4 * complete,
                "flops": complete * H * P * D * 2 * 6}
    outs = S * Hq * (D + 1) * 4
    if case["op"] == "dense":
        return {"bytes": tokens * H * D * 2 * eb + outs + S * Hq * D * eb,
                "flops": 4 * tokens * Hq * D}
    k = -(-case["budget"] // P)
    att = sum(min(k * P, L) for L in lens)
    outs += S * H * k * 4 + S * Hq * k * 4
    b = complete * (H * rec + 4) + att * H * D * 2 * eb + S * Hq * D * eb + outs
    f = complete * Hq * (2 * D * r + 2 * D + 2 * P * r + 2 * P) + 4 * att * Hq * D
    if case["grow"]:
        full = sum(L % P == 0 for L in lens)
        b += S * H * D * eb * 4 + full * H * (P * D * eb + rec)
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["op"] == "build":
        # record bytes that differ from the 64-bit build's: 2e-5 to 8e-5 measured (codes
        # and scales whose value lies within float32 rounding of a tie)
        return {"rel": 0.0, "differ": 5e-4}
    if case["op"] == "kivi":
        return "exact"                   # every operation is one IEEE float32 rounding
    # outputs measured 2e-6 to 6e-6 from the 64-bit ones (scores and normalisers 1e-7)
    if case["op"] == "dense":
        return {"rel": 2.5e-5, "max": 1e-3}
    return {"rel": 2.5e-5, "max": 1e-3, "differ": 0.01}


# ---------------------------------------------------------------- 64-bit results

def _decode(rec, r, P, basis):
    """Records [n][stride] -> V [n][r][128], C [n][P][r], mu [n][128] in 64 bits."""
    n = rec.shape[0]
    col = 64 if basis == "int4" else 128
    v = rec[:, :col * r].reshape(n, r, col)
    if basis == "int4":
        v = torch.stack([v & 15, v >> 4], -1).reshape(n, r, D).double() - 8
    else:
        v = v.double() - 128
    o = col * r
    c = rec[:, o:o + P * r].reshape(n, P, r).double() - 128
    o += P * r
    m = rec[:, o:o + D].double() - 128
    o += D
    sc = rec[:, o:o + 2 * (r + P + 1)].contiguous().view(torch.float16).double()
    return v * sc[:, :r, None], c * sc[:, r:r + P, None], m * sc[:, r + P:]


def _exact_record(keys, r, basis):
    """The record of one page of keys [P][128] from its 64-bit eigendecomposition."""
    K = keys.double().cpu().numpy()
    mu = K.mean(0)
    Dv = K - mu
    lam, U = np.linalg.eigh(Dv @ Dv.T)
    lam, U = np.maximum(lam[::-1][:r], 0.0), U[:, ::-1][:, :r]
    keep = lam > max(1e-6 * lam[0], 1e-10 * np.mean(np.sum(K * K, 1)))
    sig = np.sqrt(np.where(keep, lam, 1.0))
    V = np.where(keep, Dv.T @ U / sig, 0.0)
    flip = np.sign(V[np.argmax(np.abs(V), 0), np.arange(r)])
    flip = np.where(flip == 0, 1.0, flip)
    V, C = V * flip, np.where(keep, U * sig * flip, 0.0)
    P = K.shape[0]
    rec = torch.zeros(1, B.summary_stride(r, B.LOCKS_BASIS_INT4, P), dtype=torch.uint8)
    _encode(torch.from_numpy(V.T.copy()).float()[None], torch.from_numpy(C).float()[None],
            torch.from_numpy(mu).float()[None], rec, basis)
    return rec[0]


def _attend(qh, K, V, mask):
    """qh [H][G][128], K and V [H][T][128], mask [H][T] -> out [H*G][128], lse [H*G]."""
    z = torch.matmul(qh, K.transpose(1, 2).contiguous()) / math.sqrt(D)
    z = z.masked_fill(~mask[:, None], -math.inf)
    lse = torch.logsumexp(z, -1)
    o = torch.matmul(torch.exp(z - lse[..., None]), V)
    return o.reshape(-1, D), lse.reshape(-1)


def exact(case, seed):
    if case["op"] == "build":
        return None                      # records of integer codes
    st = prepare(case, seed)
    cfg, lens, pt = st["cfg"], st["lens"], st["pt"].long()
    S, H, P, G, r, k = (cfg.num_seqs, cfg.num_kv_heads, cfg.page_size, cfg.group, cfg.rank, cfg.k)
    if case["op"] == "kivi":
        levels = 2 ** case["bits"] - 1
        for s, L in enumerate(lens):
            nc = L // P
            for b in pt[s, :nc].split(4096):
                for cache, dim in ((st["k"], 2), (st["v"], 4)):
                    x = cache[b].double()
                    x = x if dim == 2 else x.view(-1, H, P, D // 32, 32)
                    lo, hi = x.amin(dim, keepdim=True), x.amax(dim, keepdim=True)
                    sc = (hi - lo) / levels
                    y = torch.round((x - lo) / torch.where(sc > 0, sc, torch.ones_like(sc)))
                    y = torch.where(sc > 0, y.clamp(max=levels) * sc + lo, x)
                    cache[b] = y.reshape(-1, H, P, D).to(cache.dtype)
        return {"k_cache": st["k"], "v_cache": st["v"]}
    q = st["q"].double().view(S, H, G, D)
    K, V = st["k"], st["v"]
    if case["op"] == "step" and case["grow"]:
        kn, vn, lst = st["new"]
        for s, L in enumerate(lens):
            K[pt[s, (L - 1) // P], :, (L - 1) % P] = kn[s]
            V[pt[s, (L - 1) // P], :, (L - 1) % P] = vn[s]
        for s, j in (lst.tolist() if lst is not None else []):
            for h in range(H):
                rec = _exact_record(K[pt[s, j], h], r, case["basis"])
                st["summ"][pt[s, j], h] = rec.to(K.device)
    outs, lses, sels = [], [], []
    for s, L in enumerate(lens):
        n, nc = -(-L // P), L // P
        if case["op"] == "dense":
            kd = K[pt[s, :n]].transpose(0, 1).reshape(H, n * P, D).double()
            vd = V[pt[s, :n]].transpose(0, 1).reshape(H, n * P, D).double()
            o, l = _attend(q[s], kd, vd, (torch.arange(n * P, device=K.device) < L).expand(H, -1))
            outs.append(o)
            lses.append(l)
            continue
        score = torch.empty(H, G, nc, dtype=torch.float64, device=K.device)
        for h in range(H):
            for b0 in range(0, nc, 16384):
                v, c, m = _decode(st["summ"][pt[s, b0:min(nc, b0 + 16384)], h], r, P, case["basis"])
                qh = q[s, h].t().contiguous()
                p = torch.matmul(v, qh)                                   # [n][r][G]
                z = (torch.matmul(c, p) + torch.matmul(m, qh)[:, None]) / math.sqrt(D)
                score[h, :, b0:b0 + v.shape[0]] = torch.logsumexp(z, 1).t()
        ids = torch.full((H, k), -1, dtype=torch.long, device=K.device)
        if n <= k:
            ids[:, :n] = torch.arange(n, device=K.device)
        else:
            share = torch.exp(score - torch.logsumexp(score, -1, keepdim=True)).mean(1)
            top = torch.sort(share[:, 1:n - 1], dim=-1, descending=True, stable=True)[1][:, :k - 2] + 1
            ids[:, 1:k - 1] = torch.sort(top, -1)[0]
            ids[:, 0] = 0
            ids[:, k - 1] = n - 1
        sel = torch.full((H, G, k), math.nan, dtype=torch.float64, device=K.device)
        ok = (ids >= 0) & (ids < nc)
        got = torch.gather(score, 2, ids.clamp(0, max(nc - 1, 0))[:, None].expand(H, G, k))
        sel = torch.where(ok[:, None], got, sel)
        blocks = pt[s][ids.clamp(min=0)]                                  # [H][k]
        hh = torch.arange(H, device=K.device)[:, None]
        tok = ids[..., None] * P + torch.arange(P, device=K.device)
        mask = ((ids >= 0)[..., None] & (tok < L)).reshape(H, k * P)
        o, l = _attend(q[s], K[blocks, hh].reshape(H, k * P, D).double(),
                       V[blocks, hh].reshape(H, k * P, D).double(), mask)
        outs.append(o)
        lses.append(l)
        sels.append(sel.reshape(H * G, k))
    r_ = {"out": torch.stack(outs), "lse": torch.stack(lses)}
    if case["op"] == "step":
        r_["sel_lse"] = torch.stack(sels)
        if case["grow"]:
            r_.update(summaries=None, k_cache=K, v_cache=V)
    return r_
