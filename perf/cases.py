"""The work that programs using this framework have it do, as timed cases.

A case is one pass through the public calls: re-ranking a candidate list,
scoring (and ranking) a whole corpus, a batch of a serving loop, converting
tokens while an index is built. Documents have ragged lengths (lognormal,
mean 70 tokens, clipped to [8, 180]) unless a case fixes them; their multiset
follows from the case alone and their order from the seed, so that a case's
work does not depend on the seed. Tokens are unit-norm Gaussian vectors.
"""
import math
import random

import torch

import paper_2606_26439_amd as M

DEV = "cuda"
CHUNK = 1 << 21  # tokens made or converted at once
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
PQ_K = 256


def listed():
    return [
        # one query against a first-stage retriever's shortest list: launches and latency
        dict(name="rerank_1q_1k", kind="rerank", dtype="f16", dim=128, pool=100_000, mean_len=70,
             fixed_len=0, n_q=1, nq_lo=32, nq_hi=32, c_lo=1000, c_hi=1000, k=100),
        # the plain FP32 parity workload: 4,096 documents of 32 tokens
        dict(name="plain_f32_4k", kind="score", dtype="f32", dim=128, pool=4096, mean_len=0,
             fixed_len=32, n_q=1, nq_lo=32, nq_hi=32),
        # one batch of the serving loop over exact documents: queries of 8 to 64
        # tokens, 1K to 100K candidates each, top-100
        dict(name="serve_exact_8", kind="rerank", dtype="f16", dim=128, pool=1_000_000,
             mean_len=70, fixed_len=0, n_q=8, nq_lo=8, nq_hi=64, c_lo=1000, c_hi=100_000, k=100),
        # the same batch over the PQ-coded pool
        dict(name="serve_pq_8", kind="pq_rerank", M=8, dsub=16, pool=1_000_000, mean_len=70,
             fixed_len=0, n_q=8, nq_lo=8, nq_hi=64, c_lo=1000, c_hi=100_000, k=100),
        # the same batch over the residual-compressed pool
        dict(name="serve_residual_8", kind="residual_rerank", dim=128, nbits=2, log2_centroids=17,
             pool=1_000_000, mean_len=70, fixed_len=0, n_q=8, nq_lo=8, nq_hi=64, c_lo=1000,
             c_hi=100_000, k=100),
        # exhaustive retrieval over a resident corpus
        dict(name="corpus_f16_1m", kind="search", dtype="f16", dim=128, pool=1_000_000,
             mean_len=70, fixed_len=0, n_q=1, nq_lo=32, nq_hi=32, k=100),
        # the corpus held in FP8 with per-token scales, every score wanted; odd sizes
        dict(name="corpus_fp8_400k", kind="score", dtype="fp8", dim=128, pool=399_989, mean_len=70,
             fixed_len=0, n_q=1, nq_lo=29, nq_hi=29),
        # wide embeddings (the dimension-tiling shape)
        dict(name="wide_bf16_768", kind="score", dtype="bf16", dim=768, pool=50_000, mean_len=0,
             fixed_len=128, n_q=1, nq_lo=32, nq_hi=32),
        # a query set evaluated against a collection in one call
        dict(name="eval_f16_16q", kind="search", dtype="f16", dim=128, pool=100_003, mean_len=70,
             fixed_len=0, n_q=16, nq_lo=32, nq_hi=32, k=100),
        # many queries against a PQ-coded collection in one call
        dict(name="pq_64q_250k", kind="pq_score", M=8, dsub=16, pool=250_000, mean_len=70,
             fixed_len=0, n_q=64, nq_lo=32, nq_hi=32),
        # one query over a residual-compressed corpus
        dict(name="residual_1m", kind="residual_score", dim=128, nbits=2, log2_centroids=17,
             pool=1_000_000, mean_len=70, fixed_len=0, n_q=1, nq_lo=32, nq_hi=32),
        # a block of an index being built: FP32 encoder output to FP8 tokens and scales
        dict(name="index_fp8_1m", kind="convert", dtype="fp8", dim=128, tokens=1_000_000),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rerank", "rerank", "search", "score", "pq_rerank", "pq_score",
                       "residual_rerank", "residual_score", "convert"])
    if kind == "convert":
        dim = rng.choice([64, 96, 128, 256, 768])
        return dict(kind=kind, dtype=rng.choice(["f16", "bf16", "fp8"]), dim=dim,
                    tokens=_logint(rng, 1000, 128_000_000 // dim))
    c = dict(kind=kind)
    row = 8  # bytes of a token, to bound the pool
    if kind in ("rerank", "search", "score"):
        c["dtype"] = rng.choice(["f16", "f16", "bf16", "fp8", "f32"])
        c["dim"] = rng.choice([64, 96, 128, 128, 128, 256, 400, 768])
        if c["dtype"] == "f32" and c["dim"] > 400:  # 64 query tokens of FP32 have to fit the LDS
            c["dim"] = 128
        row = c["dim"] * {"f32": 4, "fp8": 1}.get(c["dtype"], 2)
    elif kind.startswith("pq"):
        c["M"], c["dsub"] = rng.choice([(8, 16), (16, 8)])
    else:
        c["dim"], c["nbits"] = rng.choice([64, 128, 128]), rng.choice([1, 2, 2, 4])
        c["log2_centroids"] = rng.randint(12, 17)
    c["pool"] = _logint(rng, 1000, min(1_000_000, 12_000_000_000 // (70 * row)))
    c["mean_len"], c["fixed_len"] = 70, 0
    if rng.random() < 0.25:
        c["mean_len"], c["fixed_len"] = 0, _logint(rng, 17, 128)
    if kind.endswith("rerank"):
        c["n_q"] = _logint(rng, 1, 12)
        c["nq_lo"], c["nq_hi"] = (8, 64) if rng.random() < 0.5 else (32, 32)
        c["c_hi"] = _logint(rng, 500, max(500, min(100_000, c["pool"], 25_000_000 // row)))
        c["c_lo"] = min(1000, c["c_hi"])
    else:
        top = {"search": 16, "score": 4, "pq_score": 64, "residual_score": 2}[kind]
        top = max(1, min(top, 16_000_000 // c["pool"], 16_000_000 * 128 // (c["pool"] * row)))
        c["n_q"] = _logint(rng, 1, top)
        n = rng.choice([32, 32, rng.randint(5, 64)])
        c["nq_lo"], c["nq_hi"] = n, n
    if kind == "search" or kind.endswith("rerank"):
        c["k"] = rng.choice([10, 100, 100, 1000])
    return c


# ------------------------------------------------------------------ inputs --

def _gen(seed, part):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 16 + part)


def _lengths(case):
    """The documents' lengths in ascending order: lognormal quantiles, or all the same."""
    n = case["pool"]
    if case["fixed_len"]:
        return torch.full((n,), case["fixed_len"], dtype=torch.int64)
    sigma = 0.5
    z = math.sqrt(2) * torch.erfinv(2 * (torch.arange(n, dtype=torch.float64) + 0.5) / n - 1)
    x = torch.exp(math.log(case["mean_len"]) - sigma * sigma / 2 + sigma * z)
    return x.round().clamp(8, 180).to(torch.int64)


def _spread(lo, hi, n, order):
    """n values spread evenly over [lo, hi], in the fixed order that `order` names (so that
    long queries and long candidate lists do not go together)."""
    v = [lo + (hi - lo) * (2 * i + 1) // (2 * n) for i in range(n)]
    random.Random(order).shuffle(v)
    return v


def _offsets(lens):
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64)
    torch.cumsum(lens, 0, out=off[1:])
    return off.to(DEV)


def _doc_offsets(case, seed):
    order = torch.randperm(case["pool"], generator=torch.Generator().manual_seed(int(seed)))
    return _offsets(_lengths(case)[order])


def _unit(n, dim, gen):
    x = torch.randn((n, dim), generator=gen, device=DEV)
    return x.div_(x.norm(dim=1, keepdim=True))


def _to_fp8(x):
    """E4M3 codes and the smallest power-of-two scale of each token that fits them."""
    k = torch.ceil(torch.log2(x.abs().amax(dim=1).double() / 448)).clamp_min(-126)
    s = torch.exp2(k)
    return (x / s[:, None].float()).to(torch.float8_e4m3fn).view(torch.uint8), s.float()


def _as(x, dtype):
    return _to_fp8(x) if dtype == "fp8" else (x.to(TORCH[dtype]), None)


def _tokens(n, dim, dtype, gen):
    """n unit-norm tokens in `dtype` and their scales (FP8)."""
    tok = torch.empty((n, dim), dtype=TORCH.get(dtype, torch.uint8), device=DEV)
    scl = torch.empty(n, dtype=torch.float32, device=DEV) if dtype == "fp8" else None
    for s in range(0, n, CHUNK):
        t, c = _as(_unit(min(CHUNK, n - s), dim, gen), dtype)
        tok[s:s + t.shape[0]] = t
        if scl is not None:
            scl[s:s + t.shape[0]] = c
    return tok, scl


def _queries(case, dim, seed):
    """FP32 query tokens, their offsets and the longest query."""
    lens = _spread(case["nq_lo"], case["nq_hi"], case["n_q"], "tokens")
    return (_unit(sum(lens), dim, _gen(seed, 1)), _offsets(torch.tensor(lens)), max(lens))


def _candidates(case, seed):
    """Candidate ids of each query, drawn without replacement."""
    sizes = _spread(case["c_lo"], case["c_hi"], case["n_q"], "candidates")
    g = _gen(seed, 2)
    ids = [torch.randperm(case["pool"], generator=g, device=DEV)[:n].to(torch.int32) for n in sizes]
    return _offsets(torch.tensor(sizes)), torch.cat(ids)


def _dim(case):
    return case["M"] * case["dsub"] if "M" in case else case["dim"]


def _docs(case, seed):
    """The document arrays of the case's form, by name."""
    d, g = {"off": _doc_offsets(case, seed)}, _gen(seed, 3)
    n, dim = int(_lengths(case).sum()), _dim(case)
    if "M" in case:
        d["codebooks"] = (0.25 * torch.randn((case["M"], PQ_K, case["dsub"]), generator=g,
                                             device=DEV)).half()
        d["codes"] = torch.randint(0, PQ_K, (n, case["M"]), generator=g, device=DEV,
                                   dtype=torch.uint8)
    elif "nbits" in case:
        n_c, levels = 1 << case["log2_centroids"], 1 << case["nbits"]
        d["centroids"] = _unit(n_c, dim, g).half()
        p = (torch.arange(levels, dtype=torch.float64) + 0.5) / levels
        d["weights"] = (0.02 * math.sqrt(2) * torch.erfinv(2 * p - 1)).half().to(DEV)
        d["ids"] = torch.randint(0, n_c, (n,), generator=g, device=DEV, dtype=torch.int32)
        d["residuals"] = torch.randint(0, 256, (n, dim * case["nbits"] // 8), generator=g,
                                       device=DEV, dtype=torch.uint8)
    else:
        d["tokens"], d["scales"] = _tokens(n, dim, case["dtype"], g)
    return d


def prepare(case, seed):
    kind = case["kind"]
    if kind == "convert":
        return dict(kind=kind, dtype=case["dtype"], x=_unit(case["tokens"], case["dim"],
                                                            _gen(seed, 0)))
    q32, q_off, q_max = _queries(case, _dim(case), seed)
    a = _docs(case, seed)
    dtype = case.get("dtype", "f16")
    s = dict(kind=kind, dtype=dtype, q32=q32, q_off=q_off, q_max=q_max, k=case.get("k"))
    if "M" in case:
        s["docs"] = M.PQDocs(a["codebooks"], a["codes"], a["off"])
    elif "nbits" in case:
        s["docs"] = M.ResidualDocs(a["centroids"], a["weights"], a["ids"], a["residuals"],
                                   a["off"], case["nbits"])
    else:
        s["docs"] = M.Tokens(a["tokens"], a["off"], dtype, a["scales"],
                             max_len=int(_lengths(case)[-1]))
    if kind.endswith("rerank"):
        c_off, c_ids = _candidates(case, seed)
        s["cand"] = M.Candidates(c_off, c_ids)
    return s


def run(s):
    if s["kind"] == "convert":
        return M.quantize(s["x"], s["dtype"])
    # a request's query arrives in FP32 and is converted on the device
    qt, qs = M.quantize(s["q32"], s["dtype"])
    q = M.Tokens(qt, s["q_off"], s["dtype"], qs, max_len=s["q_max"])
    docs, kind = s["docs"], s["kind"]
    if kind in ("rerank", "search"):
        return M.score_topk(q, docs, s["k"], s.get("cand"))
    if kind == "score":
        return M.score(q, docs)
    if kind == "pq_score":
        return M.pq_score(q, docs)
    if kind == "residual_score":
        return M.residual_score(q, docs)
    cand = s["cand"]
    score = M.pq_score if kind == "pq_rerank" else M.residual_score
    scores = score(q, docs, cand)
    return (scores,) + tuple(M.topk(scores, cand.offsets, s["k"], ids=cand.doc_ids))


def work(case):
    """Each input read once, each output written once; two operations per
    multiply-add of every query token with every token it is scored against."""
    kind = case["kind"]
    if kind == "convert":
        n, d = case["tokens"], case["dim"]
        return dict(bytes=n * (4 * d + (d + 4 if case["dtype"] == "fp8" else 2 * d)),
                    flops=n * d)
    dim, pool = _dim(case), case["pool"]
    tokens = int(_lengths(case).sum())
    nq = _spread(case["nq_lo"], case["nq_hi"], case["n_q"], "tokens")
    fixed = sum(nq) * dim * 4
    if "M" in case:
        row = case["M"]
        fixed += case["M"] * PQ_K * case["dsub"] * 2
    elif "nbits" in case:
        row = 4 + dim * case["nbits"] // 8
        fixed += (1 << case["log2_centroids"]) * dim * 2
    else:
        row = dim * {"f32": 4, "fp8": 1}.get(case["dtype"], 2) + (4 if case["dtype"] == "fp8" else 0)
    per_doc = tokens / pool
    if kind.endswith("rerank"):
        sizes = _spread(case["c_lo"], case["c_hi"], case["n_q"], "candidates")
        miss = 1.0
        for c in sizes:
            miss *= 1 - c / pool
        read = pool * (1 - miss) * (per_doc * row + 8) + 4 * sum(sizes)
        pairs, flops = sum(sizes), sum(2 * n * c for n, c in zip(nq, sizes)) * per_doc * dim
    else:
        read, pairs, flops = tokens * row + 8 * pool, case["n_q"] * pool, 2 * sum(nq) * tokens * dim
    out = 8 * case["n_q"] * case["k"] if case.get("k") else 0
    if kind not in ("rerank", "search"):
        out += 4 * pairs
    return dict(bytes=read + fixed + out, flops=flops)


# --------------------------------------------------- the same in 64 bits --

def _decoder(case, a):
    """idx -> the FP64 vectors of those document tokens."""
    if "M" in case:
        cb, m = a["codebooks"].double(), torch.arange(case["M"], device=DEV)
        return lambda idx: cb[m, a["codes"][idx].long()].reshape(idx.numel(), -1)
    if "nbits" in case:
        cen, w, nb = a["centroids"].double(), a["weights"].double(), case["nbits"]
        shift = torch.arange(0, 8, nb, device=DEV)

        def decode(idx):
            f = (a["residuals"][idx].long()[:, :, None] >> shift) & ((1 << nb) - 1)
            return cen[a["ids"][idx].long()] + w[f.reshape(idx.numel(), -1)]
        return decode
    if a["scales"] is None:
        return lambda idx: a["tokens"][idx].double()
    return lambda idx: (a["tokens"][idx].view(torch.float8_e4m3fn).double()
                        * a["scales"][idx].double()[:, None])


def _maxsim64(queries, docs, off, decode, dim):
    """Scores of every query in `queries` (FP64 token matrices) against `docs`."""
    out = torch.empty((len(queries), docs.numel()), dtype=torch.float64, device=DEV)
    cols = sum(q.shape[0] for q in queries)
    qt = torch.cat(queries).t().contiguous()
    lens = off[1:] - off[:-1]
    longest = int(lens.max())
    step = max(1, (1 << 31) // (8 * longest * max(cols, 2 * dim)))
    for s in range(0, docs.numel(), step):
        d = docs[s:s + step]
        n = lens[d]
        width = int(n.max())
        pos = torch.minimum(torch.arange(width, device=DEV)[None, :], n[:, None] - 1)
        idx = (off[d][:, None] + pos).reshape(-1)
        best = torch.mm(decode(idx), qt).view(d.numel(), width, cols).amax(dim=1)
        at = 0
        for i, q in enumerate(queries):
            out[i, s:s + d.numel()] = best[:, at:at + q.shape[0]].sum(dim=1)
            at += q.shape[0]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "convert":
        x = _unit(case["tokens"], case["dim"], _gen(seed, 0))
        if case["dtype"] == "fp8":
            return None, _to_fp8(x)[1].double()
        return x.double(), None
    dim = _dim(case)
    q32, q_off, _ = _queries(case, dim, seed)
    a = _docs(case, seed)
    tok, scl = _as(q32, case.get("dtype", "f16"))
    q64 = tok.double() if scl is None else (tok.view(torch.float8_e4m3fn).double()
                                            * scl.double()[:, None])
    o = q_off.tolist()
    queries = [q64[o[i]:o[i + 1]] for i in range(case["n_q"])]
    decode = _decoder(case, a)
    if kind.endswith("rerank"):
        c_off, c_ids = _candidates(case, seed)
        c = c_off.tolist()
        per = [_maxsim64([q], c_ids[c[i]:c[i + 1]].long(), a["off"], decode, dim)[0]
               for i, q in enumerate(queries)]
    else:
        ids = torch.arange(case["pool"], device=DEV)
        per = list(_maxsim64(queries, ids, a["off"], decode, dim))
    if not case.get("k"):
        return torch.cat(per)
    top = torch.full((len(per), case["k"]), -math.inf, dtype=torch.float64, device=DEV)
    for i, p in enumerate(per):
        n = min(case["k"], p.numel())
        top[i, :n] = torch.topk(p, n).values
    return (top, None) if kind in ("rerank", "search") else (torch.cat(per), top, None)
