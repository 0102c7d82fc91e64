"""Timed cases of the scoring library: the calls that a retrieval program makes, over the sizes it
makes them at.

A case is a dict of plain values:
  op        full      exhaustive scoring of every document and its top-K
            topk      Col-Bandit top-K, elimination rounds on the stored embeddings
            topk_i8   Col-Bandit top-K, elimination rounds on int8 codes of the corpus
            quantize  int8 coding of a corpus (done once for an index)
  corpus    text (iid tokens with planted relevant documents), topics (topic mixture), pages
            (documents of one length, T queries from a few centroids): see synth.py
  dtype, N, Lmin, Lmax, nq, T, d    storage type and sizes
  K, alpha, B, M                    top-K and the knobs of the estimator (delta is 0.01)
The largest cases are the benchmark's workload (500,000 documents of 32 to 180 tokens, 128 queries
of 32 tokens, width 128, bf16); the others are the repository's remaining configurations, a single
query, and small, odd shapes of the same kind.
"""
import math

import numpy as np
import torch

from paper_2602_02827_amd import binding, synth

DELTA = 0.01


def _case(name, op, corpus, dtype, N, L, nq, T, d=128, K=5, alpha=0.2, B=4, M=5):
    c = dict(op=op, corpus=corpus, dtype=dtype, N=N, Lmin=L[0], Lmax=L[1], nq=nq, T=T, d=d, K=K,
             alpha=alpha, B=B, M=M)
    if name:
        c["name"] = name
    return c


def listed():
    text = (32, 180)
    return [
        # one query reranks a candidate list of 1,000 short passages in fp32: both scoring paths at
        # the smallest size, where a call is launches and latency
        _case("full_1k_1q_f32", "full", "text", "f32", 1000, (32, 64), 1, 32),
        _case("topk_1k_1q_f32", "topk", "text", "f32", 1000, (32, 64), 1, 32),
        # a few odd-length queries of a half-width (Matryoshka) encoder rerank a ragged candidate list
        _case("topk_6k_7q_d64_odd", "topk", "topics", "bf16", 6007, (1, 301), 7, 21, d=64, K=10),
        # fp32 embeddings kept by a program that does not want bf16: a batch over a mid-size corpus
        _case("full_20k_16q_f32", "full", "topics", "f32", 20000, text, 16, 32),
        # the mid-size text configuration: Col-Bandit over 50,000 passages, 64 queries
        _case("topk_50k_64q", "topk", "text", "bf16", 50000, text, 64, 32),
        # page images of 1,030 patch tokens, short vision queries (T = 24): both paths
        _case("full_pages_64q", "full", "pages", "bf16", 20000, (1030, 1030), 64, 24),
        _case("topk_pages_64q", "topk", "pages", "bf16", 20000, (1030, 1030), 64, 24),
        # one user query against the whole large corpus: latency of a corpus pass
        _case("full_500k_1q", "full", "topics", "bf16", 500000, text, 1, 32),
        # the benchmark's workload: exhaustive, Col-Bandit, Col-Bandit with int8 rounds
        _case("full_500k_128q", "full", "topics", "bf16", 500000, text, 128, 32),
        _case("topk_500k_128q", "topk", "topics", "bf16", 500000, text, 128, 32),
        _case("topk_i8_500k_128q", "topk_i8", "topics", "bf16", 500000, text, 128, 32),
        # coding that corpus when the index is built
        _case("quantize_53m_tokens", "quantize", "topics", "bf16", 500000, text, 1, 32),
    ]


# limits of a drawn case: those of the largest listed one, and for fp32 (which no tuned case of
# this size stands for) documents read once per query from HBM or cache in about a quarter second
MAX_TOKENS = 53e6
MAX_FLOPS = 5.6e13
MAX_F32_BYTES = 2e11
MAX_PAIRS = 6.4e7


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    op = rng.choice(["full", "full", "full", "topk", "topk", "topk", "topk_i8", "topk_i8", "quantize"])
    corpus = rng.choice(["text", "topics", "topics", "pages"])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    d = rng.choice([128, 128, 128, 64, 64, 96, 32]) if op in ("full", "topk") else rng.choice([128, 128, 64])
    T = rng.choice([32, 32, 24, rng.randint(5, 48), rng.randint(5, 64),
                    rng.randint(33, 64 if dtype == "f32" else 128)])
    N = log(500, 30000) if corpus == "pages" else log(500, 500000)
    nq = log(1, 256)
    if corpus == "pages":
        Lmin = Lmax = rng.choice([729, 1030, rng.randint(200, 1500)])
    else:
        Lmin, Lmax = rng.choice([(32, 180), (32, 64), (1, 2 * rng.randint(20, 150) + 1)])
    mean = (Lmin + Lmax) / 2.0
    N = int(min(N, MAX_TOKENS / mean))
    if corpus == "text":                     # 20 planted documents for each query
        nq = min(nq, 64, N // 25)
    flops_q = 2.0 * T * d * N * mean
    nq = int(max(1, min(nq, MAX_FLOPS / flops_q, MAX_PAIRS / N)))
    if dtype == "f32" and op != "quantize":
        nq = int(max(1, min(nq, MAX_F32_BYTES / (4.0 * d * N * mean))))
    return _case(None, op, corpus, dtype, N, (Lmin, Lmax), nq, T, d=d, K=rng.choice([1, 5, 10, 10, 50, 100]),
                 alpha=rng.choice([0.05, 0.1, 0.2, 0.2, 0.3, 0.5, 1.0]), B=rng.choice([4, 4, 4, 2, 3, 8]),
                 M=rng.choice([0, 5, 5, 10]))


def _workload(case, seed, device="cuda"):
    c = case
    if c["op"] == "quantize":                # documents do not matter to the codes, only the rows do
        c = dict(c, Lmin=(c["Lmin"] + c["Lmax"]) // 2, Lmax=(c["Lmin"] + c["Lmax"]) // 2)
    a = ("case", c["N"])
    if c["corpus"] == "text":
        n = 5 if c["N"] <= 2000 else 20
        return synth.text_iid(*a, c["Lmin"], c["Lmax"], c["nq"], c["T"], c["d"], c["dtype"], n,
                              (0.3,) if n == 5 else (0.2, 0.4, 0.6), seed, device)
    if c["corpus"] == "pages":
        return synth.pages(*a, c["Lmin"], c["nq"], c["T"], c["d"], c["dtype"], 256, seed, device)
    return synth.text_topics(*a, c["Lmin"], c["Lmax"], c["nq"], c["T"], c["d"], c["dtype"],
                             1024 if c["N"] > 200000 else 512, seed, device)


def prepare(case, seed):
    """The corpus, the queries, the workspace and the output arrays that a serving loop keeps."""
    w = _workload(case, seed)
    st = {"case": case, "docs": w.docs, "offsets": w.offsets, "Q": w.Q, "seed": seed}
    if case["op"] == "quantize":
        return st
    nq, K = case["nq"], case["K"]
    dev = w.docs.device
    st["ws"] = binding.new_workspace(nq, case["T"], case["d"], case["N"], w.total_tokens, dev)
    st["out"] = {"topk_ids": torch.empty((nq, K), dtype=torch.int64, device=dev),
                 "topk_scores": torch.empty((nq, K), dtype=torch.float32, device=dev)}
    if case["op"] == "full":
        st["out"]["scores"] = torch.empty((nq, case["N"]), dtype=torch.float32, device=dev)
    if case["op"] == "topk_i8":
        st["codes"], st["scale"] = binding.colbandit_quantize_i8(w.docs)
    return st


def run(state):
    s, c = state, state["case"]
    if c["op"] == "quantize":
        codes, scales = binding.colbandit_quantize_i8(s["docs"])
        return {"codes": codes, "scales": scales}
    if c["op"] == "full":
        r = binding.colbandit_full_maxsim(s["Q"], s["docs"], s["offsets"], K=c["K"], workspace=s["ws"],
                                          out=s["out"])
        return {"ids": r["topk_ids"], "scores": r["scores"], "topk_scores": r["topk_scores"]}
    more = {"docs_i8": s["codes"], "docs_scale": s["scale"]} if c["op"] == "topk_i8" else {}
    r = binding.colbandit_topk(s["Q"], s["docs"], s["offsets"], c["K"], c["alpha"], DELTA, c["M"],
                               s["seed"], B=c["B"], workspace=s["ws"], out=s["out"], want_stats=False,
                               **more)
    return {"ids": r["topk_ids"], "topk_scores": r["topk_scores"]}


def work(case):
    """full: every token against every query row, the corpus read once.  topk: the first reveal
    batch of every (query, document) pair, which no elimination can avoid, and the corpus (or its
    codes) read once.  quantize: the corpus read once, the codes written once."""
    c = case
    tokens = c["N"] * (c["Lmin"] + c["Lmax"]) / 2.0 if c["op"] != "quantize" else \
        float(c["N"] * ((c["Lmin"] + c["Lmax"]) // 2))
    elem = 4 if c["dtype"] == "f32" else 2
    if c["op"] == "quantize":
        return {"bytes": tokens * c["d"] * (elem + 1), "flops": 0.0}
    queries = c["nq"] * c["T"] * c["d"] * elem + 8.0 * c["N"]
    results = 12.0 * c["nq"] * c["K"]
    if c["op"] == "full":
        return {"bytes": tokens * c["d"] * elem + queries + results + 4.0 * c["nq"] * c["N"],
                "flops": 2.0 * c["nq"] * c["T"] * c["d"] * tokens}
    rows = tokens * c["d"] * (1 if c["op"] == "topk_i8" else elem)
    return {"bytes": rows + queries + results,
            "flops": 2.0 * c["nq"] * min(c["B"], c["T"]) * c["d"] * tokens}


def tolerance(case):
    """Cells are products of the stored values summed in 32 bits: about 1e-7 from the 64-bit
    scores (measured 3e-8 to 6e-8 on every path), so documents change places only where their
    scores tie.  Col-Bandit decides on 32-bit bounds: a document whose bound lies within rounding
    of the threshold may be kept by one implementation and dropped by another, which exchanges
    one returned document of a query for a neighbour of nearly the same score."""
    if case["op"] == "quantize":
        return "exact"
    if case["op"] == "full":
        return {"rel": 5e-7, "max": 5e-6, "differ": 0.01}
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.01}


# ------------------------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ------------------------------------------------------------------------------------------
_MASK = 2**64 - 1


def _order(seed, q, T):
    """Reveal order of query q: a Fisher-Yates shuffle on a SplitMix64 stream."""
    s = (seed + (q + 1) * 0x9E3779B97F4A7C15) & _MASK
    pi = list(range(T))
    for i in range(T - 1, 0, -1):
        s = (s + 0x9E3779B97F4A7C15) & _MASK
        z = s
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _MASK
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _MASK
        z ^= z >> 31
        j = z % (i + 1)
        pi[i], pi[j] = pi[j], pi[i]
    return pi


def _cells(Q, docs, offsets, want_cells):
    """Largest dot product of each document with each query row, in 64 bits: cells
    [documents, query rows], or the scores [documents, queries] alone."""
    nq, T, d = Q.shape
    N = offsets.numel() - 1
    rows = Q.reshape(nq * T, d).double().t().contiguous()
    lens = offsets[1:] - offsets[:-1]
    out = torch.empty((N, nq * T) if want_cells else (N, nq), dtype=torch.float64, device=docs.device)
    longest = int(lens.max())
    step = max(1, int(5e8 / (longest * nq * T)))
    at = torch.arange(longest, device=docs.device)
    for lo in range(0, N, step):
        hi = min(N, lo + step)
        width = int(lens[lo:hi].max())
        # short documents repeat their last token, which changes no maximum
        idx = torch.minimum(offsets[lo:hi, None] + at[None, :width], offsets[lo + 1:hi + 1, None] - 1)
        h = (docs[idx.reshape(-1)].double() @ rows).view(hi - lo, width, nq * T).amax(1)
        out[lo:hi] = h if want_cells else h.view(hi - lo, nq, T).sum(2)
    return out


def _top(scores, ids, K):
    """(score descending, id ascending); ids ascending on entry."""
    o = torch.argsort(scores, descending=True, stable=True)[:K]
    return scores[o], ids[o]


def _clip(x, permille=999):
    """Nearest-rank percentile of |x|."""
    a = x.abs().float().reshape(-1)
    drop = a.numel() - (a.numel() * permille + 999) // 1000      # values above the wanted one
    if drop > 1000000:                                           # a long corpus: in parts
        parts = [p.topk(min(p.numel(), drop + 1)).values for p in a.split(1 << 28)]
        a = torch.cat(parts)
    return a.sort(descending=True).values[drop]


def _col_bandit(H, T, case, seed, q):
    """Algorithm 1 on one query's cells H [N, T]: ids of the survivors, ascending."""
    N = H.shape[0]
    K, M, B = case["K"], case["M"], case["B"]
    alpha, delta = float(np.float32(case["alpha"])), float(np.float32(DELTA))
    pi = _order(seed, q, T)
    live = torch.arange(N, device=H.device)
    seen = 0
    while live.numel() > K + M and seen < T:
        n = min(T, seen + B)
        cells = H[live][:, torch.as_tensor(pi[:n], device=H.device)]
        total = cells.sum(1)
        low, high = total - (T - n), total + (T - n)
        if n >= T:
            low = high = total
        elif n > 1:
            rho = 1 - (n - 1) / T if 2 * n <= T else (1 - n / T) * (1 + 1 / n)
            radius = alpha * T * math.sqrt(2 * math.log(N * T / delta) / n) * math.sqrt(rho) * cells.std(1)
            low, high = torch.maximum(low, T * total / n - radius), torch.minimum(high, T * total / n + radius)
        tau = low.topk(K).values[-1]
        live = live[high >= tau]
        seen = n
    return live


def exact(case, seed):
    c = case
    w = _workload(c, seed)
    T, K, nq, N = c["T"], c["K"], c["nq"], c["N"]
    if c["op"] == "quantize":
        if w.docs.numel() > 2e9:
            return None
        return {"codes": None, "scales": (_clip(w.docs).double() / 127).reshape(1)}
    if c["op"] == "full":
        S = _cells(w.Q, w.docs, w.offsets, False).t().contiguous()
        ids = torch.arange(N, device=S.device)
        return {"ids": None, "scores": S, "topk_scores": torch.stack([_top(S[q], ids, K)[0] for q in range(nq)])}
    if 8.0 * nq * N * T > 40e9:
        return None
    if c["op"] == "topk_i8":
        # codes in single precision, as they are defined; their products in 64 bits
        codes, scale = binding.colbandit_quantize_i8(w.docs)
        clips = torch.stack([_clip(w.Q[q]) for q in range(nq)])
        Q8 = torch.clamp(torch.round(w.Q.float() * (127.0 / clips).view(nq, 1, 1)), -127, 127)
        H = _cells(Q8, codes, w.offsets, True).view(N, nq, T)
        H *= (clips.double() / 127 * scale.double()).view(1, nq, 1)
    else:
        H = _cells(w.Q, w.docs, w.offsets, True).view(N, nq, T)
    out = torch.full((nq, K), -math.inf, dtype=torch.float64, device=H.device)
    lens = w.offsets[1:] - w.offsets[:-1]
    for q in range(nq):
        live = _col_bandit(H[:, q], T, c, seed, q)
        if c["op"] == "topk_i8":             # the survivors' scores are those of the stored embeddings
            keep = lens[live]
            off = torch.zeros(live.numel() + 1, dtype=torch.int64, device=H.device)
            off[1:] = torch.cumsum(keep, 0)
            rows = torch.repeat_interleave(w.offsets[live] - off[:-1], keep) + torch.arange(int(off[-1]), device=H.device)
            S = _cells(w.Q[q:q + 1], w.docs[rows], off, False)[:, 0]
        else:
            S = H[live, q].sum(1)
        top = _top(S, live, K)[0]
        out[q, :top.numel()] = top
    return {"ids": None, "topk_scores": out}
