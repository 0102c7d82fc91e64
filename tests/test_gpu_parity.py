"""GPU <-> oracle parity through the C-ABI (run with -m gpu on an MI355X).

Tolerances (relative, on scores): 1e-5 for fp32 inputs, 2e-3 for bf16 inputs with fp32
accumulation; the oracle reads the same storage-rounded values.  Index results are exact
wherever the deciding gap exceeds the tolerance.  The Col-Bandit rounds are compared by
feeding the oracle the GPU's own MaxSim cells, so that only the bookkeeping differs; a
document may then differ only if its UCB lies within EPS_BAND of the round's threshold.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-3}
EPS_BAND = 2e-4          # fp32 bound arithmetic vs the oracle's double, on values of size <= T


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2602_02827_amd import binding
    binding.lib()          # raises if the HIP library is not built: no fallback
    return binding


@pytest.fixture(scope="module")
def S():
    from paper_2602_02827_amd import synth
    return synth


def _custom(S, lengths, nq, T, d, dtype, seed):
    """Corpus with prescribed document lengths (iid unit tokens), on the GPU."""
    g = torch.Generator(device="cpu"); g.manual_seed(seed)
    L = torch.tensor(lengths, dtype=torch.int64)
    off = torch.zeros(len(lengths) + 1, dtype=torch.int64); off[1:] = torch.cumsum(L, 0)
    E = torch.randn((int(off[-1]), d), generator=g)
    E = E / E.norm(dim=1, keepdim=True)
    Q = torch.randn((nq, T, d), generator=g)
    Q = Q / Q.norm(dim=2, keepdim=True)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    return S.Workload(f"custom-{dtype}", dtype, Q.to(td).cuda(), E.to(td).cuda(), off.cuda(), seed=seed)


def _oracle_scores(oracle_mod, w, qs=None):
    E, off = w.host_docs()
    Qh = w.host_queries()
    qs = range(w.nq) if qs is None else qs
    H = np.stack([oracle_mod.maxsim_cells(Qh[q], E, off) for q in qs])
    return H, H.sum(axis=2)


def _kernels(fn, into=None):
    """The names of the kernels that fn launches, one for each launch; its result is appended to `into`.  A profile now and
    then comes back without any kernel record (API records only): then fn runs again."""
    from torch.profiler import ProfilerActivity, profile
    for _ in range(5):
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            result = fn()
            torch.cuda.synchronize()
        names = " ".join(e.key for e in p.events())
        if "cb::" in names:
            break
    if into is not None:
        into.append(result)
    return names


def _past_small(lengths, nq, d, dtype):
    """The lengths repeated until nq queries over them are no longer a call small enough to gather
    (40 MB of reading)."""
    row = d * (2 if dtype == "bf16" else 4)
    return list(lengths) * (int(4.2e7 / (nq * row * sum(lengths))) + 1)


def _check_topk(ids, scores, S_or, K, tol):
    """ids/scores: GPU top-K of one query; S_or: oracle scores of all docs."""
    order = np.lexsort((np.arange(len(S_or)), -S_or))
    kth = S_or[order[K - 1]]
    band = tol * max(1.0, abs(kth))
    assert len(set(ids.tolist())) == K
    assert np.all(np.diff(scores) <= 0)                       # returned in score order
    assert np.all(S_or[ids] >= kth - band)                    # nothing clearly below the cut
    must = order[:K][S_or[order[:K]] > kth + band]            # clearly above the cut
    assert set(must.tolist()) <= set(ids.tolist())
    np.testing.assert_allclose(scores, S_or[ids], rtol=tol, atol=tol)
    gaps = -np.diff(S_or[order[:K + 1]]) if len(S_or) > K else -np.diff(S_or[order[:K]])
    if np.all(gaps > 2 * band):                                # no near-ties: exact order
        np.testing.assert_array_equal(ids, order[:K])


# ------------------------------------------------------------------ Full-MaxSim
def test_full_maxsim_fp32_config1(B, S, oracle_mod):
    w = S.config(0, device="cuda")                              # N=1000, fp32, 1 query
    H, Sor = _oracle_scores(oracle_mod, w)
    r = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=5, want_cells=True)
    torch.cuda.synchronize()
    np.testing.assert_allclose(r["cells"].cpu().numpy(), H, rtol=1e-5, atol=1e-6)
    np.testing.assert_allclose(r["scores"].cpu().numpy(), Sor, rtol=1e-5, atol=1e-6)
    _check_topk(r["topk_ids"][0].cpu().numpy(), r["topk_scores"][0].cpu().numpy(), Sor[0], 5, 1e-5)
    assert set(w.planted[0]) == set(r["topk_ids"][0].tolist())  # the planted docs are the top-5


@pytest.mark.parametrize("nq,T,d", [(1, 32, 128), (3, 32, 128), (6, 24, 128), (20, 32, 128),
                                     (5, 7, 128), (3, 40, 128), (2, 100, 128), (4, 32, 64),
                                     (40, 16, 64), (4, 32, 96), (3, 24, 32), (2, 100, 96)])
def test_full_maxsim_bf16_dense_ragged(B, S, oracle_mod, nq, T, d):
    # lengths span 1 token, block edges (15/16/17), stage edges (63/64/65), ring wrap (>256)
    # and documents longer than a workgroup's token chunk (at most 4096)
    rng = np.random.default_rng(nq * 1000 + T)
    lengths = [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 255, 257, 700, 1030, 4500, 1] + \
        rng.integers(1, 200, 150).tolist() + [5000, 3] + rng.integers(30, 181, 100).tolist()
    w = _custom(S, _past_small(lengths, nq, d, "bf16"), nq, T, d, "bf16", 7)
    H, Sor = _oracle_scores(oracle_mod, w)
    res = []
    assert "k_dense<cb::bf16_tag" in _kernels(
        lambda: B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=7, want_cells=True), res)
    r = res[0]
    np.testing.assert_allclose(r["cells"].cpu().numpy(), H, rtol=TOL["bf16"], atol=1e-5)
    np.testing.assert_allclose(r["scores"].cpu().numpy(), Sor, rtol=TOL["bf16"], atol=1e-4)
    # fp32 accumulation of exact bf16 products is far tighter than the stated tolerance
    assert np.abs(r["scores"].cpu().numpy() - Sor).max() < 5e-5 * T
    for q in range(nq):
        _check_topk(r["topk_ids"][q].cpu().numpy(), r["topk_scores"][q].cpu().numpy(), Sor[q], 7,
                    TOL["bf16"])


@pytest.mark.parametrize("dtype,nq,T,d,tokens,kernel",
                         [("bf16", 1, 32, 128, 0, "128, 2, 2, false, 4"), ("bf16", 2, 42, 128, 0, "128, 4, 4, false, 2"),
                          ("bf16", 1, 100, 64, 0, "64, 8, 8, false, 4"), ("bf16", 2, 70, 96, 0, "96, 8, 8, false, 2"),
                          ("bf16", 3, 32, 96, 0, "96, 2, 2, false, 0"), ("bf16", 40, 16, 32, 0, "32, 8, 1, false, 0"),
                          ("f32", 3, 32, 128, 0, None), ("f32", 9, 30, 128, 0, None), ("f32", 4, 24, 96, 0, None),
                          ("f32", 5, 50, 32, 0, None), ("f32", 1, 16, 64, 0, None), ("f32", 3, 64, 64, 0, None),
                          ("f32", 9, 24, 64, 0, None), ("f32", 17, 16, 32, 0, None), ("f32", 5, 32, 64, 0, None),
                          ("f32", 4, 32, 128, 260e3, "128, 2, 2, false, 0"), ("f32", 12, 30, 128, 150e3, "128, 2, 2, false, 0"),
                          ("f32", 16, 32, 128, 40e3, "128, 4, 2, false, 0"), ("f32", 4, 16, 128, 560e3, "128, 2, 1, false, 2"),
                          ("f32", 8, 32, 96, 80e3, "96, 4, 2, false, 0"), ("f32", 23, 16, 96, 30e3, "96, 2, 1, false, 0"),
                          ("f32", 8, 50, 32, 90e3, "32, 4, 4, false, 0"), ("f32", 8, 16, 64, 70e3, "64, 2, 1, false, 0"),
                          ("f32", 4, 64, 64, 90e3, "64, 4, 4, false, 0"), ("f32", 12, 24, 64, 300e3, "64, 2, 2, false, 0"),
                          ("f32", 40, 32, 32, 30e3, "32, 4, 2, false, 0")])
def test_corpus_pass_of_every_width_and_type(B, S, oracle_mod, dtype, nq, T, d, tokens, kernel):
    """Exhaustive scores beyond the calls small enough to gather: every width (96: rows padded in
    LDS), fp32, the batches whose wavefronts split the documents, and token chunks of 128 to 1,024
    with documents longer than a chunk; the same corpus through Col-Bandit's reveal pass.  kernel: the
    corpus kernel of the exhaustive call (fp32 batches that fill few of its column tiles gather)."""
    rng = np.random.default_rng(nq * 1000 + T + d)
    unit = [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 255, 257, 700, 1030, 1] + \
        rng.integers(1, 200, 150).tolist()
    lengths = unit * (int(tokens / sum(unit)) + 1) if tokens else _past_small(unit, nq, d, dtype)
    w = _custom(S, lengths, nq, T, d, dtype, 7)
    some = range(min(nq, 3 if tokens < 1e5 else 1))
    H, Sor = _oracle_scores(oracle_mod, w, some)
    res = []
    names = _kernels(lambda: B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=7, want_cells=True), res)
    assert (f"k_dense<cb::{dtype}_tag, {kernel}" if kernel else "k_gather_all<cb::f32_tag") in names
    r = res[0]
    for q in some:
        np.testing.assert_allclose(r["cells"][q].cpu().numpy(), H[q], rtol=TOL[dtype], atol=1e-5)
        np.testing.assert_allclose(r["scores"][q].cpu().numpy(), Sor[q], rtol=TOL[dtype], atol=1e-4)
        _check_topk(r["topk_ids"][q].cpu().numpy(), r["topk_scores"][q].cpu().numpy(), Sor[q], 7, TOL[dtype])
    assert f"k_dense<cb::{dtype}_tag, {d}, " in _kernels(
        lambda: B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.5, 0.01, 5, 3, trace=True), res)
    dense = res[1]
    gathered = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.5, 0.01, 5, 3, trace=True, force_gather=True)
    torch.cuda.synchronize()
    _same_run(dense, gathered)
    assert torch.equal(dense["topk_scores"], torch.gather(r["scores"], 1, dense["topk_ids"]))


@pytest.mark.parametrize("dtype,N,L,nq,T,d,kernel",
                         [("f32", 5000, 100, 1, 16, 128, "k_gather_all"), ("f32", 5000, 100, 2, 33, 64, "k_gather_all"),
                          ("f32", 5000, 100, 5, 32, 128, "k_gather_all"), ("f32", 5000, 100, 4, 32, 128, "k_dense"),
                          ("f32", 5000, 100, 8, 16, 128, "k_dense"), ("f32", 1000, 48, 32, 32, 128, "k_dense"),
                          ("f32", 50, 3000, 8, 32, 128, "k_gather_all"), ("f32", 3, 7001, 16, 48, 32, "k_gather_all"),
                          ("f32", 200, 520, 6, 32, 96, "k_gather_all"), ("bf16", 10, 3000, 1, 32, 128, "k_gather_all"),
                          ("bf16", 1, 5000, 3, 100, 64, "k_gather_all"), ("bf16", 767, 40, 1, 24, 96, "k_gather_all"),
                          ("bf16", 768, 40, 1, 8, 96, "k_gather_all"), ("bf16", 1000, 520, 1, 32, 32, "k_gather_all"),
                          ("bf16", 3000, 100, 3, 32, 128, "k_dense"), ("f32", 30, 3000, 2, 32, 128, "k_gather_all"),
                          ("f32", 600, 520, 2, 48, 64, "k_gather_all")])
def test_paths_of_exhaustive_scoring(B, dtype, N, L, nq, T, d, kernel):
    """Which path serves a call, on both sides of the rules (tiles filled against tiles multiplied, few
    long documents, the smallest calls), with documents shared by a workgroup's wavefronts and not:
    scores and cells against products in 64 bits; Doc-Uniform takes its cells from the same path."""
    g = torch.Generator(device="cuda"); g.manual_seed(N + L + nq)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    docs = torch.nn.functional.normalize(torch.randn((N * L, d), generator=g, device="cuda"), dim=1).to(td)
    Q = torch.nn.functional.normalize(torch.randn((nq, T, d), generator=g, device="cuda"), dim=2).to(td)
    off = torch.arange(0, N * L + 1, L, device="cuda", dtype=torch.int64)
    res = []
    K = min(N, 3)
    assert kernel in _kernels(lambda: B.colbandit_full_maxsim(Q, docs, off, K=K, want_cells=True), res)
    if T <= 64:
        assert kernel in _kernels(lambda: B.colbandit_doc_uniform(Q, docs, off, K, T), res)
    rows = Q.reshape(nq * T, d).double().t()
    for lo in range(0, N, 500):
        hi = min(N, lo + 500)
        H = (docs[lo * L:hi * L].double() @ rows).view(hi - lo, L, nq, T).amax(1).permute(1, 0, 2)
        for r in res:
            assert (r["scores"][:, lo:hi] - H.sum(2)).abs().max() < 1e-6 * T      # 32-bit sums of T cells below 1
        assert (res[0]["cells"][:, lo:hi] - H).abs().max() < 1e-6
    order = torch.argsort(res[0]["scores"], dim=1, descending=True, stable=True)[:, :K]
    assert torch.equal(order, res[0]["topk_ids"])


@pytest.mark.parametrize("T,d", [(1, 128), (8, 64), (9, 128), (17, 128), (24, 96), (25, 64), (33, 128), (48, 64),
                                 (49, 128), (65, 64), (96, 128), (97, 64), (7, 32), (20, 32), (47, 32), (90, 32)])
def test_packed_query_tiles_give_the_bits_of_whole_tiles(B, S, oracle_mod, T, d):
    """Batches whose query lengths leave column tiles partly empty share tiles between queries (T up to
    8, 17..24, 33..48, 65..96; the neighbours of those lengths do not); scores and cells carry the same
    bits as the small-batch kernels give, on the embeddings and on int8 codes, and agree with the oracle."""
    rng = np.random.default_rng(T)
    unit = [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 255, 257, 700, 1] + rng.integers(1, 120, 60).tolist()
    per = 1 if T <= 16 else 2 if T <= 32 else 4 if T <= 64 else 8
    nq = 37 // per + 16                                    # more than 16 tiles, an incomplete last wavefront
    step = 2
    w = _custom(S, _past_small(unit, step, d, "bf16"), nq, T, d, "bf16", 70 + T)
    packed = T <= 8 or 17 <= T <= 24 or 33 <= T <= 48 or 65 <= T <= 96
    kernel = f"{d}, 6, {per}, false, 0, true>" if packed else f"{d}, 8, {per}, false, 0, false>"
    res = []
    assert f"k_dense<cb::bf16_tag, {kernel}" in _kernels(
        lambda: B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=3, want_cells=True), res)
    r = res[0]
    H, Sor = _oracle_scores(oracle_mod, w, [nq - 1])
    np.testing.assert_allclose(r["cells"][nq - 1].cpu().numpy(), H[0], rtol=TOL["bf16"], atol=1e-5)
    np.testing.assert_allclose(r["scores"][nq - 1].cpu().numpy(), Sor[0], rtol=TOL["bf16"], atol=1e-4)
    split = f"k_dense<cb::bf16_tag, {d}, {max(2, per)}, {per}, false, {4 if per == 1 else 2}"
    assert split in _kernels(lambda: B.colbandit_full_maxsim(w.Q[:step], w.docs, w.offsets, K=0))
    for q in range(0, nq, step):
        few = B.colbandit_full_maxsim(w.Q[q:q + step], w.docs, w.offsets, K=0, want_cells=True)
        assert torch.equal(few["scores"], r["scores"][q:q + step])
        assert torch.equal(few["cells"], r["cells"][q:q + step])
    if d % 64 == 0:
        codes, scale = B.colbandit_quantize_i8(w.docs)
        assert f"k_dense<cb::i8_tag, {kernel}" in _kernels(
            lambda: B.colbandit_coarse_maxsim(w.Q, codes, scale, w.offsets, want_cells=True), res)
        c = res[1]
        for q in range(0, nq, step):
            few = B.colbandit_coarse_maxsim(w.Q[q:q + step], codes, scale, w.offsets, want_cells=True)
            assert torch.equal(few["scores"], c["scores"][q:q + step])
            assert torch.equal(few["cells"], c["cells"][q:q + step])


@pytest.mark.parametrize("codes,nq,T,Bsz", [(False, 5, 24, 4), (False, 9, 16, 3), (False, 3, 60, 4), (True, 40, 24, 4), (False, 33, 9, 4),
                                            (True, 12, 40, 16), (True, 16, 13, 4), (True, 5, 24, 4), (True, 3, 60, 4)])
def test_sixteen_tiles_of_two_wavefronts_give_the_bits_of_other_batches(B, codes, nq, T, Bsz):
    """The corpus kernel of two wavefronts (9 to 16 tiles of 128-byte rows, 2.1 M tokens or more) on ragged documents: scores and
    cells are those of single queries, a round's decisions and bounds those of gathers."""
    g = torch.Generator(device="cuda"); g.manual_seed(nq)
    d = 128 if codes else 64
    L = torch.randint(900, 1180, (2048,), device="cuda", generator=g)
    L[:900] = torch.randint(1, 2070, (900,), device="cuda", generator=g)
    L[40:200] = torch.randint(1, 20, (160,), device="cuda", generator=g)
    L[-1] += max(0, 2100000 - int(L.sum()))
    off = torch.zeros(2049, dtype=torch.int64, device="cuda"); off[1:] = L.cumsum(0)
    unit = lambda *s: torch.nn.functional.normalize(torch.randn(*s, device="cuda", generator=g), dim=-1).bfloat16()
    E, Q = unit(int(off[-1]), d), unit(nq, T, d)
    more = {}
    if codes:
        more["docs_i8"], more["docs_scale"] = B.colbandit_quantize_i8(E)
        full = lambda q: B.colbandit_coarse_maxsim(q.contiguous(), more["docs_i8"], more["docs_scale"], off, want_cells=True)
    else:
        full = lambda q: B.colbandit_full_maxsim(q.contiguous(), E, off, K=3, want_cells=True)
    tq = 1 if T <= 16 else 2 if T <= 32 else 4               # column tiles of a query
    if 9 <= nq * tq <= 16:
        res = []
        names = _kernels(lambda: full(Q), res)
        assert f"k_dense<cb::{'i8' if codes else 'bf16'}_tag, {d}, 4, {tq}, false, -2, false>" in names
        for q in (0, nq // 2, nq - 1):
            one = full(Q[q:q + 1])
            assert torch.equal(one["scores"][0], res[0]["scores"][q]) and torch.equal(one["cells"][0], res[0]["cells"][q])
    call = lambda **o: B.colbandit_topk(Q, E, off, 5, 0.3, 0.01, 5, 3, B=Bsz, trace=True, **more, **o)
    rows = nq * (16 if Bsz > 8 else 4)
    if 128 < rows <= 256:
        assert f"k_dense<cb::{'i8' if codes else 'bf16'}_tag, {d}, 4, 1, true, -2, false>" in _kernels(call)
    _same_run(call(), call(force_gather=True))


@pytest.mark.parametrize("codes,N,longest,nq,T", [(False, 3017, 0, 3, 60), (True, 3017, 0, 12, 16), (False, 172000, 49, 10, 16),
                                                  (True, 172000, 49, 4, 60), (False, 44000, 1100, 3, 33), (True, 44000, 1100, 40, 9)])
def test_halved_chunks_of_two_wavefronts(B, codes, N, longest, nq, T):
    """The corpus kernel of two wavefronts where chunks are halved: pages of 729 tokens (one or two to a chunk), short ragged
    documents whose chunks would leave a turn half empty, and as many chunks as the table of three queries holds."""
    g = torch.Generator(device="cuda"); g.manual_seed(nq)
    d = 128 if codes else 64
    L = torch.randint(1, longest + 1, (N,), device="cuda", generator=g) if longest else torch.full((N,), 729, device="cuda")
    L[N // 3:N // 3 + 5] = 0
    off = torch.zeros(N + 1, dtype=torch.int64, device="cuda"); off[1:] = L.cumsum(0)
    unit = lambda *s: torch.nn.functional.normalize(torch.randn(*s, device="cuda", generator=g), dim=-1).bfloat16()
    E, Q = torch.empty((int(off[-1]), d), dtype=torch.bfloat16, device="cuda"), unit(nq, T, d)
    for part in E.split(4000000):
        part.copy_(unit(*part.shape))
    more = {}
    if codes:
        more["docs_i8"], more["docs_scale"] = B.colbandit_quantize_i8(E)
        full = lambda q: B.colbandit_coarse_maxsim(q.contiguous(), more["docs_i8"], more["docs_scale"], off)["scores"]
    else:
        full = lambda q: B.colbandit_full_maxsim(q.contiguous(), E, off, K=3)["scores"]
    tq = 1 if T <= 16 else 4
    if nq * tq <= 16:
        res = []
        assert f"k_dense<cb::{'i8' if codes else 'bf16'}_tag, {d}, 4, {tq}, false, -2, false>" in _kernels(lambda: full(Q), res)
        for q in (0, nq - 1):
            assert torch.equal(full(Q[q:q + 1])[0], res[0][q])
    if nq * 4 > 128:
        call = lambda **o: B.colbandit_topk(Q, E, off, 5, 0.2, 0.01, 5, 3, **more, **o)
        assert f"k_dense<cb::i8_tag, {d}, 4, 1, true, -2, false>" in _kernels(lambda: call(want_stats=False))
        a, b = call(), call(force_gather=True)
        assert torch.equal(a["topk_ids"], b["topk_ids"]) and torch.equal(a["topk_scores"], b["topk_scores"])
        assert [s["survivors"] for s in a["stats"]] == [s["survivors"] for s in b["stats"]]


def test_documents_much_longer_than_a_token_chunk(B, S, oracle_mod):
    """Documents of several chunks leave runs of empty chunks behind them (a chunk belongs to the
    document that starts in it); every workgroup with an empty chunk must exit and the others
    must cover the long rows - exhaustive cells for a wide and a narrow batch, and the reveal
    pass through Col-Bandit's first round."""
    unit = [20000, 3, 9000, 1, 1, 4096, 4097, 8192, 17, 12289, 40]
    # one and two queries: the wavefronts of a workgroup split the documents
    for nq, kernel in ((1, "2, 2, false, 4"), (2, "2, 2, false, 2"), (20, "8, 2, false, 0")):
        w = _custom(S, _past_small(unit, nq, 128, "bf16"), nq, 32, 128, "bf16", 5 + nq)
        H, Sor = _oracle_scores(oracle_mod, w)
        res = []
        assert f"k_dense<cb::bf16_tag, 128, {kernel}" in _kernels(
            lambda: B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=3, want_cells=True), res)
        r = res[0]
        np.testing.assert_allclose(r["cells"].cpu().numpy(), H, rtol=TOL["bf16"], atol=1e-5)
        np.testing.assert_allclose(r["scores"].cpu().numpy(), Sor, rtol=TOL["bf16"], atol=1e-4)
    w = _custom(S, _past_small(unit, 3, 128, "bf16"), 3, 32, 128, "bf16", 9)
    assert "k_dense<cb::bf16_tag, 128, 1, 1, true" in _kernels(
        lambda: B.colbandit_topk(w.Q, w.docs, w.offsets, 2, 0.5, 0.01, 1, 3, B=4))
    _run_colbandit_case(B, oracle_mod, w, 2, 1, 4, 0.5, seed=3)


def test_full_maxsim_fp32_ragged_and_d64(B, S, oracle_mod):
    rng = np.random.default_rng(5)
    lengths = [1, 16, 17, 300] + rng.integers(1, 90, 120).tolist()
    for d, T in [(128, 32), (64, 24), (128, 50), (96, 32), (32, 40)]:
        w = _custom(S, lengths, 3, T, d, "f32", 11)
        H, Sor = _oracle_scores(oracle_mod, w)
        r = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=4, want_cells=True)
        torch.cuda.synchronize()
        np.testing.assert_allclose(r["cells"].cpu().numpy(), H, rtol=1e-5, atol=1e-6)
        np.testing.assert_allclose(r["scores"].cpu().numpy(), Sor, rtol=1e-5, atol=1e-6)


GATHER = "k_gather_all<cb::f32_tag"


@pytest.mark.parametrize("nq,T,d,times,kernel", [
    (1, 32, 128, 1, GATHER), (3, 48, 96, 1, GATHER), (1, 48, 96, 250, GATHER), (2, 40, 64, 2000, GATHER), (1, 32, 64, 9000, GATHER),
    # two and one of four wavefronts take the tiles of the batch and split the documents
    (2, 16, 32, 5300, "32, 2, 1, false, 4"), (1, 9, 64, 1, GATHER), (2, 16, 64, 2800, "64, 2, 1, false, 4"),
    (2, 16, 96, 11000, "96, 2, 1, false, 4"), (2, 13, 128, 1400, "128, 2, 1, false, 4"),
    (3, 14, 32, 1400, "32, 2, 1, false, 2"), (4, 16, 64, 240, "64, 2, 1, false, 2"), (3, 14, 96, 1900, "96, 2, 1, false, 2"),
    (4, 16, 128, 150, "128, 2, 1, false, 2"), (2, 32, 32, 6000, "32, 2, 2, false, 2"), (2, 32, 64, 6000, "64, 2, 2, false, 2"),
    (2, 20, 128, 11500, "128, 2, 2, false, 2"),
    # every wavefront its own tiles; eight wavefronts with 16 tiles in d = 96 and 128
    (3, 32, 128, 1400, "128, 2, 2, false, 0"), (9, 32, 32, 250, "32, 2, 2, false, 0"), (16, 32, 128, 150, "128, 4, 2, false, 0"),
    (16, 32, 96, 150, "96, 4, 2, false, 0"), (8, 64, 128, 1500, "128, 4, 4, false, 0")])
def test_fp32_products_on_the_bf16_pipes_keep_fp32_precision(B, S, nq, T, d, times, kernel):
    """fp32 products are sums of six bf16 products of the values' pieces.  Components spread over 2^+-40 in
    either sign, some short of bits, and some infinite: a cell is the largest sum, each within the rounding of
    an fp32 sum whatever its order.  A sum takes at most 6 d / 32 = 24 instructions and each of them five levels
    of additions, at a rounding (2^-24) of the magnitudes' sum each: 29 roundings; truncation instead of
    rounding would double it: 64 are allowed, which also covers the pieces left out (2^-24).  kernel: what serves the call,
    the gather or a corpus kernel of those compiled for fp32; documents end in the middle of blocks, at their
    ends and several in one."""
    lengths = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 5] * times
    off = torch.zeros(len(lengths) + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(torch.tensor(lengths), 0)
    docs, Q = torch.empty((int(off[-1]), d), device="cuda"), torch.empty((nq, T, d), device="cuda")
    w = S.Workload("wide-f32", "f32", Q, docs, off.cuda(), seed=3)
    g = torch.Generator(device="cuda").manual_seed(4)
    rnd = lambda *shape: torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
    for x in (w.docs, w.Q):
        v = torch.exp2(rnd(*x.shape) * 80 - 40) * torch.where(rnd(*x.shape) < 0.5, -1.0, 1.0)
        v = torch.where(rnd(*x.shape) < 0.1, torch.exp2(torch.round(torch.log2(v.abs()))), v)
        x.copy_(v)
        del v
    off = w.offsets
    inf_doc = len(lengths) - 3
    w.docs[int(off[inf_doc]) + 2, 5] = float("inf")
    w.docs[int(off[inf_doc]) + 2, d - 1] = -float("inf")
    w.docs[int(off[inf_doc + 1]) - 1, 7] = -float("inf")
    res = []
    names = _kernels(lambda: B.colbandit_full_maxsim(w.Q, w.docs, off, K=1, want_cells=True), res)
    assert (kernel if kernel is GATHER else f"k_dense<cb::f32_tag, {kernel}") in names
    E, Q = w.docs.double(), w.Q.reshape(nq * T, d).double()
    cells = res[0]["cells"].permute(1, 0, 2).reshape(len(lengths), nq * T).double()
    lens = off[1:] - off[:-1]
    doc = torch.repeat_interleave(torch.arange(len(lengths), device="cuda"), lens)
    # a product with a token's infinite component decides; two of opposite sign have no sum and no say
    dots = torch.nan_to_num(E @ Q.t(), nan=-float("inf"), posinf=float("inf"), neginf=-float("inf"))
    mags = torch.where(torch.isfinite(E), E, 0).abs() @ Q.abs().t()
    ref = torch.full_like(cells, -float("inf")).scatter_reduce(0, doc[:, None].expand_as(dots), dots, "amax")
    mag = torch.zeros_like(cells).scatter_reduce(0, doc[:, None].expand_as(dots), mags, "amax")
    fin = torch.isfinite(ref)
    assert torch.equal(cells[~fin], ref[~fin]) and (~fin).any()
    assert ((cells - ref).abs() <= 64 * 2.0 ** -24 * mag)[fin].all()


@pytest.mark.parametrize("nq,T,d,N,kernel", [(1, 32, 128, 300, "k_gather_all"), (2, 50, 96, 300, "k_gather_all"),
                                             (1, 16, 32, 300, "k_gather_all"), (32, 32, 128, 1000, "k_dense"),
                                             (40, 32, 32, 1000, "k_dense"), (32, 32, 64, 1000, "k_dense")])
def test_fp32_components_as_large_as_they_get(B, nq, T, d, N, kernel):
    """Components between bf16's largest number and fp32's, which a rounding to bf16 would make infinite, and around
    the limits from which the pieces are looked at (2, 2^40), keep the precision of fp32; products that
    overflow are infinite, and so are those of an infinity.  Bound: as for ordinary components, 64 roundings
    of the magnitudes' sum."""
    g = torch.Generator(device="cuda").manual_seed(nq + d)
    lengths = torch.randint(1, 95, (N,), generator=g, device="cuda")
    off = torch.zeros(N + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(lengths, 0)
    n = int(off[-1])
    docs = torch.randn((n, d), generator=g, device="cuda")
    Q = torch.randn((nq, T, d), generator=g, device="cuda") * 2.0 ** -30
    top = torch.tensor([0x7f7fffff, 0x7f7f8000, 0x7f7f7fff, 0x7f7f0001, 0x7e123457, 0x537fffff, 0x53800001, 0x40000000, 0x3fffffff],
                       dtype=torch.int32, device="cuda").view(torch.float32)
    at = torch.randperm(n, generator=g, device="cuda")
    for i in range(6 * top.numel()):                    # one large component in a token
        docs[at[i], (7 * i) % d] = top[i % top.numel()] * (1 if i % 4 < 2 else -1)
    a, b = at[100], at[101]
    docs[a, 5], docs[b, d - 1] = 1.2345678 * 2.0 ** 100, float("inf")
    q = nq - 1
    Q[q, 0, 5], Q[q, 1, 5] = 1.3456789 * 2.0 ** 60, -1.3456789 * 2.0 ** 60     # both signs: one overflows to +inf
    Q[q, 2, 9] = float("inf")
    res = []
    names = _kernels(lambda: B.colbandit_full_maxsim(Q, docs, off, K=1, want_cells=True), res)
    assert kernel + "<cb::f32_tag" in names
    cells = res[0]["cells"].permute(1, 0, 2).reshape(N, nq * T).double()
    E, R = docs.double(), Q.reshape(nq * T, d).double()
    doc = torch.repeat_interleave(torch.arange(N, device="cuda"), lengths)
    dots = E @ R.t()
    dots = torch.nan_to_num(dots, nan=-float("inf"), posinf=float("inf"), neginf=-float("inf"))
    dots[dots > 3.5e38], dots[dots < -3.5e38] = float("inf"), -float("inf")
    mags = torch.where(torch.isfinite(E), E, 0).abs() @ torch.where(torch.isfinite(R), R, 0).abs().t()
    ref = torch.full_like(cells, -float("inf")).scatter_reduce(0, doc[:, None].expand_as(dots), dots, "amax")
    mag = torch.zeros_like(cells).scatter_reduce(0, doc[:, None].expand_as(dots), mags, "amax")
    fin = torch.isfinite(ref)
    assert (ref == float("inf")).any() and torch.equal(cells[~fin], ref[~fin])
    assert ((cells - ref).abs() <= 64 * 2.0 ** -24 * mag)[fin].all()


def test_documents_without_tokens_get_minus_infinity_and_disturb_nothing(B, S, oracle_mod):
    """Empty documents violate the input contract (colbandit_validate_offsets reports them), but
    the scoring kernels must stay in bounds: such a document scores -inf and its neighbours,
    which share 16-token blocks with it, keep their exact scores."""
    rng = np.random.default_rng(41)
    lengths = rng.integers(1, 40, 400).tolist()
    for i in (0, 1, 7, 8, 9, 100, 250, 251, 252, 399):
        lengths[i] = 0
    unit = lengths
    # gathered, then the corpus kernels: split documents, two tiles, six packed ones, eight
    for nq, T, kernel in ((3, 32, "k_gather_all"), (1, 32, "128, 2, 2, false, 4"), (3, 32, "128, 2, 2, false, 0"),
                          (40, 24, "128, 6, 2, false, 0, true>"), (20, 32, "128, 8, 2, false, 0, false>")):
        lengths = unit if kernel == "k_gather_all" else _past_small(unit, nq, 128, "bf16")
        w = _custom(S, lengths, nq, T, 128, "bf16", 43)
        res = []
        assert kernel in _kernels(lambda: B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=0), res)
        got = res[0]["scores"].cpu().numpy()
        keep = [i for i, n in enumerate(lengths) if n > 0]
        E, off = w.host_docs(keep)
        Qh = w.host_queries()
        for q in range(min(w.nq, 6)):
            want = oracle_mod.row_sums(oracle_mod.maxsim_cells(Qh[q], E, off))
            np.testing.assert_allclose(got[q][keep], want, rtol=TOL["bf16"], atol=1e-4)
        assert np.all(np.isneginf(got[:, [i for i, n in enumerate(lengths) if n == 0]]))


@pytest.mark.parametrize("dtype,nq,d,last", [("f32", 3, 128, 1024), ("f32", 3, 128, 1025), ("bf16", 1, 128, 1024),
                                             ("bf16", 20, 64, 1025), ("bf16", 3, 96, 1024), ("f32", 40, 32, 1025)])
def test_documents_without_tokens_behind_the_last_token_are_written(B, S, dtype, nq, d, last):
    """The corpus pass: such documents begin where no chunk does (1,024: the tokens end with a chunk)
    or are alone in theirs (1,025), and score -inf; no output keeps what was in the buffer before."""
    row = d * (2 if dtype == "bf16" else 4)
    lengths = [1024] * (int(4.2e7 / (nq * row * 1024)) + 1) + [last, 0, 0, 0]
    w = _custom(S, lengths, nq, 32, d, dtype, 47)
    assert nq * w.total_tokens * row > 40e6                      # not a call small enough to gather
    out = {"scores": torch.full((nq, w.N), 7.0, device="cuda")}
    full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=4, out=out)
    torch.cuda.synchronize()
    assert torch.isneginf(full["scores"][:, -3:]).all() and (full["scores"][:, :-3].abs() < 32).all()
    assert (full["topk_ids"] < w.N - 3).all()
    res = [B.colbandit_topk(w.Q, w.docs, w.offsets, 4, 0.5, 0.01, 5, 3, trace=True, **o)
           for o in ({"later_rounds": 1}, {"force_gather": True})]
    torch.cuda.synchronize()
    _same_run(*res)


def test_nan_rows_and_token_less_documents_do_not_damage_other_documents(B, S, oracle_mod):
    """Inputs outside the contract: one document whose embeddings are NaN, one without tokens.
    Their own scores are meaningless, but they must neither enter a top-K nor wipe out a query's
    threshold: every other document keeps its exact score, the exhaustive top-K is the ordered
    head of the valid scores, and Col-Bandit returns K valid documents with those scores."""
    rng = np.random.default_rng(61)
    lengths = rng.integers(20, 90, 1200).tolist()
    p_nan, r_empty = 333, 700
    lengths[r_empty] = 0
    w = _custom(S, lengths, 4, 32, 128, "bf16", 67)
    off = w.offsets.cpu().numpy()
    w.docs[int(off[p_nan]):int(off[p_nan + 1])] = float("nan")
    K = 6
    full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=K)
    res = B.colbandit_topk(w.Q, w.docs, w.offsets, K, 0.3, 0.01, 5, 8, trace=True)
    plain = B.colbandit_topk(w.Q, w.docs, w.offsets, K, 0.3, 0.01, 5, 8)       # untraced code paths
    gathered = B.colbandit_topk(w.Q, w.docs, w.offsets, K, 0.3, 0.01, 5, 8, force_gather=True,
                                no_cell_cache=True)
    torch.cuda.synchronize()
    for other in (plain, gathered):
        assert torch.equal(other["topk_ids"], res["topk_ids"])
        assert torch.equal(other["topk_scores"], res["topk_scores"])
    sc = full["scores"].cpu().numpy()
    bad = np.array([p_nan, r_empty])
    good = np.setdiff1d(np.arange(w.N), bad)
    # the hardware maximum drops a NaN operand, so the NaN document scores -inf (NaN would do too)
    assert np.all(np.isnan(sc[:, p_nan]) | np.isneginf(sc[:, p_nan])) and np.all(np.isneginf(sc[:, r_empty]))
    E, offg = w.host_docs(good.tolist())
    for q in range(w.nq):
        want = oracle_mod.row_sums(oracle_mod.maxsim_cells(w.host_queries()[q], E, offg))
        np.testing.assert_allclose(sc[q][good], want, rtol=TOL["bf16"], atol=1e-4)
        order = good[np.lexsort((good, -sc[q][good]))][:K]
        np.testing.assert_array_equal(full["topk_ids"][q].cpu().numpy(), order)
        ids = res["topk_ids"][q].cpu().numpy()
        assert len(set(ids.tolist())) == K and not (set(ids.tolist()) & set(bad.tolist())) and ids.min() >= 0
        np.testing.assert_array_equal(res["topk_scores"][q].cpu().numpy(), sc[q][ids])
        st = res["stats"][q]
        assert st["rounds"] >= 1 and st["survivors"][st["rounds"]] >= K
        assert not res["trace"].alive[0, q][bad].any()          # both dropped in the first round
        assert not np.isnan(res["trace"].tau[0, q])


def test_topk_ties_resolve_to_lower_index(B, S):
    # documents 10.. are exact copies of documents 0..9 -> exact score ties
    base = _custom(S, [20] * 10, 2, 32, 128, "bf16", 3)
    docs = torch.cat([base.docs, base.docs, base.docs])
    off = (torch.arange(31, dtype=torch.int64) * 20).cuda()
    r = B.colbandit_full_maxsim(base.Q, docs, off, K=12)
    torch.cuda.synchronize()
    sc = r["scores"].cpu().numpy()
    np.testing.assert_array_equal(sc[:, :10], sc[:, 10:20])
    for q in range(2):
        order = np.lexsort((np.arange(30), -sc[q]))[:12]
        np.testing.assert_array_equal(r["topk_ids"][q].cpu().numpy(), order)


def test_mid_text_config2_scaled(B, S, oracle_mod):
    w = S.config(1, device="cuda", scale=0.06, nq=8)            # N=3000, bf16, planted docs
    H, Sor = _oracle_scores(oracle_mod, w)
    r = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=5)
    torch.cuda.synchronize()
    np.testing.assert_allclose(r["scores"].cpu().numpy(), Sor, rtol=TOL["bf16"], atol=1e-4)
    for q in range(w.nq):
        _check_topk(r["topk_ids"][q].cpu().numpy(), r["topk_scores"][q].cpu().numpy(), Sor[q], 5,
                    TOL["bf16"])


# ------------------------------------------------------------------ Col-Bandit
def _compare_rounds(oracle_mod, tr, q, Hq, K, M, Bsz, alpha, delta, pi, a=-1.0, b=1.0, Hexact=None):
    """Oracle on the GPU's cells vs the GPU trace, EVERY executed round of query column q.

    Each round's live set, LCB, UCB (within EPS_BAND) and threshold are compared; the survivor
    sets may differ only at documents whose UCB lies within 2*EPS_BAND of the threshold.  When
    such a band document makes the two survivor sets differ, the oracle is entered again at the
    next round with the GPU's own active set (oracle.colbandit_resume) and the comparison goes
    on to the last round, so no later round escapes.  Returns (number of re-entries, the oracle
    result that the last rounds were compared with); its final_ids are the GPU's final set.
    Hexact: the rounds decide on Hq (coarse cells) and the rescore reads Hexact."""
    N, T = Hq.shape
    if Hexact is None:
        orc = oracle_mod.colbandit_from_H(Hq, K, M, Bsz, alpha, delta, pi, a, b)
    else:
        orc = oracle_mod.colbandit_coarse(Hq, Hexact, K, M, Bsz, alpha, delta, pi, a, b)
    reentries = 0
    r = 0
    while r < orc.rounds:
        assert tr.count[r, q] == orc.counts[r], (q, r)
        live = ~np.isnan(orc.lcb[r])
        g_live = ~np.isnan(tr.lcb[r, q])
        np.testing.assert_array_equal(g_live, live)
        np.testing.assert_allclose(tr.lcb[r, q][live], orc.lcb[r][live], rtol=0, atol=EPS_BAND)
        np.testing.assert_allclose(tr.ucb[r, q][live], orc.ucb[r][live], rtol=0, atol=EPS_BAND)
        assert abs(tr.tau[r, q] - orc.tau[r]) <= EPS_BAND, (q, r)
        assert not np.any(tr.alive[r, q] & ~live), (q, r)         # nobody comes back
        mism = np.flatnonzero(tr.alive[r, q] != orc.alive[r])
        if len(mism):
            assert np.all(np.abs(orc.ucb[r][mism] - orc.tau[r]) <= 2 * EPS_BAND), (q, r, mism)
            reentries += 1
            orc = oracle_mod.colbandit_resume(Hq, K, M, Bsz, alpha, delta, pi,
                                              np.flatnonzero(tr.alive[r, q]), r + 2, a, b,
                                              H_exact=Hexact)
        r += 1
    # the GPU ran exactly these rounds, and its last active set is the oracle's final set
    assert tr.count[orc.rounds, q] == orc.counts[orc.rounds], q
    if orc.rounds < tr.tau.shape[0]:
        assert np.isnan(tr.tau[orc.rounds, q]), q                  # no further round ran
    if orc.rounds >= 1:
        np.testing.assert_array_equal(np.flatnonzero(tr.alive[orc.rounds - 1, q]), orc.final_ids)
    return reentries, orc


def _run_colbandit_case(B, oracle_mod, w, K, M, Bsz, alpha, delta=0.01, seed=0, a=0.0, b=0.0,
                        force_gather=False, later_rounds=0, coarse=None, **kw):
    """coarse = (docs_i8, docs_scale): the rounds run on int8 codes; the oracle then decides on
    the GPU's coarse cells and rescored from its exact ones.  Every round of every query is
    compared (see _compare_rounds); the number of queries that needed a re-entry at a band
    document is bounded as a sanity check on the band's width."""
    full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=0, want_cells=True)
    ckw = {} if coarse is None else {"docs_i8": coarse[0], "docs_scale": coarse[1]}
    res = B.colbandit_topk(w.Q, w.docs, w.offsets, K, alpha, delta, M, seed, B=Bsz, a=a, b=b,
                           trace=True, force_gather=force_gather, later_rounds=later_rounds, **ckw, **kw)
    Hc = None
    if coarse is not None:
        cm = B.colbandit_coarse_maxsim(w.Q, coarse[0], coarse[1], w.offsets, want_cells=True)
        torch.cuda.synchronize()
        Hc = cm["cells"].cpu().numpy().astype(np.float64)
    torch.cuda.synchronize()
    H = full["cells"].cpu().numpy().astype(np.float64)
    Sfull = full["scores"].cpu().numpy()
    ids = res["topk_ids"].cpu().numpy()
    sc = res["topk_scores"].cpu().numpy()
    tr = res["trace"]
    aa, bb = (-1.0, 1.0) if a == 0.0 and b == 0.0 else (a, b)
    diverged = 0
    for q in range(w.nq):
        pi = B.colbandit_permutation(seed, q, w.T)
        np.testing.assert_array_equal(pi, oracle_mod.permutation(seed, q, w.T))
        if Hc is None:
            div, orc = _compare_rounds(oracle_mod, tr, q, H[q], K, M, Bsz, alpha, delta, pi, aa, bb)
        else:
            div, orc = _compare_rounds(oracle_mod, tr, q, Hc[q], K, M, Bsz, alpha, delta, pi, aa, bb,
                                       Hexact=H[q])
        st = res["stats"][q]
        # survivor scores carry the same bits as the exhaustive path
        ok = ids[q] >= 0
        np.testing.assert_array_equal(sc[q][ok], Sfull[q][ids[q][ok]])
        # accounting identity (cells touched) from the GPU's own survivor counts
        T = w.T
        cells = sum((min((r + 1) * Bsz, T) - r * Bsz) * st["survivors"][r] for r in range(st["rounds"]))
        assert st["cells_elim"] == cells
        assert st["cells_rescore"] == T * st["survivors"][st["rounds"]]
        n_last = min(st["rounds"] * Bsz, T)
        assert st["cells_unique"] == cells + (T - n_last) * st["survivors"][st["rounds"]]
        assert st["survivors"] == [int(x) for x in tr.count[: st["rounds"] + 1, q]]
        # rounds, final set and top-K against the oracle that saw the GPU's active sets
        assert st["rounds"] == orc.rounds
        kk = min(K, len(orc.final_ids))
        fin_scores = Sfull[q][orc.final_ids].astype(np.float64)
        order = orc.final_ids[np.lexsort((orc.final_ids, -fin_scores))][:kk]
        np.testing.assert_array_equal(ids[q][:kk], order)
        assert np.all(ids[q][kk:] == -1)
        assert st["cells_rescore"] == orc.cells_rescore
        if div == 0:
            assert (st["cells_elim"], st["cells_unique"]) == (orc.cells_elim, orc.cells_unique)
        else:
            diverged += 1
    assert diverged <= max(1, int(0.15 * w.nq)), diverged
    # what a gathered round 2 has to read: the pairs that entered it and their document tokens
    if tr.count.shape[0] >= 3:
        L = np.diff(w.offsets.cpu().numpy())
        goes_on = [q for q in range(w.nq) if res["stats"][q]["rounds"] >= 1 and tr.count[1, q] > K + M]
        assert res["stats"][0]["pairs_round2"] == sum(int(tr.count[1, q]) for q in goes_on)
        assert res["stats"][0]["tokens_round2"] == sum(int(L[tr.alive[0, q]].sum()) for q in goes_on)
    return res, tr


def test_colbandit_fp32_config1(B, S, oracle_mod):
    w = S.config(0, device="cuda")
    res, tr = _run_colbandit_case(B, oracle_mod, w, 5, 5, 4, 0.2)
    # end to end against the oracle working from the embeddings themselves
    E, off = w.host_docs()
    pi = oracle_mod.permutation(0, 0, w.T)
    orc = oracle_mod.colbandit_lazy(w.host_queries()[0], E, off, 5, 5, 4, 0.2, 0.01, pi)
    np.testing.assert_array_equal(res["topk_ids"][0].cpu().numpy(), orc.topk_ids)
    np.testing.assert_allclose(res["topk_scores"][0].cpu().numpy(), orc.topk_scores, rtol=1e-5)
    assert res["stats"][0]["cells_unique"] == orc.cells_unique
    assert set(w.planted[0]) == set(orc.topk_ids.tolist())


@pytest.mark.parametrize("alpha,K,M,Bsz", [(0.2, 5, 5, 4), (1.0, 5, 5, 4), (0.05, 1, 0, 4),
                                           (0.2, 50, 5, 4), (0.5, 10, 5, 3), (0.2, 5, 5, 16),
                                           (0.2, 5, 0, 1), (1.0, 3, 2, 5)])
def test_colbandit_bf16_rounds_match_oracle(B, S, oracle_mod, alpha, K, M, Bsz):
    w = S.config(1, device="cuda", scale=0.04, nq=6)            # N=2000, planted docs
    _run_colbandit_case(B, oracle_mod, w, K, M, Bsz, alpha)


def test_colbandit_topic_corpus_and_pages(B, S, oracle_mod):
    w = S.config(2, device="cuda", scale=0.008, nq=10)          # N=4000 topic mixture
    _run_colbandit_case(B, oracle_mod, w, 5, 5, 4, 0.2)
    _run_colbandit_case(B, oracle_mod, w, 10, 5, 4, 0.2, seed=9)
    w = S.config(3, device="cuda", scale=0.01, nq=5)            # 200 pages x 1030 tokens, T=24
    _run_colbandit_case(B, oracle_mod, w, 5, 5, 4, 0.2)
    _run_colbandit_case(B, oracle_mod, w, 5, 5, 4, 1.0)


def test_colbandit_gather_and_dense_first_round_agree(B, S, oracle_mod):
    w = S.config(1, device="cuda", scale=0.03, nq=5)
    r1 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, 0.01, 5, 3, trace=True)
    r2 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, 0.01, 5, 3, trace=True, force_gather=True)
    torch.cuda.synchronize()
    for f in ("count", "tau", "lcb", "ucb", "alive"):
        np.testing.assert_array_equal(getattr(r1["trace"], f), getattr(r2["trace"], f))
    assert torch.equal(r1["topk_ids"], r2["topk_ids"]) and torch.equal(r1["topk_scores"], r2["topk_scores"])


def _same_run(r1, r2):
    for f in ("count", "tau", "lcb", "ucb", "alive"):
        np.testing.assert_array_equal(getattr(r1["trace"], f), getattr(r2["trace"], f))
    assert torch.equal(r1["topk_ids"], r2["topk_ids"]) and torch.equal(r1["topk_scores"], r2["topk_scores"])
    # which path computed a round's cells may differ between the runs; nothing else may
    counts = lambda st: {k: v for k, v in st.items() if not k.startswith("ms_")
                         and k not in ("corpus_pass_rounds", "cells_computed")}
    assert [counts(a) for a in r1["stats"]] == [counts(b) for b in r2["stats"]]


@pytest.mark.parametrize("alpha,Bsz,T", [(0.2, 4, 32), (1.0, 4, 32), (0.5, 3, 24), (0.2, 8, 40), (1.0, 16, 100)])
def test_cell_cache_and_regather_give_identical_runs(B, S, alpha, Bsz, T):
    """Caching a visited document's cells must not change a single decision or bit."""
    rng = np.random.default_rng(T)
    w = _custom(S, rng.integers(1, 120, 1500).tolist(), 4, T, 128, "bf16", 5)
    r1 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, alpha, 0.01, 5, 3, B=Bsz, trace=True)
    r2 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, alpha, 0.01, 5, 3, B=Bsz, trace=True,
                          no_cell_cache=True)
    torch.cuda.synchronize()
    assert max(s["rounds"] for s in r1["stats"]) >= 2
    _same_run(r1, r2)


@pytest.mark.parametrize("dtype,coarse", [("bf16", False), ("f32", False), ("bf16", True)])
def test_without_a_round_all_documents_are_scored_like_an_exhaustive_call(B, S, dtype, coarse):
    """N <= K + M: the gather of whole matrices, not one workgroup per survivor; ids and bits of the
    exhaustive call, also when codes were given."""
    w = _custom(S, np.random.default_rng(8).integers(1, 32, 300).tolist(), 20, 24, 64, dtype, 8)
    kw = {}
    if coarse:
        kw["docs_i8"], kw["docs_scale"] = B.colbandit_quantize_i8(w.docs)
    res = []
    names = _kernels(lambda: B.colbandit_topk(w.Q, w.docs, w.offsets, 7, 0.2, 0.01, 293, 3, want_stats=False, **kw), res)
    assert "k_gather_all" in names and "k_gather_survivors" not in names and "k_select_prune" not in names
    full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=7)
    torch.cuda.synchronize()
    assert torch.equal(res[0]["topk_ids"], full["topk_ids"]) and torch.equal(res[0]["topk_scores"], full["topk_scores"])


def test_few_long_fp32_documents_do_not_stream_round_after_round(B, S):
    """A corpus pass takes as long as a document in one workgroup; where that outweighs the gather of the few
    pairs there are, the rounds gather."""
    w = _custom(S, np.random.default_rng(5).integers(800, 4000, 131).tolist(), 34, 16, 64, "f32", 5)
    res = [B.colbandit_topk(w.Q, w.docs, w.offsets, 43, 0.3, 0.01, 0, 3, trace=True, **o) for o in ({}, {"later_rounds": 1})]
    torch.cuda.synchronize()
    assert all(s["corpus_pass_rounds"] == [] for s in res[0]["stats"])
    _same_run(*res)


def test_rounds_that_a_pass_could_not_shorten_launch_none(B, S):
    """Lists beyond the cell cache that are gathered in less than two passes and a round's launches: the
    corpus kernel runs in round 1 only, and the decisions are those of passes in every round."""
    w = _custom(S, np.random.default_rng(7).integers(32, 65, 17000).tolist(), 3, 53, 32, "bf16", 7)
    call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, 100, 0.1, 0.01, 0, 2, B=2, **o)
    call()
    assert [_kernels(lambda: call(**o)).count("k_dense<") for o in ({}, {"later_rounds": 1})] == [1, 27]
    _same_run(call(trace=True), call(trace=True, later_rounds=1))


@pytest.mark.parametrize("nq,T,d,coarse", [(7, 21, 64, False), (12, 32, 64, False), (7, 24, 128, True)])
def test_full_lists_of_a_corpus_in_the_last_level_cache_launch_no_later_round(B, S, nq, T, d, coarse):
    """Lists that fit the cell cache, over documents few enough to gather whole: one gathered round, and the same run
    as with a corpus pass in every round."""
    w = _custom(S, np.random.default_rng(nq).integers(1, 260, 5000).tolist(), nq, T, d, "bf16", 9)
    more = {}
    if coarse:
        more["docs_i8"], more["docs_scale"] = B.colbandit_quantize_i8(w.docs)
    for alpha in (0.2, 1.0):
        names = _kernels(lambda: B.colbandit_topk(w.Q, w.docs, w.offsets, 10, alpha, 0.01, 5, 3, want_stats=False, **more))
        assert names.count("k_gather_round<") == 1 and names.count("k_dense<") == 1
        r = [B.colbandit_topk(w.Q, w.docs, w.offsets, 10, alpha, 0.01, 5, 3, trace=True, later_rounds=m, **more) for m in (0, 1)]
        torch.cuda.synchronize()
        _same_run(*r)


@pytest.mark.parametrize("nq,T,d", [(48, 64, 128), (33, 40, 96), (60, 64, 32)])
def test_full_fp32_lists_of_a_corpus_in_the_last_level_cache(B, S, nq, T, d):
    """fp32 queries of several tiles, whose full lists cost more matrix work than their bytes say: round 2 gathers them
    and is the last launched, and the run is that of a corpus pass in every round."""
    w = _custom(S, np.random.default_rng(nq).integers(1, 180, 3000).tolist(), nq, T, d, "f32", 9)
    for alpha in (0.2, 1.0):
        call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, 10, alpha, 0.01, 5, 3, **o)
        names = _kernels(lambda: call(want_stats=False))
        assert names.count("k_gather_round<") == 1 and names.count("k_dense<") == 1
        r = [call(trace=True, later_rounds=m) for m in (0, 1)]
        torch.cuda.synchronize()
        _same_run(*r)


@pytest.mark.parametrize("N,nq,T,longest", [(20000, 5, 32, 3), (40000, 3, 48, 2), (9000, 9, 24, 5), (30000, 2, 100, 2)])
def test_gathered_rounds_of_more_pairs_than_workers(B, S, N, nq, T, longest):
    """Lists of unequal length whose pairs (beyond 32,768) are dealt out in streams, held as ids and in
    the cell cache: the decisions, bounds and bits of the corpus passes and of gathers in every round."""
    rng = np.random.default_rng(N)
    w = _custom(S, rng.integers(1, longest + 1, N).tolist(), nq, T, 128, "bf16", N)
    w.Q[0] *= 0.25                                           # close scores: a list that shrinks late
    runs = [B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.9, 0.01, 5, 3, trace=True, **o)
            for o in ({"later_rounds": 2}, {"later_rounds": 1}, {"later_rounds": 2, "no_cell_cache": True})]
    torch.cuda.synchronize()
    assert runs[0]["stats"][0]["pairs_round2"] > 32768
    for r in runs[1:]:
        _same_run(runs[0], r)


@pytest.mark.parametrize("N,nq,T,d,alpha,coarse,shared", [
    (600, 9, 24, 128, 1.0, False, True), (600, 9, 24, 128, 0.05, False, False), (1100, 5, 16, 64, 1.0, False, True),
    (700, 21, 40, 96, 1.0, False, True), (500, 17, 100, 32, 1.0, False, True), (800, 11, 9, 128, 1.0, True, True),
    (700, 13, 33, 64, 1.0, True, True), (17000, 6, 32, 32, 0.5, False, True)])
def test_long_documents_are_gathered_for_several_queries_at_once(B, S, N, nq, T, d, alpha, coarse, shared):
    """Round 2 by document (k_gather_docs): groups of queries of every size, documents of ragged length and without tokens,
    all widths and the codes, lists that are too few for it, lists beyond the cell cache.  The decisions, bounds and bits
    are those of gathers pair by pair in every round, and of corpus passes."""
    rng = np.random.default_rng(N + T)
    L = rng.integers(200, 460, N)
    L[rng.integers(0, N, 5)] = 0
    L[rng.integers(0, N, 40)] = rng.integers(1, 40, 40)
    L[:3] = (16, 17, 1500)
    w = _custom(S, L.tolist(), nq, T, d, "bf16", 3)
    w.Q[0] *= 0.25                                           # lists of unequal length
    more = {}
    if coarse:
        more["docs_i8"], more["docs_scale"] = B.colbandit_quantize_i8(w.docs)
    call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, 5, alpha, 0.01, 5, 3, trace=True, **more, **o)
    names = _kernels(lambda: B.colbandit_topk(w.Q, w.docs, w.offsets, 5, alpha, 0.01, 5, 3, want_stats=False, **more))
    assert "k_gather_docs<" in names                         # (which ends at once where round 2 is not its own)
    runs = [call(), call(no_cell_cache=True, later_rounds=2), call(later_rounds=1), call(later_rounds=2)]
    torch.cuda.synchronize()
    # with later_rounds=2 no pass takes the round, and the lists entered decide
    assert 2 in runs[2]["stats"][0]["corpus_pass_rounds"] and not runs[3]["stats"][0]["corpus_pass_rounds"]
    enough = 4096 if N <= 8192 else N // 2
    held = sum(int(c) for c in runs[3]["trace"].count[1] if 10 < c <= 16384 and 4 * c * nq >= enough)
    assert (held >= enough) == shared
    for r in runs[1:]:
        _same_run(runs[0], r)


def test_many_queries_and_wild_documents_gathered_for_several_queries_at_once(B, S):
    """k_gather_docs with 300 queries, and documents outside the contract that round 1 has not dropped: rows of NaN, which no
    maximum takes, and components that make some cells infinite but, for many queries, none of those revealed by then.  The
    run of gathers pair by pair that keep no cells, to the bit."""
    w = _custom(S, np.random.default_rng(5).integers(250, 320, 600).tolist(), 300, 20, 64, "bf16", 5)
    off = w.offsets.tolist()
    for i in range(0, 600, 30):
        w.docs[off[i] + 3:off[i] + 40] = float("nan")
        w.docs[off[i + 1] + 17, 5] = float("inf")
        w.docs[off[i + 2] + 64, 9] = -float("inf")
    call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 1.0, 0.01, 5, 3, B=2, trace=True, later_rounds=2, **o)
    names = _kernels(call)
    assert "k_gather_docs<" in names
    runs = [call(), call(no_cell_cache=True)]
    torch.cuda.synchronize()
    assert runs[0]["trace"].count[1].min() > 100
    in_round_2 = runs[0]["trace"].alive[0]
    for first, some in ((0, 300), (1, 30), (2, 30)):
        assert in_round_2[:, first::30].any(1).sum() >= some
    _same_run(*runs)


def test_lists_entered_by_document_before_a_corpus_pass(B, S):
    """Round 2 is a corpus pass although lists have been entered by document: the last of them leave the table unfilled."""
    w = _custom(S, np.random.default_rng(8).integers(270, 310, 1113).tolist(), 166, 24, 64, "bf16", 8)
    call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 1.0, 0.01, 5, 3, **o)
    assert "k_gather_docs<" in _kernels(lambda: call(want_stats=False))
    runs = [call(trace=True), call(trace=True, later_rounds=2)]
    torch.cuda.synchronize()
    assert 2 in runs[0]["stats"][0]["corpus_pass_rounds"] and not runs[1]["stats"][0]["corpus_pass_rounds"]
    _same_run(*runs)


@pytest.mark.parametrize("dtype,N,nq,T,d,Bsz,alpha,coarse",
                         [("bf16", 11, 1, 1, 128, 1, 1.0, None), ("bf16", 1000, 3, 32, 128, 4, 0.2, None),
                          ("bf16", 1025, 4, 128, 96, 7, 1.0, None), ("bf16", 4097, 1, 65, 32, 16, 1.0, None),
                          ("f32", 1000, 1, 32, 128, 4, 0.5, None), ("f32", 5000, 1, 17, 64, 3, 1.0, None),
                          ("bf16", 900, 3, 32, 128, 4, 0.5, "int8"), ("bf16", 16384, 1, 24, 64, 4, 1.0, None)])
def test_smallest_calls_that_visit_every_document_once(B, S, oracle_mod, dtype, N, nq, T, d, Bsz, alpha, coarse):
    """Small corpora have all cells computed and cached in round 1: the decisions, bounds and bits
    of the rounds that gather anew, and the oracle's answer; lists around the sizes that the prune
    kernel holds in registers, the longest list that the cache holds, T up to its limit."""
    rng = np.random.default_rng(N + T)
    w = _custom(S, rng.integers(1, 4 if N > 5000 else 16, N).tolist(), nq, T, d, dtype, 6 + N)
    kw = dict(B=Bsz, trace=True)
    if coarse:
        kw["docs_i8"], kw["docs_scale"] = B.colbandit_quantize_i8(w.docs)
    runs = [B.colbandit_topk(w.Q, w.docs, w.offsets, 5, alpha, 0.01, 5, 3, **kw, **o)
            for o in ({}, {"no_cell_cache": True}, {"force_gather": True}, {"later_rounds": 2})]
    torch.cuda.synchronize()
    for r in runs[1:]:
        _same_run(runs[0], r)
    st = runs[0]["stats"]
    # on int8 codes the exact rescore computes the survivors' cells once more
    assert all(s["cells_computed"] == T * N + (s["cells_rescore"] if coarse else 0) for s in st)
    assert all(s["corpus_pass_rounds"] == [] for s in st)
    if not coarse:
        _run_colbandit_case(B, oracle_mod, w, 5, 5, Bsz, alpha, seed=3)


@pytest.mark.parametrize("dtype,d,nq,N,T,Bsz,reveals", [
    ("bf16", 64, 8, 2100, 32, 4, True), ("bf16", 64, 9, 1365, 24, 4, True), ("bf16", 64, 9, 1366, 24, 4, False),
    ("bf16", 64, 13, 1000, 70, 16, False), ("bf16", 64, 12, 1000, 128, 3, True),
    ("f32", 128, 1, 4500, 48, 4, True), ("f32", 128, 3, 1365, 40, 4, True), ("f32", 128, 3, 1366, 40, 4, False),
    ("f32", 128, 4, 300, 64, 3, False), ("f32", 128, 5, 900, 32, 4, True), ("f32", 128, 6, 900, 32, 4, False),
    ("f32", 96, 6, 800, 33, 2, False), ("f32", 96, 8, 900, 32, 4, True), ("bf16", 128, 5, 900, 65, 4, True),
    ("bf16", 128, 6, 900, 65, 4, False), ("bf16", 128, 8, 900, 64, 4, True)])
def test_round_one_revealed_as_the_cells_are_cached(B, S, dtype, d, nq, N, T, Bsz, reveals):
    """Both sides of the rule by which the smallest calls reveal round 1 while they compute the cells, with the seeded order and
    with a table (one that holds a token twice among them): the run of gathers that keep no cells."""
    w = _custom(S, np.random.default_rng(nq).integers(1, 12, N).tolist(), nq, T, d, dtype, 11)
    pi = torch.stack([torch.randperm(T, generator=torch.Generator().manual_seed(q)) for q in range(nq)]).to(torch.int32)
    pi[-1, 1] = pi[-1, 0]
    tiles = next(t for t in (1, 2, 4, 8) if 16 * t >= T)
    for more in ({}, {"pi": pi.cuda()}):
        call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.3, 0.01, 5, 3, B=Bsz, **more, **o)
        assert f"k_cache_all<cb::{dtype}_tag, {d}, {tiles}, {str(reveals).lower()}>" in _kernels(lambda: call(want_stats=False))
        _same_run(call(trace=True), call(trace=True, no_cell_cache=True))


def test_queries_that_end_in_round_one_are_finished_with_the_others(B, S):
    """Lists that all fit the cell cache: the prune of round 2 ends the call, also for queries that had ended in round 1 or
    hold K documents or fewer by then; without a launch for their scores, and with the run of gathers that keep no cells."""
    w = _custom(S, np.random.default_rng(2).integers(20, 90, 3000).tolist(), 6, 32, 128, "bf16", 12)
    off = w.offsets.cpu().tolist()
    for q, docs in ((0, range(40, 50)), (3, range(7, 12)), (4, range(100, 160))):
        for i in docs:                                       # every token of the query found in the document
            n = min(32, off[i + 1] - off[i])
            w.docs[off[i]:off[i] + n] = w.Q[q, :n]
    for K, M in ((5, 5), (5, 0), (70, 3)):
        call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, K, 0.05, 0.01, M, 3, **o)
        names = _kernels(lambda: call(want_stats=False))
        assert names.count("k_select_prune<") == 2 and "k_gather_survivors" not in names and "k_topk" not in names
        runs = [call(trace=True), call(trace=True, no_cell_cache=True), call(trace=True, later_rounds=1)]
        torch.cuda.synchronize()
        rounds = [s["rounds"] for s in runs[0]["stats"]]
        assert max(rounds) > 1 and (K > 5 or min(rounds) == 1)
        for r in runs[1:]:
            _same_run(runs[0], r)


@pytest.mark.parametrize("N,T,Bsz,K,M,coarse", [(64, 32, 4, 5, 0, False), (65, 32, 4, 5, 5, False), (128, 21, 4, 1, 0, False),
                                              (129, 100, 3, 7, 0, False), (192, 70, 16, 30, 3, False), (255, 32, 5, 60, 4, False),
                                              (256, 32, 4, 250, 0, False), (257, 24, 2, 5, 0, False), (300, 32, 4, 64, 0, True),
                                              (1000, 128, 7, 65, 1, False), (1030, 32, 1, 3, 2, True)])
def test_short_cached_lists_by_one_wavefront(B, S, N, T, Bsz, K, M, coarse):
    """Lists around 64, 128, 192 and 256 entries, which one wavefront takes from some round on (batches of up to
    four and of more, reveal orders beyond 64 tokens, lists that shrink by a place or not), and final lists
    around 64: every round's survivors, bounds and threshold, and the top-K, are those of rounds that read
    nothing from a cache."""
    rng = np.random.default_rng(N + T)
    w = _custom(S, rng.integers(1, 40, N).tolist(), 3, T, 64, "bf16", N)
    more = {}
    if coarse:
        more["docs_i8"], more["docs_scale"] = B.colbandit_quantize_i8(w.docs)
    for alpha in (0.1, 0.3, 1.0):
        r = [B.colbandit_topk(w.Q, w.docs, w.offsets, K, alpha, 0.01, M, 3, B=Bsz, trace=True, no_cell_cache=c, **more)
             for c in (False, True)]
        torch.cuda.synchronize()
        _same_run(*r)
        plain = B.colbandit_topk(w.Q, w.docs, w.offsets, K, alpha, 0.01, M, 3, B=Bsz, want_stats=False, **more)
        assert torch.equal(plain["topk_ids"], r[0]["topk_ids"]) and torch.equal(plain["topk_scores"], r[0]["topk_scores"])


@pytest.mark.parametrize("alpha,Bsz,T,nq", [(1.0, 4, 32, 4), (0.5, 3, 24, 9), (1.0, 16, 100, 2), (0.2, 4, 32, 40)])
def test_later_rounds_by_corpus_pass_or_by_gather_are_identical(B, S, oracle_mod, alpha, Bsz, T, nq):
    """Rounds >= 2 revealed by the corpus-streaming pass (merged into the running statistics by
    the prune kernel), by per-pair gathers, or by the device-side choice between them: the
    same cells, the same merge, so every bound, threshold, survivor and output bit agrees."""
    rng = np.random.default_rng(100 + T)
    w = _custom(S, rng.integers(1, 90, 3000).tolist(), nq, T, 128, "bf16", 17)
    runs = [B.colbandit_topk(w.Q, w.docs, w.offsets, 5, alpha, 0.01, 5, 4, B=Bsz, trace=True,
                             later_rounds=m) for m in (2, 1, 0)]
    torch.cuda.synchronize()
    assert max(s["rounds"] for s in runs[0]["stats"]) >= 3
    _same_run(runs[0], runs[1])
    _same_run(runs[0], runs[2])
    # the statistics name the rounds that streamed the corpus: none when gathers are forced,
    # every round >= 2 that still had an ids-mode query when the pass is forced
    assert all(s["corpus_pass_rounds"] == [] for s in runs[0]["stats"])
    forced = runs[1]["stats"][0]["corpus_pass_rounds"]
    assert forced and forced[0] == 2 and forced == list(range(2, 2 + len(forced)))
    assert set(runs[2]["stats"][0]["corpus_pass_rounds"]) <= set(forced)
    # the streaming pass also under the cache-free mode, and against the oracle
    r3 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, alpha, 0.01, 5, 4, B=Bsz, trace=True,
                          later_rounds=1, no_cell_cache=True)
    torch.cuda.synchronize()
    _same_run(runs[0], r3)
    _run_colbandit_case(B, oracle_mod, w, 5, 5, Bsz, alpha, seed=4, later_rounds=1)


def test_device_side_choice_takes_the_corpus_pass_for_large_active_sets(B, S):
    """A conservative radius on a topic corpus keeps thousands of documents per query alive:
    the automatic mode must then not fall behind the exhaustive path by gathering them all."""
    w = S.config(4, device="cuda", scale=0.2, nq=64)                 # N=20,000, 64 queries
    ws = B.new_workspace(w.nq, w.T, w.d, w.N, w.total_tokens, "cuda")
    res = {}
    for m in (0, 2):
        r = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 1.0, 0.01, 5, w.seed, workspace=ws,
                             later_rounds=m)
        res[m] = r
    torch.cuda.synchronize()
    assert torch.equal(res[0]["topk_ids"], res[2]["topk_ids"])
    assert torch.equal(res[0]["topk_scores"], res[2]["topk_scores"])
    c = lambda st: {k: v for k, v in st.items() if not k.startswith("ms_")
                    and k not in ("corpus_pass_rounds", "cells_computed")}
    assert [c(a) for a in res[0]["stats"]] == [c(b) for b in res[2]["stats"]]
    assert 2 in res[0]["stats"][0]["corpus_pass_rounds"] and res[2]["stats"][0]["corpus_pass_rounds"] == []
    print("later reveals: auto %.3f ms, gather %.3f ms" %
          (res[0]["stats"][0]["ms_later_reveals"], res[2]["stats"][0]["ms_later_reveals"]))


def test_cells_computed_counts_what_the_kernels_multiply(B, S):
    """cells_computed against the path each round took: per-pair gathers without the cache
    compute exactly the revealed cells; with the cache the first gathered round computes all T
    cells of its documents and nothing afterwards; a corpus pass computes the batch for all N."""
    rng = np.random.default_rng(12)
    w = _custom(S, rng.integers(1, 90, 3000).tolist(), 4, 32, 128, "bf16", 19)
    N, T, Bsz = w.N, w.T, 4
    plain = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.5, 0.01, 5, 4, no_cell_cache=True, later_rounds=2)
    cached = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.5, 0.01, 5, 4, later_rounds=2)
    passes = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.5, 0.01, 5, 4, later_rounds=1, no_cell_cache=True)
    torch.cuda.synchronize()
    assert max(s["rounds"] for s in plain["stats"]) >= 3
    for sp, sc, sd in zip(plain["stats"], cached["stats"], passes["stats"]):
        assert sp["survivors"] == sc["survivors"] == sd["survivors"]
        surv, R = sp["survivors"], sp["rounds"]
        assert sp["cells_computed"] == sp["cells_elim"] + sp["cells_rescore"]
        want = Bsz * N + (T * surv[1] if R >= 2 else T * surv[R])      # round 1, then one visit
        assert sc["cells_computed"] == want
        assert sd["cells_computed"] == Bsz * N * R + T * surv[R]       # every round a pass, then the rescore
        assert sd["corpus_pass_rounds"] == list(range(2, 2 + len(sd["corpus_pass_rounds"])))


def test_active_sets_larger_than_the_cell_cache(B, S, oracle_mod):
    """N above the cache capacity with a conservative radius: the first gathered rounds
    run uncached and a query switches to its cache only once its active set fits."""
    rng = np.random.default_rng(8)
    w = _custom(S, rng.integers(2, 9, 40000).tolist(), 3, 32, 128, "bf16", 21)
    r1 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 1.0, 0.01, 5, 1, trace=True)
    r2 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 1.0, 0.01, 5, 1, trace=True, no_cell_cache=True)
    torch.cuda.synchronize()
    surv = [s["survivors"] for s in r1["stats"]]
    assert any(len(x) > 2 and x[1] > 16384 for x in surv), surv     # really started above capacity
    _same_run(r1, r2)
    _run_colbandit_case(B, oracle_mod, w, 5, 5, 4, 1.0, seed=1)


@pytest.mark.parametrize("K", [5, 300])
def test_long_lists_take_the_sampled_prefilter(B, S, oracle_mod, K):
    """Lists far longer than the selection kernels' sample: the threshold of a strided sample
    pre-filters candidates before the exact selection.  Checked against the oracle (rounds,
    survivors, top-K) and against a full sort of the GPU's own scores."""
    rng = np.random.default_rng(77)
    w = _custom(S, rng.integers(1, 4, 150000).tolist(), 2, 32, 128, "bf16", 31)
    full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=K)
    torch.cuda.synchronize()
    sc = full["scores"].cpu().numpy()
    for q in range(w.nq):
        order = np.lexsort((np.arange(w.N), -sc[q]))[:K]
        np.testing.assert_array_equal(full["topk_ids"][q].cpu().numpy(), order)
        np.testing.assert_array_equal(full["topk_scores"][q].cpu().numpy(), sc[q][order])
    _run_colbandit_case(B, oracle_mod, w, K, 5, 4, 0.2, seed=2)


@pytest.mark.parametrize("nq", [1, 3])
def test_long_lists_stay_long_under_a_conservative_radius(B, S, oracle_mod, nq):
    """alpha_ef = 1 keeps most of 150,000 documents alive for several rounds: explicit lists
    longer than the pre-filter limit, cut down by several workgroups per query, revealed by the
    corpus pass (statistics merged for the candidates only) or by gathers - same decisions."""
    rng = np.random.default_rng(78)
    w = _custom(S, rng.integers(1, 4, 150000).tolist(), nq, 32, 128, "bf16", 37)
    runs = [B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 1.0, 0.01, 5, 6, trace=True, later_rounds=m)
            for m in (1, 2)]
    torch.cuda.synchronize()
    surv = runs[0]["stats"][0]["survivors"]
    assert len(surv) > 3 and surv[2] > 131072, surv          # long lists beyond round 1
    _same_run(runs[0], runs[1])
    _run_colbandit_case(B, oracle_mod, w, 5, 5, 4, 1.0, seed=6, later_rounds=1)


@pytest.mark.parametrize("N,nq,later", [(40000, 3, 0), (40000, 3, 1), (90000, 2, 2)])
def test_long_lists_under_a_small_radius_are_pruned_by_the_last_workgroup_to_come(B, S, oracle_mod, N, nq, later):
    """k_select_round (small alpha_ef, few workgroups) on lists that stay longer than a tile for some rounds and fall below
    it, in gathered rounds and corpus passes: every round as the oracle has it."""
    w = _custom(S, np.random.default_rng(N).integers(1, 4, N).tolist(), nq, 32, 64, "bf16", 23)
    call = lambda **o: B.colbandit_topk(w.Q, w.docs, w.offsets, 200, 0.25, 1e-30, 5, 4, B=2, later_rounds=later, **o)
    names = _kernels(lambda: call(want_stats=False))
    assert "k_select_round" in names and names.count("k_select_segments") == 1
    counts = call(trace=True)["trace"].count
    assert (counts[2] > 16384).all() and (counts[-2] < 16384).any()
    _run_colbandit_case(B, oracle_mod, w, 200, 5, 2, 0.25, delta=1e-30, seed=4, later_rounds=later)


def test_first_workgroups_of_the_merged_rounds_lie_side_by_side(B, S, tmp_path):
    """k_select_round: of a query's eight workgroups the first prunes a short list alone; consecutive workgroups go to the eight
    XCDs in turn, so the queries are the grid's fast axis."""
    import json
    from torch.profiler import ProfilerActivity, profile
    w = _custom(S, np.random.default_rng(3).integers(1, 8, 60000).tolist(), 16, 32, 32, "bf16", 3)
    for _ in range(5):
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.1, 0.01, 5, 3, want_stats=False)
            torch.cuda.synchronize()
        p.export_chrome_trace(str(tmp_path / "t.json"))
        events = json.load(open(tmp_path / "t.json"))["traceEvents"]
        grids = [e["args"]["grid"] for e in events if "k_select_round" in e.get("name", "") and "grid" in e.get("args", {})]
        if grids:
            break
    assert grids and all(g == [16, 8, 1] for g in grids)


def test_wild_documents_in_long_lists_pruned_by_the_last_workgroup_to_come(B, S):
    """k_select_round on lists that hold documents outside the contract, in any segment: the run of the same queries in a batch
    too large for it, whose rounds are filtered and pruned by two launches."""
    rng = np.random.default_rng(77)
    lengths = rng.integers(1, 4, 40000)
    lengths[rng.integers(0, 40000, 50)] = 0
    w = _custom(S, lengths.tolist(), 200, 32, 32, "bf16", 24)
    tokens = int(w.offsets[-1])
    w.docs[torch.from_numpy(rng.integers(0, tokens, 200)).cuda()] = float("nan")
    w.docs[torch.from_numpy(rng.integers(0, tokens, 200)).cuda(), 3] = float("inf")
    w.docs[torch.from_numpy(rng.integers(0, tokens, 200)).cuda(), 7] = -float("inf")
    call = lambda n, **o: B.colbandit_topk(w.Q[:n].contiguous(), w.docs, w.offsets, 200, 0.25, 1e-30, 5, 4, B=2, **o)
    assert "k_select_round" in _kernels(lambda: call(3, want_stats=False))
    assert "k_select_round" not in _kernels(lambda: call(200, want_stats=False))
    few, many = call(3, trace=True), call(200, trace=True, trace_queries=[0, 1, 2])
    torch.cuda.synchronize()
    assert (few["trace"].count[2] > 16384).all() and few["trace"].alive[1].any()
    for f in ("count", "tau", "lcb", "ucb", "alive"):
        np.testing.assert_array_equal(getattr(few["trace"], f), getattr(many["trace"], f))
    assert torch.equal(few["topk_ids"], many["topk_ids"][:3]) and torch.equal(few["topk_scores"], many["topk_scores"][:3])


@pytest.mark.parametrize("N,K,alpha", [(1024, 5, 0.2), (1025, 32, 1.0), (4096, 5, 1.0), (4097, 33, 1.0), (8192, 5, 1.0),
                                       (8193, 1, 1.0), (16384, 300, 1.0), (16385, 5, 1.0), (24577, 1000, 1.0),
                                       (40961, 500, 0.9), (33000, 508, 1.0), (33100, 508, 1.0)])
def test_selection_at_the_edges_of_its_tiles(B, S, oracle_mod, N, K, alpha):
    """Lists around what the selection kernels hold in registers (1,024 entries per place of a
    thread, 4,096 in all), around the tile beyond which a list is pre-filtered (16,384), and K around
    the number of group maxima (32); cached lists longer than the registers run their first
    rounds from memory; longer lists and K on both sides of what LDS holds of a sampled bound's
    entries.  A tenth of the documents are copies of one document."""
    rng = np.random.default_rng(N + K)
    w = _custom(S, rng.integers(1, 3, N).tolist(), 2, 32, 128, "bf16", 91 + N)
    off = w.offsets.cpu().numpy()
    for i in rng.choice(N, N // 10, replace=False):
        w.docs[off[i]] = w.docs[0]
    _run_colbandit_case(B, oracle_mod, w, K, 5, 4, alpha, seed=N)


def test_long_lists_with_massive_ties(B, S):
    """150,000 documents that are copies of 40 distinct ones: the K-th score is shared by
    thousands; ties resolve to the lowest indices."""
    base = _custom(S, [3] * 40, 2, 32, 128, "bf16", 13)
    reps = 3750
    docs = base.docs.repeat(reps, 1)
    off = (torch.arange(40 * reps + 1, dtype=torch.int64) * 3).cuda()
    r = B.colbandit_full_maxsim(base.Q, docs, off, K=100)
    torch.cuda.synchronize()
    sc = r["scores"].cpu().numpy()
    for q in range(2):
        order = np.lexsort((np.arange(40 * reps), -sc[q]))[:100]
        np.testing.assert_array_equal(r["topk_ids"][q].cpu().numpy(), order)


def test_colbandit_support_wider_than_default(B, S, oracle_mod):
    w = S.config(1, device="cuda", scale=0.02, nq=3)
    _run_colbandit_case(B, oracle_mod, w, 5, 5, 4, 0.2, a=-1.5, b=1.25)


def test_colbandit_small_candidate_sets(B, S, oracle_mod):
    # N <= K+M: no round runs and the answer is the exhaustive top-K; also N == K and N == 1
    for N, K, M in [(9, 4, 5), (10, 5, 5), (5, 5, 0), (1, 1, 0), (11, 5, 5)]:
        w = _custom(S, [33] * N, 2, 32, 128, "bf16", N)
        full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=K)
        res = B.colbandit_topk(w.Q, w.docs, w.offsets, K, 0.2, 0.01, M, 0)
        torch.cuda.synchronize()
        if N <= K + M:
            assert all(s["rounds"] == 0 and s["cells_elim"] == 0 and s["cells_rescore"] == 32 * N
                       for s in res["stats"])
            assert torch.equal(res["topk_ids"], full["topk_ids"])
            assert torch.equal(res["topk_scores"], full["topk_scores"])


@pytest.mark.parametrize("nq,T,d,N,K,M,Bsz,alpha,coarse", [
    (2, 1, 128, 300, 3, 2, 4, 0.2, False),          # one query token: a single round, then exact
    (2, 128, 128, 300, 5, 5, 16, 0.3, False),       # the largest T and B of this build
    (1, 32, 128, 1100, 1024, 0, 4, 0.2, False),     # the largest K
    (300, 16, 64, 500, 5, 5, 4, 0.2, False),        # many queries: several column groups, d=64
    (3, 40, 64, 400, 4, 3, 5, 0.5, True),           # int8 rounds with d=64 and B not dividing T
    (2, 100, 128, 300, 5, 5, 7, 1.0, True),         # int8 rounds, 7 tiles of query tokens
    (4, 32, 128, 6, 5, 5, 4, 0.2, True),            # N <= K + M: no round at all
    (2, 64, 128, 300, 5, 5, 1, 0.6, False),         # one token per round: the 64-round limit
    (3, 32, 96, 400, 5, 5, 4, 0.3, False),          # widths that only the gather kernels cover
    (2, 24, 32, 300, 3, 2, 4, 0.5, False),
])
def test_colbandit_corner_shapes(B, S, oracle_mod, nq, T, d, N, K, M, Bsz, alpha, coarse):
    rng = np.random.default_rng(N + T)
    w = _custom(S, rng.integers(1, 70, N).tolist(), nq, T, d, "bf16", 59)
    co = B.colbandit_quantize_i8(w.docs) if coarse else None
    if nq > 16:                                     # keep the oracle leg to a few queries
        full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=K, want_cells=True)
        res = B.colbandit_topk(w.Q, w.docs, w.offsets, K, alpha, 0.01, M, 5, B=Bsz, trace=True)
        torch.cuda.synchronize()
        for q in (0, 17, nq - 1):
            Hq = full["cells"][q].cpu().numpy().astype(np.float64)
            pi = B.colbandit_permutation(5, q, T)
            div, orc = _compare_rounds(oracle_mod, res["trace"], q, Hq, K, M, Bsz, alpha, 0.01, pi)
            assert res["stats"][q]["rounds"] == orc.rounds
            got = res["topk_ids"][q]
            assert torch.equal(res["topk_scores"][q], full["scores"][q][got])
            sfin = full["scores"][q].cpu().numpy()[orc.final_ids].astype(np.float64)
            order = orc.final_ids[np.lexsort((orc.final_ids, -sfin))][:K]
            np.testing.assert_array_equal(got.cpu().numpy(), order)
        return
    _run_colbandit_case(B, oracle_mod, w, K, M, Bsz, alpha, seed=5, coarse=co)


def test_explicit_permutation_and_determinism(B, S):
    w = S.config(1, device="cuda", scale=0.02, nq=4)
    pi = torch.tensor(np.stack([B.colbandit_permutation(77, q, w.T) for q in range(w.nq)]),
                      dtype=torch.int32, device="cuda")
    r1 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, 0.01, 5, 77, trace=True)
    r2 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, 0.01, 5, 123456, pi=pi, trace=True)
    r3 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, 0.01, 5, 77, trace=True)
    torch.cuda.synchronize()
    for other in (r2, r3):
        assert torch.equal(r1["topk_ids"], other["topk_ids"])
        assert torch.equal(r1["topk_scores"], other["topk_scores"])
        np.testing.assert_array_equal(r1["trace"].alive, other["trace"].alive)
    assert [s["survivors"] for s in r1["stats"]] == [s["survivors"] for s in r2["stats"]]


def test_async_call_without_stats(B, S):
    w = S.config(1, device="cuda", scale=0.02, nq=4)
    r1 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, 0.01, 5, 1)
    r2 = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, 0.01, 5, 1, want_stats=False)
    torch.cuda.synchronize()
    assert r2["stats"] is None
    assert torch.equal(r1["topk_ids"], r2["topk_ids"]) and torch.equal(r1["topk_scores"], r2["topk_scores"])


def test_both_calls_can_be_captured_in_a_graph_and_replayed(B, S):
    """Without statistics both entry points only enqueue kernels on the caller's stream (no
    allocation, no memset, no read-back), so a caller may capture them in a HIP graph.  Every
    replay, with eager work of the same library in between, must reproduce the eager result."""
    w = S.config(1, device="cuda", scale=0.06, nq=8)            # N=3000
    K = 5
    ws = B.new_workspace(w.nq, w.T, w.d, w.N, w.total_tokens, "cuda")
    d8, ds = B.colbandit_quantize_i8(w.docs)
    outs = [{"topk_ids": torch.empty((w.nq, K), dtype=torch.int64, device="cuda"),
             "topk_scores": torch.empty((w.nq, K), dtype=torch.float32, device="cuda")} for _ in range(3)]
    scores = torch.empty((w.nq, w.N), dtype=torch.float32, device="cuda")

    def run():
        B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=K, workspace=ws,
                                out={**outs[0], "scores": scores})
        B.colbandit_topk(w.Q, w.docs, w.offsets, K, 0.2, 0.01, 5, 3, workspace=ws, out=outs[1],
                         want_stats=False)
        B.colbandit_topk(w.Q, w.docs, w.offsets, K, 0.2, 0.01, 5, 3, workspace=ws, out=outs[2],
                         want_stats=False, docs_i8=d8, docs_scale=ds)

    run()
    torch.cuda.synchronize()
    ref = [(o["topk_ids"].clone(), o["topk_scores"].clone()) for o in outs]
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            run()
    torch.cuda.synchronize()
    for _ in range(3):
        for o in outs:
            o["topk_ids"].fill_(-7)
            o["topk_scores"].fill_(0.0)
        ws.fill_(0xAB)                                # the calls must not rely on workspace contents
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for o, (ids, sc) in zip(outs, ref):
            assert torch.equal(o["topk_ids"], ids) and torch.equal(o["topk_scores"], sc)
        other = B.colbandit_topk(w.Q, w.docs, w.offsets, 3, 0.5, 0.01, 2, 9, workspace=ws)   # eager, other knobs
        torch.cuda.synchronize()
        assert other["stats"][0]["rounds"] >= 1


def test_validate_offsets(B, S):
    w = S.config(0, device="cuda")
    assert B.colbandit_validate_offsets(w.offsets, w.total_tokens) == 0
    bad = w.offsets.clone(); bad[10] = bad[9]                   # an empty document
    assert B.colbandit_validate_offsets(bad, w.total_tokens) == -8
    assert B.colbandit_validate_offsets(w.offsets, w.total_tokens - 1) == -8
    # a bad table must not fault: rows are clamped, results are merely meaningless
    B.colbandit_full_maxsim(w.Q, w.docs, bad, K=0)
    torch.cuda.synchronize()


# ------------------------------------------------------------------ int8 coarse elimination pass
def _host_values(x):
    return x.float().cpu().numpy()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows,d,nseg,permille", [(3001, 128, 1, 999), (64, 128, 4, 999), (32 * 9, 64, 9, 999),
                                                   (1, 128, 1, 999), (500, 128, 1, 1000), (500, 128, 5, 500),
                                                   (1200, 128, 2, 999), (1026, 100, 2, 900), (1001, 100, 1, 999)])
def test_quantize_i8_codes_and_scales_match_oracle(B, oracle_mod, dtype, rows, d, nseg, permille):
    """Percentile clip and codes are integer results: exact equality with the oracle, which
    takes the deciding arithmetic in single precision as well."""
    g = torch.Generator(device="cpu"); g.manual_seed(rows * 7 + d + nseg)
    x = torch.randn((rows, d), generator=g) * 0.09
    x[0, 0] = 3.0                                   # an outlier far above the clip
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()
    codes, scales = B.colbandit_quantize_i8(x, n_segments=nseg, permille=permille)
    torch.cuda.synchronize()
    xs = _host_values(x).reshape(nseg, -1)
    for sidx in range(nseg):
        clip = oracle_mod.abs_percentile(xs[sidx], permille)
        assert scales[sidx].item() == np.float32(clip) / np.float32(127.0)
        want = oracle_mod.quantize_i8(xs[sidx], clip)
        np.testing.assert_array_equal(codes.cpu().numpy().reshape(nseg, -1)[sidx], want)
    if permille == 999 and rows * d // nseg >= 2000:
        assert codes.abs().max().item() == 127       # the outlier saturates
    z = torch.zeros((4, d), dtype=x.dtype, device="cuda")
    cz, sz = B.colbandit_quantize_i8(z)
    assert int(cz.abs().max()) == 0 and float(sz[0]) == 0.0


@pytest.mark.parametrize("rows,d", [(1 << 20, 128), (1000000, 128), (1 << 20, 64), (1 << 20, 96)])
def test_one_counting_pass_finds_the_clip_of_columns_of_unequal_scale(B, rows, d):
    """The sampled bound of a long segment serves columns whose scales differ a hundredfold, also where
    the distance of the samples shares factors with the rows: the clip is known after the counting
    pass (the state at the head of the workspace says so) and is the exact order statistic."""
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + d)
    for scale in (torch.logspace(0, -2, d), torch.logspace(-2, 0, d)):
        x = (torch.randn((rows, d), generator=g, device="cuda") * scale.cuda()).to(torch.bfloat16)
        codes = torch.empty(x.shape, dtype=torch.int8, device="cuda")
        scales = torch.empty(1, device="cuda")
        ws = torch.zeros(B.lib().colbandit_quantize_workspace_bytes(1), dtype=torch.uint8, device="cuda")
        rc = B.lib().colbandit_quantize_i8(x.data_ptr(), 1, 1, rows, d, 999, codes.data_ptr(), scales.data_ptr(),
                                           ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert rc == 0
        assert ws[:24].view(torch.int32)[5].item() == 1           # rank (two words), prefix, mask, bound, done
        drop = x.numel() - (x.numel() * 999 + 999) // 1000
        clip = x.abs().reshape(-1).topk(drop + 1).values[drop].float().cpu().numpy()
        assert scales.cpu().numpy()[0] == clip / np.float32(127)


@pytest.mark.parametrize("kind,permille", [("normal", 999), ("normal", 1000), ("normal", 986), ("normal", 900),
                                           ("constant", 999), ("rare", 999), ("wide", 999), ("sorted", 999)])
def test_quantize_long_bf16_segment_by_its_tail(B, kind, permille):
    """Segments of 2^26 values and more count only what lies above a sampled bound; a bound that the
    values defeat (all equal, nearly all zero, a tail wider than the bins, large values that the sample
    misses) falls back on the full passes.  The clip is the exact order statistic either way."""
    g = torch.Generator(device="cuda")
    g.manual_seed(permille)
    rows = (1 << 19) + 3
    x = torch.randn((rows, 128), generator=g, device="cuda")
    if kind == "constant":
        x = torch.full_like(x, -0.75)
    elif kind == "rare":
        x = torch.where(torch.rand(x.shape, generator=g, device="cuda") < 0.0005, x, torch.zeros_like(x))
    elif kind == "wide":
        x = torch.exp(20 * x)
    elif kind == "sorted":
        x = x.abs().reshape(-1).sort().values.reshape(x.shape)
    x = x.to(torch.bfloat16)
    codes, scale = B.colbandit_quantize_i8(x, permille=permille)
    n = x.numel()
    counts = torch.bincount((x.view(torch.int16).reshape(-1) & 0x7fff).to(torch.int32), minlength=32768)
    rank = (n * permille + 999) // 1000
    key = int(torch.searchsorted(torch.cumsum(counts, 0), torch.tensor([rank], device="cuda"))[0])
    clip = torch.tensor([key], dtype=torch.int16, device="cuda").view(torch.bfloat16).float()
    clip = clip.cpu().numpy()[0]                       # single-precision divisions on the host
    assert scale.cpu().numpy()[0] == clip / np.float32(127)
    inv = float(np.float32(127) / clip) if clip > 0 else 0.0
    for lo in range(0, rows, 1 << 18):
        want = torch.clamp(torch.round(x[lo:lo + (1 << 18)].float() * inv), -127, 127).to(torch.int8)
        assert torch.equal(codes[lo:lo + (1 << 18)], want)


@pytest.mark.parametrize("kind,done", [("normal", 2), ("edge", 1), ("biased", 1), ("constant", 2)])
def test_quantize_guesses_the_clip_of_a_very_long_segment(B, kind, done):
    """2^29 values and more: a sixteenth of the runs of 4 KB names the clip and one pass codes and counts.  The state
    at the head of the workspace says whether that pass was enough (2) or the clip had to be found first (1): a
    rank at the edge of equal values is not guessed, runs unlike the rest give a wrong guess.  Codes are those
    of the exact clip either way."""
    g = torch.Generator(device="cuda").manual_seed(7)
    rows, d = (1 << 22) + 37, 128
    # (times 0.86, and times 0.8 again, the clip lies well inside the values that round to it)
    x = (torch.randn((rows, d), generator=g, device="cuda") * 0.86).to(torch.bfloat16)
    n = x.numel()
    drop = n - (n * 999 + 999) // 1000                  # values above the clip
    flat = x.view(-1)
    if kind == "constant":
        x.fill_(-0.75)
    elif kind == "edge":
        x.clamp_(-1, 1)
        at = torch.randint(0, n, (drop + 1 + n // 10000,), generator=g, device="cuda").unique()
        flat[at[torch.randperm(at.numel(), generator=g, device="cuda")[:drop + 1]]] = 2.0
    elif kind == "biased":
        i = np.arange(n // 8 // (256 * 16), dtype=np.uint32)
        h = i * np.uint32(0x9E3779B1)
        h = (h ^ (h >> np.uint32(15))) * np.uint32(0x85EBCA77)
        h ^= h >> np.uint32(13)
        run = i.astype(np.int64) * 16 + ((h.astype(np.uint64) * np.uint64(16)) >> np.uint64(32)).astype(np.int64)
        flat[:n // 2048 * 2048].view(-1, 2048)[torch.from_numpy(run).cuda()] *= 0.8
    codes = torch.empty(x.shape, dtype=torch.int8, device="cuda")
    scales = torch.empty(1, device="cuda")
    ws = torch.zeros(B.lib().colbandit_quantize_workspace_bytes(1), dtype=torch.uint8, device="cuda")
    rc = B.lib().colbandit_quantize_i8(x.data_ptr(), 1, 1, rows, d, 999, codes.data_ptr(), scales.data_ptr(),
                                       ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and ws[:24].view(torch.int32)[5].item() == done
    counts = sum(torch.bincount((p.view(torch.int16) & 0x7fff).to(torch.int32), minlength=32768) for p in flat.split(1 << 27))
    key = int(torch.searchsorted(torch.cumsum(counts, 0), torch.tensor([n - drop], device="cuda"))[0])
    clip = torch.tensor([key], dtype=torch.int16).view(torch.bfloat16).float().numpy()[0]
    assert scales.cpu().numpy()[0] == clip / np.float32(127)
    inv = float(np.float32(127) / clip)
    for lo in range(0, rows, 1 << 19):
        want = torch.clamp(torch.round(x[lo:lo + (1 << 19)].float() * inv), -127, 127).to(torch.int8)
        assert torch.equal(codes[lo:lo + (1 << 19)], want)


def _sampled(n, step):
    """The places of n samples, one of each run of `step` (the library's sample_piece)."""
    i = np.arange(n, dtype=np.uint32)
    h = i * np.uint32(0x9E3779B1)
    h = (h ^ (h >> np.uint32(15))) * np.uint32(0x85EBCA77)
    h ^= h >> np.uint32(13)
    at = i.astype(np.int64) * step + ((h.astype(np.uint64) * np.uint64(step)) >> np.uint64(32)).astype(np.int64)
    return torch.from_numpy(at).cuda()


@pytest.mark.parametrize("kind,permille,work", [
    ("alike", 999, {"k_quant_codes<true, true, true>": [1], "k_quant_tail": [0], "k_quant_hist": [0, 0], "k_quant_codes<true, true, false>": [0]}),
    ("clusters", 999, {"k_quant_codes<true, true, true>": [0], "k_quant_tail": [1], "k_quant_hist": [0, 0], "k_quant_codes<true, true, false>": [1]}),
    ("high", 999, {"k_quant_codes<true, true, true>": [1], "k_quant_tail": [0], "k_quant_hist": [1, 1], "k_quant_codes<true, true, false>": [1]}),
    ("alike", 1000, {"k_quant_codes<true, true, true>": [], "k_quant_tail": [1], "k_quant_hist": [0, 0], "k_quant_codes<true, true, false>": [1]})])
def test_passes_that_code_a_very_long_segment(B, kind, permille, work):
    """Which passes read the segment (more than 60 us: a pass over 1.07 GB takes 150 at least, one that returns at
    once 10 at most).  clusters: the values of the tail lie in an eighth of the runs of 4 KB, so that a sixteenth says
    less of them than of independent ones (one deviation is 2.1 % of the tail, not 0.55; the values that round to the
    clip are 6 %), and no guess is made where one from independent values would be.  high: the sampled pieces
    and the runs of the sixteenth are twice as large as the rest, the bound is too high for the whole segment, and
    no second count is made with it.  permille 1000: one value decides, which no sixteenth can name."""
    from torch.profiler import ProfilerActivity, profile
    g = torch.Generator(device="cuda").manual_seed(13)
    rows, d = 1 << 22, 128
    n = rows * d
    # (times 0.8594 the clip lies in the middle of the values that round to it, 3 % of the tail from either edge)
    x = torch.randn((rows, d), generator=g, device="cuda") * 0.8594
    if kind == "clusters":                              # (the clip of the whole stays in the middle of its values)
        hot = torch.rand(n // 2048, generator=g, device="cuda") < 0.125
        x.view(-1, 2048).mul_(torch.where(hot, 0.38876 / 0.8594, 0.1)[:, None])
    x = x.to(torch.bfloat16)
    runs = x.view(-1, 2048)
    if kind == "high":
        runs[_sampled(n // 8 // 4096, 16)] *= 2
        pieces = _sampled(16384, n // 8 // 16384)
        pieces = pieces[~torch.isin(pieces // 256, _sampled(n // 8 // 4096, 16))]
        x.view(-1, 8)[pieces] *= 2
    B.colbandit_quantize_i8(x[:1024])
    for _ in range(5):
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            codes, scales = B.colbandit_quantize_i8(x, permille=permille)
            torch.cuda.synchronize()
        ran = sorted((e.time_range.start, e.key, e.time_range.elapsed_us()) for e in p.events() if "k_quant" in e.key)
        if ran:
            break
    got = {k: [int(us > 60) for _, name, us in ran if k in name] for k in work}
    got["k_quant_tail"] = [int(us > 60) for _, name, us in ran if "k_quant_tail(" in name][len(work["k_quant_codes<true, true, true>"]):]
    assert got == work, [(name, us) for _, name, us in ran]
    counts = sum(torch.bincount((p.view(torch.int16) & 0x7fff).to(torch.int32), minlength=32768) for p in x.view(-1).split(1 << 27))
    rank = (n * permille + 999) // 1000
    key = int(torch.searchsorted(torch.cumsum(counts, 0), torch.tensor([rank], device="cuda"))[0])
    clip = torch.tensor([key], dtype=torch.int16).view(torch.bfloat16).float().numpy()[0]
    assert scales.cpu().numpy()[0] == clip / np.float32(127)
    inv = float(np.float32(127) / clip)
    for lo in range(0, rows, 1 << 19):
        want = torch.clamp(torch.round(x[lo:lo + (1 << 19)].float() * inv), -127, 127).to(torch.int8)
        assert torch.equal(codes[lo:lo + (1 << 19)], want)


@pytest.mark.parametrize("nq,T,d", [(1, 32, 128), (5, 32, 128), (20, 24, 128), (3, 40, 128), (2, 100, 128),
                                    (4, 32, 64), (70, 16, 64)])
def test_coarse_maxsim_cells_are_the_integer_maxima(B, S, oracle_mod, nq, T, d):
    """Cells from int8 codes: the integer dot products and their maxima are exact, so the
    decoded cell must equal float(int) * (sq * sd) bit for bit."""
    lengths = [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 100, 255, 257, 1030] + \
        np.random.default_rng(d + T).integers(1, 200, 150).tolist()
    w = _custom(S, lengths, nq, T, d, "bf16", 11 + nq)
    d8, ds = B.colbandit_quantize_i8(w.docs)
    cm = B.colbandit_coarse_maxsim(w.Q, d8, ds, w.offsets, want_cells=True)
    torch.cuda.synchronize()
    q8 = cm["q_codes"].cpu().numpy()
    qs = cm["q_scales"].cpu().numpy()
    Qh = w.host_queries()
    off = w.offsets.cpu().numpy()
    D8 = d8.cpu().numpy()
    sd = np.float32(ds.cpu().numpy()[0])
    cells = cm["cells"].cpu().numpy()
    for q in range(nq):
        # the call's own query codes follow the same scheme
        clip = oracle_mod.abs_percentile(Qh[q], 999)
        assert qs[q] == np.float32(clip) / np.float32(127.0)
        np.testing.assert_array_equal(q8[q], oracle_mod.quantize_i8(Qh[q], clip))
        if q < 6:
            _, Hint = oracle_mod.maxsim_cells_i8(q8[q], qs[q], D8, sd, off)
            want = Hint.astype(np.float32) * (np.float32(qs[q]) * sd)
            np.testing.assert_array_equal(cells[q], want)
    # row sums in the kernels' fixed order vs a plain sum
    np.testing.assert_allclose(cm["scores"].cpu().numpy(), cells.sum(axis=2), rtol=1e-5, atol=1e-5)


def test_every_position_of_a_document_end_inside_a_block(B, S, oracle_mod):
    """The wide dense kernels fold a block in which a document ends by code specialised for the
    row at which it ends; here every such row 1..15 occurs (a document of b tokens from a block
    start, then one of 32 - b tokens that ends with a block), and two and three ends in one
    block (which take the general fold).  Exhaustive cells (bf16, 20 queries: eight column tiles
    per wavefront), integer cells of the int8 codes, and the round-1 statistics of Col-Bandit
    over 72 queries (eight tiles per wavefront in the reveal pass) against the oracle."""
    lengths = []
    for b in range(1, 16):
        lengths += [b, 32 - b]
    lengths += [3, 4, 9, 5, 5, 6, 16, 1, 1, 1, 13] + list(range(1, 40))
    nq, T, d = 20, 32, 128
    lengths = _past_small(lengths, nq, d, "bf16")
    w = _custom(S, lengths, nq, T, d, "bf16", 77)
    H, Sor = _oracle_scores(oracle_mod, w)
    ran = []
    assert "k_dense<cb::bf16_tag, 128, 8, 2, false, 0, false>" in _kernels(
        lambda: B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=3, want_cells=True), ran)
    r = ran[0]
    np.testing.assert_allclose(r["cells"].cpu().numpy(), H, rtol=TOL["bf16"], atol=1e-5)
    np.testing.assert_allclose(r["scores"].cpu().numpy(), Sor, rtol=TOL["bf16"], atol=1e-4)
    # int8 codes: exact integer maxima
    d8, ds = B.colbandit_quantize_i8(w.docs)
    cm = B.colbandit_coarse_maxsim(w.Q, d8, ds, w.offsets, want_cells=True)
    torch.cuda.synchronize()
    q8, qs = cm["q_codes"].cpu().numpy(), cm["q_scales"].cpu().numpy()
    off, D8 = w.offsets.cpu().numpy(), d8.cpu().numpy()
    sd = np.float32(ds.cpu().numpy()[0])
    for q in (0, 7, 19):
        _, Hint = oracle_mod.maxsim_cells_i8(q8[q], qs[q], D8, sd, off)
        np.testing.assert_array_equal(cm["cells"][q].cpu().numpy(),
                                      Hint.astype(np.float32) * (np.float32(qs[q]) * sd))
    # the reveal pass with eight tiles per wavefront: 72 queries x 4 revealed tokens
    w2 = _custom(S, lengths, 72, T, d, "bf16", 78)
    full = B.colbandit_full_maxsim(w2.Q, w2.docs, w2.offsets, K=0, want_cells=True)
    e8, es = B.colbandit_quantize_i8(w2.docs)
    assert "k_dense<cb::bf16_tag, 128, 8, 1, true" in _kernels(
        lambda: B.colbandit_topk(w2.Q, w2.docs, w2.offsets, 3, 1.0, 0.01, 2, 9, B=4, trace=True), ran)
    assert "k_dense<cb::i8_tag, 128, 8, 1, true" in _kernels(
        lambda: B.colbandit_topk(w2.Q, w2.docs, w2.offsets, 3, 1.0, 0.01, 2, 9, B=4, trace=True, docs_i8=e8,
                                 docs_scale=es), ran)
    res, res8 = ran[1:]
    cm2 = B.colbandit_coarse_maxsim(w2.Q, e8, es, w2.offsets, want_cells=True)
    torch.cuda.synchronize()
    for q in (0, 35, 71):
        Hq = full["cells"][q].cpu().numpy().astype(np.float64)
        Hc = cm2["cells"][q].cpu().numpy().astype(np.float64)
        pi = B.colbandit_permutation(9, q, T)
        div, orc = _compare_rounds(oracle_mod, res["trace"], q, Hq, 3, 2, 4, 1.0, 0.01, pi)
        assert res["stats"][q]["rounds"] == orc.rounds
        div, orc = _compare_rounds(oracle_mod, res8["trace"], q, Hc, 3, 2, 4, 1.0, 0.01, pi, Hexact=Hq)
        assert res8["stats"][q]["rounds"] == orc.rounds


@pytest.mark.parametrize("alpha,K,M,Bsz", [(0.2, 5, 5, 4), (1.0, 5, 5, 4), (0.5, 10, 5, 3), (0.2, 5, 0, 16)])
def test_colbandit_on_int8_codes_rounds_match_oracle(B, S, oracle_mod, alpha, K, M, Bsz):
    """Rounds decided on coarse cells, survivors rescored exactly (implementation appendix):
    every bound, threshold and survivor against the oracle's coarse-elimination mode, and the
    returned scores carry the exhaustive path's bits."""
    w = S.config(1, device="cuda", scale=0.04, nq=6)            # N=2000, planted docs
    d8, ds = B.colbandit_quantize_i8(w.docs)
    _run_colbandit_case(B, oracle_mod, w, K, M, Bsz, alpha, coarse=(d8, ds))
    w = S.config(3, device="cuda", scale=0.005, nq=4)           # 100 pages x 1030 tokens, T=24
    d8, ds = B.colbandit_quantize_i8(w.docs)
    _run_colbandit_case(B, oracle_mod, w, K, M, Bsz, alpha, coarse=(d8, ds))


def test_colbandit_on_int8_codes_all_reveal_paths_agree(B, S, oracle_mod):
    rng = np.random.default_rng(3)
    w = _custom(S, rng.integers(1, 120, 2500).tolist(), 5, 32, 128, "bf16", 23)
    d8, ds = B.colbandit_quantize_i8(w.docs)
    kw = dict(docs_i8=d8, docs_scale=ds, trace=True)
    base = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.5, 0.01, 5, 3, **kw)
    for extra in (dict(force_gather=True), dict(no_cell_cache=True), dict(later_rounds=1),
                  dict(later_rounds=2), dict(later_rounds=1, no_cell_cache=True)):
        other = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.5, 0.01, 5, 3, **kw, **extra)
        torch.cuda.synchronize()
        _same_run(base, other)
    # fp32 embeddings with int8 codes: the rounds use the codes, the rescore the fp32 gather
    w32 = _custom(S, rng.integers(1, 60, 600).tolist(), 2, 32, 128, "f32", 29)
    d8, ds = B.colbandit_quantize_i8(w32.docs)
    _run_colbandit_case(B, oracle_mod, w32, 5, 5, 4, 0.3, coarse=(d8, ds))


# ------------------------------------------------------------------ non-adaptive baselines
def _clustered_queries(w, S, n_dir, noise, seed):
    """Replaces the workload's queries by tokens scattered around n_dir directions with random
    norms, so that a sweep of the cosine threshold gives anything from one cluster to T."""
    g = torch.Generator(device="cpu"); g.manual_seed(seed)
    nq, T, d = w.Q.shape
    base = torch.randn((nq, n_dir, d), generator=g)
    base = base / base.norm(dim=2, keepdim=True)
    pick = torch.randint(0, n_dir, (nq, T), generator=g)
    Q = torch.gather(base, 1, pick[..., None].expand(nq, T, d)) + noise * torch.randn((nq, T, d), generator=g) / d ** 0.5
    Q = Q * (0.5 + 1.5 * torch.rand((nq, T, 1), generator=g))
    w.Q = Q.to(w.Q.dtype).cuda()
    return w


@pytest.mark.parametrize("dtype,nq,T,d,m", [("bf16", 3, 32, 128, 4), ("bf16", 20, 32, 128, 13),
                                            ("bf16", 2, 64, 128, 64), ("bf16", 5, 7, 64, 1),
                                            ("bf16", 4, 30, 128, 30), ("f32", 2, 32, 128, 8),
                                            ("f32", 3, 24, 64, 5), ("bf16", 3, 32, 96, 5),
                                            ("f32", 2, 24, 32, 7)])
def test_doc_uniform_masks_scores_and_topk_match_oracle(B, S, oracle_mod, dtype, nq, T, d, m):
    """Doc-Uniform (appendix "Compared Methods"): the per-document token subsets are the oracle's
    bit for bit (same counter-based generator, implemented on each side), the partial row sums
    agree within the score tolerance, the top-K follows them."""
    rng = np.random.default_rng(T * 100 + m)
    lengths = [1, 16, 17, 63, 65, 300, 1] + rng.integers(1, 120, 260).tolist()
    w = _custom(S, lengths, nq, T, d, dtype, 41)
    seed, K = 1234567, 6
    r = B.colbandit_doc_uniform(w.Q, w.docs, w.offsets, K, m, seed=seed, want_masks=True)
    torch.cuda.synchronize()
    H, _ = _oracle_scores(oracle_mod, w)
    masks = r["masks"].cpu().numpy().view(np.uint64)
    got = r["scores"].cpu().numpy()
    tol = TOL[dtype]
    for q in range(nq):
        mo, So, _, _ = oracle_mod.doc_uniform_from_H(H[q], m, seed, q, K)
        np.testing.assert_array_equal(masks[q], mo)
        np.testing.assert_allclose(got[q], So, rtol=tol, atol=tol)
        _check_topk(r["topk_ids"][q].cpu().numpy(), r["topk_scores"][q].cpu().numpy(), So, K, tol)
    if m == T:      # every cell revealed: the exhaustive scores (other summation order)
        full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=0)
        torch.cuda.synchronize()
        np.testing.assert_allclose(got, full["scores"].cpu().numpy(), rtol=1e-5, atol=1e-5)
    # top-K only (scores kept in the workspace) gives the same ranking
    r2 = B.colbandit_doc_uniform(w.Q, w.docs, w.offsets, K, m, seed=seed, want_scores=False)
    torch.cuda.synchronize()
    assert torch.equal(r2["topk_ids"], r["topk_ids"]) and torch.equal(r2["topk_scores"], r["topk_scores"])


@pytest.mark.parametrize("dtype,nq,T,d,tau", [("bf16", 3, 32, 128, 0.7), ("bf16", 40, 32, 128, 0.9),
                                              ("bf16", 6, 32, 128, 0.4), ("bf16", 2, 64, 128, 0.8),
                                              ("bf16", 5, 7, 64, 0.6), ("bf16", 4, 30, 128, 1.0),
                                              ("bf16", 1, 1, 128, 0.5), ("f32", 2, 32, 128, 0.7),
                                              ("f32", 3, 24, 64, 0.5), ("bf16", 3, 32, 96, 0.7),
                                              ("f32", 2, 24, 32, 0.6)])
def test_ball_carving_clusters_centroids_scores_match_oracle(B, S, oracle_mod, dtype, nq, T, d, tau):
    """Ball-carving (appendix "Compared Methods"): cluster labels and cluster counts are exact
    (the membership test is taken in the same double-precision form on both sides), the
    centroids are the oracle's bit for bit, scores and top-K agree within the score tolerance."""
    rng = np.random.default_rng(T * 10 + nq)
    lengths = [1, 16, 17, 63, 65, 300, 1] + rng.integers(1, 120, 260).tolist()
    w = _clustered_queries(_custom(S, lengths, nq, T, d, dtype, 43), S, 4, 0.6, 5)
    K = 6
    r = B.colbandit_ball_carving(w.Q, w.docs, w.offsets, K, tau)
    torch.cuda.synchronize()
    E, off = w.host_docs()
    Qh = w.host_queries()
    tol = TOL[dtype]
    ks = []
    for q in range(nq):
        k, labels, C, So, _, _ = oracle_mod.ball_carving(Qh[q], E, off, tau, K, round_bf16=(dtype == "bf16"))
        ks.append(k)
        assert int(r["n_clusters"][q]) == k
        np.testing.assert_array_equal(r["labels"][q].cpu().numpy(), labels)
        np.testing.assert_array_equal(r["centroids"][q].float().cpu().numpy(), C)
        scale = max(1.0, float(np.abs(So).max()))
        np.testing.assert_allclose(r["scores"][q].cpu().numpy(), So, rtol=tol, atol=tol * scale)
        _check_topk(r["topk_ids"][q].cpu().numpy(), r["topk_scores"][q].cpu().numpy(), So, K, tol)
    if tau == 1.0:
        assert ks == [T] * nq
        full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=0)
        torch.cuda.synchronize()
        np.testing.assert_allclose(r["scores"].cpu().numpy(), full["scores"].cpu().numpy(),
                                   rtol=1e-4, atol=1e-4)
    if T >= 24 and tau <= 0.7:
        assert min(ks) < T                               # the sweep point does compress


def test_ball_carving_identical_tokens_collapse_to_one_centroid(B, S, oracle_mod):
    w = _custom(S, np.random.default_rng(3).integers(1, 90, 150).tolist(), 2, 32, 128, "bf16", 47)
    w.Q = (w.Q[:, :1, :].float() * torch.tensor([1.0, 2.0, 0.5, 4.0] * 8, device="cuda")[None, :, None]) \
        .to(torch.bfloat16).contiguous()
    r = B.colbandit_ball_carving(w.Q, w.docs, w.offsets, 3, 1.0)
    torch.cuda.synchronize()
    assert r["n_clusters"].tolist() == [1, 1] and int(r["labels"].abs().sum()) == 0
    E, off = w.host_docs()
    for q in range(2):
        k, _, C, So, _, _ = oracle_mod.ball_carving(w.host_queries()[q], E, off, 1.0, 3, round_bf16=True)
        assert k == 1
        np.testing.assert_array_equal(r["centroids"][q].float().cpu().numpy(), C)
        np.testing.assert_allclose(r["scores"][q].cpu().numpy(), So, rtol=TOL["bf16"], atol=1e-3)


def _rounds_of_sampled_queries(B, oracle_mod, w, res, qs, K, alpha, scores_of, coarse=None):
    """Full-size protocol for a traced batch call `res` (trace_queries=qs): for each sampled
    query the GPU's own cells of that query (one exhaustive single-query call with the cell
    output) go through the oracle and every round is compared (_compare_rounds); then rounds,
    counters, final set and the returned top-K.  scores_of(q) -> the exhaustive path's scores of
    query q as a host array.  coarse = (docs_i8, docs_scale) when the rounds ran on int8 codes.
    Returns the number of queries that needed a re-entry at a band document."""
    tr, T = res["trace"], w.T
    diverged = 0
    for j, q in enumerate(qs):
        Qq = w.Q[q:q + 1].contiguous()
        one = B.colbandit_full_maxsim(Qq, w.docs, w.offsets, K=0, want_cells=True)
        torch.cuda.synchronize()
        Sq = scores_of(q)
        np.testing.assert_array_equal(one["scores"][0].cpu().numpy(), Sq)   # batch position does not matter
        Hq = one["cells"][0].cpu().numpy().astype(np.float64)
        del one
        Hc = None
        if coarse is not None:
            cm = B.colbandit_coarse_maxsim(Qq, coarse[0], coarse[1], w.offsets, want_cells=True)
            torch.cuda.synchronize()
            Hc = cm["cells"][0].cpu().numpy().astype(np.float64)
            del cm
        pi = B.colbandit_permutation(w.seed, q, T)
        np.testing.assert_array_equal(pi, oracle_mod.permutation(w.seed, q, T))
        if Hc is None:
            div, orc = _compare_rounds(oracle_mod, tr, j, Hq, K, w.M, w.B, alpha, w.delta, pi)
        else:
            div, orc = _compare_rounds(oracle_mod, tr, j, Hc, K, w.M, w.B, alpha, w.delta, pi, Hexact=Hq)
        st = res["stats"][q]
        assert st["survivors"] == [int(x) for x in tr.count[: st["rounds"] + 1, j]]
        assert st["rounds"] == orc.rounds and st["cells_rescore"] == orc.cells_rescore
        if div == 0:
            assert (st["cells_elim"], st["cells_unique"]) == (orc.cells_elim, orc.cells_unique)
        diverged += div > 0
        kk = min(K, len(orc.final_ids))
        order = orc.final_ids[np.lexsort((orc.final_ids, -Sq[orc.final_ids].astype(np.float64)))][:kk]
        np.testing.assert_array_equal(res["topk_ids"][q].cpu().numpy()[:kk], order)
        np.testing.assert_array_equal(res["topk_scores"][q].cpu().numpy()[:kk], Sq[order])
        # the rescore is the exact row sum: fp32 fixed-order sum vs the double sum of the same cells
        np.testing.assert_allclose(Sq[order], Hq[order].sum(axis=1), rtol=1e-5)
        print(f"  query {q}: {orc.rounds} rounds, survivors {st['survivors']}, re-entries {div}", flush=True)
    return diverged


# ------------------------------------------------------------------ full size, bench launch configuration
@pytest.fixture(scope="module")
def big(B, S):
    """The benchmark's workload and call pattern: N=500,000 documents, 128 queries, preallocated
    workspace and outputs, K=5, alpha_ef=0.2."""
    print("generating the full-size corpus ...", flush=True)
    w = S.config(2, device="cuda")
    ws = B.new_workspace(w.nq, w.T, w.d, w.N, w.total_tokens, "cuda")
    K = 5
    out = {"topk_ids": torch.empty((w.nq, K), dtype=torch.int64, device="cuda"),
           "topk_scores": torch.empty((w.nq, K), dtype=torch.float32, device="cuda"),
           "scores": torch.empty((w.nq, w.N), dtype=torch.float32, device="cuda")}
    print("full-size Full-MaxSim ...", flush=True)
    full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=K, workspace=ws, out=out)
    torch.cuda.synchronize()
    return w, ws, full, K


def test_full_size_scores_on_sampled_documents(B, oracle_mod, big):
    w, ws, full, K = big
    assert (w.N, w.nq, w.T, w.d, w.dtype) == (500000, 128, 32, 128, "bf16")
    rng = np.random.default_rng(2026)
    qs = [0, 31, 77, 127]
    Qh = w.host_queries(qs)
    ids_gpu = full["topk_ids"].cpu().numpy()
    for j, q in enumerate(qs):
        # random documents, the first and last of the corpus, and the GPU's winners
        docs = np.unique(np.concatenate([rng.integers(0, w.N, 40), [0, w.N - 1], ids_gpu[q]]))
        E, off = w.host_docs(docs.tolist())
        H = oracle_mod.maxsim_cells(Qh[j], E, off)
        want = H.sum(axis=1)
        got = full["scores"][q][torch.as_tensor(docs, device="cuda")].cpu().numpy()
        np.testing.assert_allclose(got, want, rtol=TOL["bf16"], atol=0)
    # the top-K is the ordered head of the GPU's own score rows
    for q in qs + [5, 64]:
        sc = full["scores"][q].cpu().numpy()
        order = np.lexsort((np.arange(w.N), -sc))[:K]
        np.testing.assert_array_equal(ids_gpu[q], order)
        np.testing.assert_array_equal(full["topk_scores"][q].cpu().numpy(), sc[order])


def test_full_size_colbandit_rounds_and_survivor_scores(B, oracle_mod, big):
    w, ws, full, K = big
    qs = [3, 90]
    alpha, delta, M, Bsz = 0.2, w.delta, w.M, w.B
    out = {"topk_ids": torch.empty((w.nq, K), dtype=torch.int64, device="cuda"),
           "topk_scores": torch.empty((w.nq, K), dtype=torch.float32, device="cuda")}
    print("full-size Col-Bandit with trace ...", flush=True)
    res = B.colbandit_topk(w.Q, w.docs, w.offsets, K, alpha, delta, M, w.seed, workspace=ws, out=out,
                           trace=True, trace_queries=qs)
    plain = B.colbandit_topk(w.Q, w.docs, w.offsets, K, alpha, delta, M, w.seed, workspace=ws,
                             want_stats=False)
    torch.cuda.synchronize()
    # tracing changes nothing
    assert torch.equal(res["topk_ids"], plain["topk_ids"])
    assert torch.equal(res["topk_scores"], plain["topk_scores"])
    # every query: survivor scores are the exhaustive path's bits; accounting identities
    ids = res["topk_ids"]
    assert bool((ids >= 0).all())
    assert torch.equal(res["topk_scores"], torch.gather(full["scores"], 1, ids))
    T = w.T
    for q, st in enumerate(res["stats"]):
        surv = st["survivors"]
        assert surv[0] == w.N and all(surv[r + 1] <= surv[r] for r in range(st["rounds"]))
        cells = sum((min((r + 1) * Bsz, T) - r * Bsz) * surv[r] for r in range(st["rounds"]))
        assert st["cells_elim"] == cells and st["cells_rescore"] == T * surv[st["rounds"]]
    # two queries: every round against the oracle, fed the GPU's own cells of these queries
    print("full-size cells of two queries ...", flush=True)
    scores_of = lambda q: full["scores"][q].cpu().numpy()
    _rounds_of_sampled_queries(B, oracle_mod, w, res, qs, K, alpha, scores_of)


def test_full_size_colbandit_rounds_at_k10_and_on_int8_codes(B, oracle_mod, big):
    """The large text configuration's second setting (K = 10) and its int8 coarse pass, in the
    benchmark's launch configuration: every round of sampled queries against the oracle."""
    w, ws, full, _ = big
    scores_of = lambda q: full["scores"][q].cpu().numpy()
    qs = [17, 101]
    print("full-size Col-Bandit, K = 10, with trace ...", flush=True)
    res = B.colbandit_topk(w.Q, w.docs, w.offsets, 10, 0.2, w.delta, w.M, w.seed, workspace=ws,
                           trace=True, trace_queries=qs)
    torch.cuda.synchronize()
    assert torch.equal(res["topk_scores"], torch.gather(full["scores"], 1, res["topk_ids"]))
    _rounds_of_sampled_queries(B, oracle_mod, w, res, qs, 10, 0.2, scores_of)
    del res
    print("full-size Col-Bandit on int8 codes, K = 5, with trace ...", flush=True)
    d8, ds = B.colbandit_quantize_i8(w.docs)
    qs = [64]
    res = B.colbandit_topk(w.Q, w.docs, w.offsets, 5, 0.2, w.delta, w.M, w.seed, workspace=ws,
                           trace=True, trace_queries=qs, docs_i8=d8, docs_scale=ds)
    torch.cuda.synchronize()
    assert torch.equal(res["topk_scores"], torch.gather(full["scores"], 1, res["topk_ids"]))
    _rounds_of_sampled_queries(B, oracle_mod, w, res, qs, 5, 0.2, scores_of, coarse=(d8, ds))


def test_full_size_baselines_on_sampled_documents(B, oracle_mod, big):
    """Doc-Uniform and Ball-carving at the benchmark's size: subsets, clusters and centroids exact
    for sampled queries; scores of sampled documents against the oracle."""
    w, ws, full, K = big
    rng = np.random.default_rng(77)
    qs = [0, 64, 127]
    docs = np.unique(np.concatenate([rng.integers(0, w.N, 30), [0, w.N - 1]]))
    E, off = w.host_docs(docs.tolist())
    Qh = w.host_queries(qs)
    dsel = torch.as_tensor(docs, device="cuda")
    print("full-size Doc-Uniform ...", flush=True)
    m, seed = 8, 99
    ru = B.colbandit_doc_uniform(w.Q, w.docs, w.offsets, K, m, seed=seed, want_masks=True)
    torch.cuda.synchronize()
    for j, q in enumerate(qs):
        H = oracle_mod.maxsim_cells(Qh[j], E, off)
        masks = ru["masks"][q][dsel].cpu().numpy().view(np.uint64)
        for n, i in enumerate(docs.tolist()):
            R = oracle_mod.uniform_subset(seed, q, i, w.T, m)
            assert int(masks[n]) == R
            want = sum(H[n, t] for t in range(w.T) if (R >> t) & 1)
            assert float(ru["scores"][q, i]) == pytest.approx(want, rel=TOL["bf16"], abs=1e-4)
        sc = ru["scores"][q].cpu().numpy()
        np.testing.assert_array_equal(ru["topk_ids"][q].cpu().numpy(), np.lexsort((np.arange(w.N), -sc))[:K])
    del ru
    print("full-size Ball-carving ...", flush=True)
    tau = 0.7
    rb = B.colbandit_ball_carving(w.Q, w.docs, w.offsets, K, tau)
    torch.cuda.synchronize()
    for j, q in enumerate(qs):
        k, labels, C, So, _, _ = oracle_mod.ball_carving(Qh[j], E, off, tau, 1, round_bf16=True)
        assert int(rb["n_clusters"][q]) == k
        np.testing.assert_array_equal(rb["labels"][q].cpu().numpy(), labels)
        np.testing.assert_array_equal(rb["centroids"][q].float().cpu().numpy(), C)
        got = rb["scores"][q][dsel].cpu().numpy()
        np.testing.assert_allclose(got, So, rtol=TOL["bf16"], atol=1e-3)
        sc = rb["scores"][q].cpu().numpy()
        np.testing.assert_array_equal(rb["topk_ids"][q].cpu().numpy(), np.lexsort((np.arange(w.N), -sc))[:K])


@pytest.mark.parametrize("idx,shape", [(1, (50000, 64, 32)), (3, (20000, 64, 24)), (4, (100000, 256, 32))])
def test_other_configurations_at_full_size(B, S, oracle_mod, idx, shape):
    """The mid-text, page-like and knob-sweep configurations at their full sizes: exhaustive
    scores of sampled documents against the oracle, then properties that hold at any size -
    the top-K is the ordered head of the score rows, Col-Bandit (bf16 reveals and int8 reveals)
    returns distinct valid documents with the exhaustive path's score bits, the cell accounting
    adds up, and the planted documents of the mid-text corpus are found.  Then every round of
    sampled queries against the oracle (the knob-sweep configuration: at its grid corners)."""
    print(f"generating configuration {idx} at full size ...", flush=True)
    w = S.config(idx, device="cuda")
    assert (w.N, w.nq, w.T) == shape and w.dtype == "bf16"
    K, T = w.K, w.T
    ws = B.new_workspace(w.nq, T, w.d, w.N, w.total_tokens, "cuda")
    full = B.colbandit_full_maxsim(w.Q, w.docs, w.offsets, K=K, workspace=ws)
    res = B.colbandit_topk(w.Q, w.docs, w.offsets, K, w.alpha_ef, w.delta, w.M, w.seed, workspace=ws)
    d8, ds = B.colbandit_quantize_i8(w.docs)
    res8 = B.colbandit_topk(w.Q, w.docs, w.offsets, K, w.alpha_ef, w.delta, w.M, w.seed, workspace=ws,
                            docs_i8=d8, docs_scale=ds)
    torch.cuda.synchronize()
    rng = np.random.default_rng(idx)
    qs = [0, w.nq // 2, w.nq - 1]
    Qh = w.host_queries(qs)
    ids_full = full["topk_ids"].cpu().numpy()
    for j, q in enumerate(qs):
        docs = np.unique(np.concatenate([rng.integers(0, w.N, 12), [0, w.N - 1], ids_full[q]]))
        E, off = w.host_docs(docs.tolist())
        want = oracle_mod.maxsim_cells(Qh[j], E, off).sum(axis=1)
        got = full["scores"][q][torch.as_tensor(docs, device="cuda")].cpu().numpy()
        np.testing.assert_allclose(got, want, rtol=TOL["bf16"], atol=0)
        sc = full["scores"][q].cpu().numpy()
        order = np.lexsort((np.arange(w.N), -sc))[:K]
        np.testing.assert_array_equal(ids_full[q], order)
        np.testing.assert_array_equal(full["topk_scores"][q].cpu().numpy(), sc[order])
    for r in (res, res8):
        ids = r["topk_ids"]
        assert bool((ids >= 0).all()) and bool((ids < w.N).all())
        assert all(len(set(row)) == K for row in ids.tolist())
        assert torch.equal(r["topk_scores"], torch.gather(full["scores"], 1, ids))
        for st in r["stats"]:
            surv = st["survivors"]
            assert surv[0] == w.N and all(surv[k + 1] <= surv[k] for k in range(st["rounds"]))
            assert surv[st["rounds"]] >= K
            cells = sum((min((k + 1) * w.B, T) - k * w.B) * surv[k] for k in range(st["rounds"]))
            assert st["cells_elim"] == cells and st["cells_rescore"] == T * surv[st["rounds"]]
            assert st["cells_unique"] <= w.N * T
    if idx == 1:      # the five strongest planted documents of each query win the exhaustive top-5
        for q in range(w.nq):
            assert set(ids_full[q].tolist()) <= set(w.planted[q])
    overlap = np.mean([len(set(ids_full[q]) & set(res["topk_ids"][q].tolist())) / K for q in range(w.nq)])
    print(f"configuration {idx}: Overlap@{K} {overlap:.3f}, "
          f"coverage {sum(s['cells_unique'] for s in res['stats']) / (w.nq * w.N * T):.3f}", flush=True)
    assert overlap >= 0.5
    # Algorithm 1 round by round against the oracle at this size, in the same batched launch
    # configuration: sampled queries at the configuration's own knobs (bf16 reveals and int8
    # reveals), and for the knob-sweep configuration the corners of its (alpha_ef, K) grid
    scores_of = lambda q: full["scores"][q].cpu().numpy()
    settings = [(w.alpha_ef, K, None, [qs[1]]), (w.alpha_ef, K, (d8, ds), [qs[2]])]
    if idx == 4:
        settings += [(1.0, 1, None, [5]), (1.0, 50, None, [200]), (0.05, 1, None, [77]),
                     (0.05, 50, None, [130]), (0.5, 10, None, [31])]
    for alpha, KK, co, tq in settings:
        print(f"configuration {idx}: traced run alpha_ef={alpha} K={KK} int8={co is not None} queries {tq}",
              flush=True)
        ckw = {} if co is None else {"docs_i8": co[0], "docs_scale": co[1]}
        rt = B.colbandit_topk(w.Q, w.docs, w.offsets, KK, alpha, w.delta, w.M, w.seed, workspace=ws,
                              trace=True, trace_queries=tq, **ckw)
        torch.cuda.synchronize()
        ok = rt["topk_ids"] >= 0
        assert torch.equal(rt["topk_scores"][ok], torch.gather(full["scores"], 1, rt["topk_ids"].clamp(min=0))[ok])
        if (alpha, KK) == (w.alpha_ef, K):                          # tracing changes nothing
            base = res8 if co is not None else res
            assert torch.equal(rt["topk_ids"], base["topk_ids"])
        _rounds_of_sampled_queries(B, oracle_mod, w, rt, tq, KK, alpha, scores_of, coarse=co)
        del rt


# ------------------------------------------------------------------ the C-ABI without Python
def test_c_abi_from_a_plain_host_program(B):
    """tests/native/abi_check.cpp drives the library with hipMalloc'ed buffers and its own
    stream (no torch anywhere in the process) and checks scores against the definition."""
    import os
    import subprocess
    exe = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "abi_check.bin")
    if not os.path.exists(exe):
        pytest.skip("tests/native/abi_check.bin is not built (__graft_entry__.build() builds it)")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "abi_check ok" in r.stdout
