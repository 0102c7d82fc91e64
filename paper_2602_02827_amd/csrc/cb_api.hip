// C-ABI of the library: argument validation, workspace carving and the host-side
// sequencing of the kernels.  No device arithmetic lives here.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "../../include/colbandit.h"
#include "cb_launch.h"

using namespace cb;

namespace {

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Token chunk owned by one workgroup of the dense kernel and one group of its query columns: 4,096,
// or for a small corpus the power of two (at least 128) that gives up to 4,095 workgroups, eight or
// more turns of those that the chip holds: the last turn, often nearly empty, then weighs little.
// (6,007 documents, 0.9 M tokens, one column group: 224 chunks of 4,096 left CUs idle, 84 us for a
// pass; 1,770 of 512 take 31 us.  100 queries x 6,000 documents of 106 tokens 464 -> 426 us
// against 2,047 workgroups; with 8,190 430, 50,000 x 64 unchanged.  fp32, 16 x 20,000: 1,300 us in
// chunks of 4,096 tokens, 1,258 of 1,024, 1,309 of 512, 1,546 of 128; 16 x 5,000 of 100 tokens 361 us against
// 482 with 8,190 workgroups.)
// Several column groups fill the chip with longer chunks, over which a workgroup's query rows are
// loaded less often.
constexpr int kChunkTokens = 4096;
constexpr int64_t kBlocksWanted = 4095;

struct Layout {
    size_t ctl, list0, list1, stat, stat2, pairs, seg_cnt, rescored, scores, cnt_hist, tau_hist, pi,
        chunk_doc, flag, cid, cstat, ccell, q8, qscale, qscratch, total;
    int cache_cap, TP;
};

// Slots per query in the cell cache.
constexpr int64_t kCacheCapMax = 16384;

Layout make_layout(int nq, int T, int d, int64_t N, int64_t total_tokens) {
    Layout L{};
    size_t o = 0;
    const size_t qn = (size_t)nq * (size_t)N;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    L.ctl = take(sizeof(QueryCtl) * (size_t)nq);
    L.list0 = take(4 * qn);
    L.list1 = take(4 * qn);
    L.stat = take(8 * qn);
    L.stat2 = take(8 * qn);
    L.pairs = take(8 * 2 * (size_t)(COLBANDIT_MAX_ROUNDS + 4));
    L.seg_cnt = take(4 * (size_t)nq * 64);
    // Two arrays share storage with arrays that are dead while they live: the exhaustive
    // path's score rows (no call uses them together with the running statistics) lie over
    // `stat`, and the rescored survivors (written after the last round) over `stat2`, which
    // only a round's corpus pass and the prune right after it use, and round 2's table of lists by
    // document (held_of), which is read only where that round is no corpus pass.
    L.scores = L.stat;
    L.rescored = L.stat2;
    L.cnt_hist = take(4 * (size_t)(COLBANDIT_MAX_ROUNDS + 2) * nq);
    L.tau_hist = take(4 * (size_t)(COLBANDIT_MAX_ROUNDS + 2) * nq);
    L.pi = take(4 * (size_t)nq * T);
    L.chunk_doc = take(4 * (size_t)(total_tokens / kChunkTokens + 16));
    L.flag = take(256);
    L.cache_cap = (int)(N < kCacheCapMax ? N : kCacheCapMax);
    {   // floats per cached document: whole 16-column tiles, in the kernels' 1/2/4/8 tile shapes
        const int tq = (T + 15) / 16;
        L.TP = 16 * (tq <= 1 ? 1 : tq <= 2 ? 2 : tq <= 4 ? 4 : 8);
    }
    L.cid = take(4 * (size_t)nq * L.cache_cap);
    L.cstat = take(8 * (size_t)nq * L.cache_cap);
    L.ccell = take(4 * (size_t)nq * L.cache_cap * L.TP);
    L.q8 = take((size_t)nq * T * d);                 // int8 codes of the queries
    L.qscale = take(4 * (size_t)nq);
    L.qscratch = take(quantize_scratch_bytes(nq));
    L.total = o;
    return L;
}

Work carve(void* ws, const Layout& L) {
    char* b = (char*)ws;
    Work W{};
    W.ctl = (QueryCtl*)(b + L.ctl);
    W.list[0] = (int32_t*)(b + L.list0);
    W.list[1] = (int32_t*)(b + L.list1);
    W.stat = (float2*)(b + L.stat);
    W.stat2 = (float2*)(b + L.stat2);
    W.pairs = (unsigned long long*)(b + L.pairs);
    W.seg_cnt = (int32_t*)(b + L.seg_cnt);
    W.rescored = (float*)(b + L.rescored);
    W.scores = (float*)(b + L.scores);
    W.cnt_hist = (int32_t*)(b + L.cnt_hist);
    W.tau_hist = (float*)(b + L.tau_hist);
    W.pi = (int32_t*)(b + L.pi);
    W.chunk_doc = (int32_t*)(b + L.chunk_doc);
    W.flag = (int*)(b + L.flag);
    W.cache_cap = L.cache_cap;
    W.TP = L.TP;
    W.cid = (int32_t*)(b + L.cid);
    W.cstat = (float2*)(b + L.cstat);
    W.ccell = (float*)(b + L.ccell);
    W.q8 = (int8_t*)(b + L.q8);
    W.qscale = (float*)(b + L.qscale);
    W.qscratch = (void*)(b + L.qscratch);
    return W;
}

// Sets the chunk length for passes over `tiles` column tiles, and the place of the chunk table.
// A group of fp32 tiles has half as many.
// pairs: workgroups of two wavefronts (in_pairs), of which a turn is 1,536 that take longer each: a last turn that is less than
// half full, or chunks of one or two documents, cost them more than the others, so their chunks are halved where that saves
// a turn of halves, or makes chunks of a document at most (exhaustive in d = 64, 10 queries of 16 tokens, us, four
// wavefronts / whole chunks / halved: 172,000 documents of 25 tokens 252 / 255 / 225, 85,000 of 100 322 / 310 / 292, 5,898
// pages of 729 147 / 153 / 145, 4,000 of 1,500 196 / 202 / 185; 30,000 of 100, which fill their turns, 125 / 119 / 122).
void choose_chunks(Work& W, const Problem& P, int64_t tiles, bool codes = false, bool pairs = false) {
    const bool f32 = P.dt == DT_F32 && !codes;
    const int64_t per_group = f32 ? 16 : 32;
    const int64_t groups = (tiles + per_group - 1) / per_group;
    const int64_t wanted = kBlocksWanted / groups > 1 ? kBlocksWanted / groups : 1;
    int c = kChunkTokens;
    while (c > 128 && P.total <= wanted * (c / 2)) c /= 2;
    constexpr int64_t kTurn = 1536, kMostHalved = 3 * kBlocksWanted;
    auto chunks = [&](int tokens) { return (P.total + tokens - 1) / tokens; };
    auto turns = [&](int tokens) { return (chunks(tokens) + kTurn - 1) / kTurn; };
    auto halves_pay = [&]() {
        const int64_t doc20 = 20 * P.total / P.N;               // twentieths of a mean document's tokens
        return doc20 < 20 * (int64_t)c && (turns(c / 2) < 2 * turns(c) || (doc20 > 11 * (int64_t)c && doc20 < 19 * (int64_t)c));
    };
    if (pairs)
        while (c > 512 && chunks(c / 2) <= kMostHalved && halves_pay()) c /= 2;
    W.chunk_tokens = c;
    // The table of short chunks (at most kBlocksWanted entries per query, and one; of halved ones three times as
    // many for three queries or more) lies over the
    // quantiser's scratch, which the coding of queries (one workgroup per query) does not use.
    static_assert((kBlocksWanted + 1) * 4 <= 16384 && (kMostHalved + 1) * 4 <= 3 * 16384, "quantize_scratch_bytes holds 16 KB per segment");
    if (c < kChunkTokens) W.chunk_doc = (int32_t*)W.qscratch;
}

// Scoring or revealing every pair by gathering, a wavefront or workgroup each, beats the corpus pass
// for the smallest calls: it needs one launch less and spreads a thousand documents better than
// chunks do (1 query x 1,000 documents of 48 fp32 tokens: 9 us against 19), until the bytes of
// every query's own reading, 5 TB/s, cost as much.
bool small_call(const Problem& P) {
    const double bytes = (double)P.nq * (double)P.total * P.d * (P.dt == DT_BF16 ? 2.0 : 4.0);
    return bytes <= 40e6;
}

// Scores of all pairs: by gathering, or by a corpus pass, for which the chunks are set.  bf16: small_call.
// fp32 weighs both: matrix work, of all column tiles that a pass multiplies, empty ones as well, against
// the filled ones; reading, once against once a query; and whether either fills the chip.  Time model
// (microseconds), from 1,171 shapes (10 to 100,000 documents of 48 to 8,000 tokens, 1 to 32 queries of 16 to 48,
// d = 32 to 128), on which it picks the faster path or one within 8 % of it but for 32 (1.3x: 8 queries of 32 tokens
// x 200 documents of 1,030 in d = 96, a pass of 122 us for a gather of 94; the others 1.2x at most):
//   pass    a token costs 13 to 13.6 ps a tile multiplied (d = 128), 1.3 times that with four tiles a query of d = 96
//           and 128, and 33 a column group for cutting it into pieces; more where chunks are short or wavefronts split
//           the documents; reading at 5.8 TB/s; never less than a document's blocks one after the other in one workgroup
//   gather  14.4 ps a tile filled, 17.6 with four tiles a query of d = 96 and 128, and 7 a query for cutting;
//           reading at 9.7 TB/s (partly from the last-level cache), by several queries of a larger corpus 8.3;
//           never less than a document's blocks in a wavefront, or shared by four
// Up to 82 MB of reading the gather saves a launch and loses at most a tenth where documents are of like length.
// gather and pass, us, T = 32: 5,000 documents of 100 tokens, d = 128: 1 query 53 and 114, 2 83 and 117, 3 124
// and 122, 8 264 and 269; 100,000 (5.1 GB): 1 914 and 1,294, 2 1,706 and 1,510; d = 64: 1 450 and 636, 2 784
// and 728, 8 2,683 and 1,451.
bool score_by_gather(Work& W, const Problem& P) {
    const ScoreShape s = score_shape(P, false);
    choose_chunks(W, P, s.tiles, false, s.nt == 4 && !s.split && in_pairs(P, s.tiles, false));
    if (small_call(P)) return true;
    if (P.dt != DT_F32) return false;
    const double d = P.d, total = (double)P.total, nq = P.nq, blocks = total / (double)P.N / 16.0;
    const double corpus = total * d * 4.0;
    if (always_gathers(s, P.d) || nq * corpus <= 82e6) return true;
    // a little more than the larger (n: how little)
    const auto both = [](double a, double b, double n) { return pow(pow(a, n) + pow(b, n), 1.0 / n); };
    const bool eight = P.d >= 96 && s.tq <= 2;       // groups of 16 tiles have eight wavefronts
    const bool four = P.d >= 96 && s.tq == 4;        // one or two wavefronts per SIMD
    const double tiles = 4.0 * s.nt * s.groups / (s.split ? s.split / 1.3 : 1.0);
    const double cut = 33.0 * s.groups * (s.split ? 1.7 : 1.0);
    const double multiply = total * (tiles * (s.nt == 2 || eight ? 13.0 : 13.6) * (four ? 1.3 : 1.0) + cut) * 1e-6 *
                            (1.0 + 58.0 / W.chunk_tokens) * d / 128.0 * (P.d == 96 ? 1.2 : 1.0);
    const double t_pass = 13.0 + fmax(both(multiply, corpus / 5.8e6, 3.0), blocks * (0.19 + (s.nt == 2 ? 0.0058 : 0.0085) * d));
    const double filled = nq * (total + 8.0 * (double)P.N) * (7.0 + 14.4 * s.tq + (four ? 13.0 : 0.0)) * 1e-6 * (d + 3.8) / 128.0;
    const double read = nq * corpus / (corpus > 256e6 && P.nq > 1 ? 8.3e6 : 9.7e6);
    const double t_gather = 14.0 + fmax(both(filled, read, 2.3),
                                        blocks * (0.12 + 0.00082 * d * (s.tq + 5)) / (gather_shares(P) ? 4.0 : 1.0));
    return t_gather < t_pass;
}

int check_shapes(const void* Q, int nq, int T, int d, int dt, const void* docs,
                 const int64_t* off, int64_t N, int64_t total) {
    if (!Q || !docs || !off) return COLBANDIT_ERR_NULL;
    if (nq < 1 || T < 1 || d < 1 || N < 1 || total < N) return COLBANDIT_ERR_SHAPE;
    if (dt != COLBANDIT_F32 && dt != COLBANDIT_BF16) return COLBANDIT_ERR_SHAPE;
    // the selection kernels form indexes up to three chunks of 8,192 entries past a list's end
    if (N > 0x7fffffff - (1 << 17) || nq > 65535) return COLBANDIT_ERR_UNSUPPORTED;
    if (d != 32 && d != 64 && d != 96 && d != 128) return COLBANDIT_ERR_UNSUPPORTED;
    if (T > (dt == COLBANDIT_BF16 ? COLBANDIT_MAX_T : 64)) return COLBANDIT_ERR_UNSUPPORTED;
    if (((uintptr_t)Q & 15) || ((uintptr_t)docs & 15) || ((uintptr_t)off & 7))
        return COLBANDIT_ERR_ALIGNMENT;
    return COLBANDIT_OK;
}

int check_workspace(const void* ws, size_t bytes, size_t need) {
    if (!ws) return COLBANDIT_ERR_NULL;
    if ((uintptr_t)ws & 255) return COLBANDIT_ERR_ALIGNMENT;
    if (bytes < need) return COLBANDIT_ERR_WORKSPACE;
    return COLBANDIT_OK;
}

// Phase timing for colbandit_stats: one HIP event per phase boundary on the call's stream.
enum { PH_FIRST_REVEAL = 0, PH_LATER_REVEAL = 1, PH_SELECT = 2, PH_RESCORE = 3, PH_ROUND2_REVEAL = 4,
       PH_COUNT = 5 };
struct PhaseTimer {
    static constexpr int kMax = 4 * (COLBANDIT_MAX_ROUNDS + 4);
    hipEvent_t ev[kMax];
    int phase[kMax];       // phase that ENDS at event i (event 0 is the start)
    int n = 0;
    bool on = false;
    hipStream_t st = nullptr;
    bool start(hipStream_t s) {
        on = true;
        st = s;
        return mark(-1);
    }
    bool mark(int ph) {
        if (!on) return true;
        if (n >= kMax) return true;
        if (hipEventCreate(&ev[n]) != hipSuccess) return false;
        phase[n] = ph;
        (void)hipEventRecord(ev[n], st);
        ++n;
        return true;
    }
    void collect(float (&ms)[PH_COUNT], float& total) {      // after the stream was synchronised
        for (int i = 0; i < PH_COUNT; ++i) ms[i] = 0.f;
        total = 0.f;
        for (int i = 1; i < n; ++i) {
            float t = 0.f;
            (void)hipEventElapsedTime(&t, ev[i - 1], ev[i]);
            if (phase[i] >= 0) ms[phase[i]] += t;
            total += t;
        }
    }
    void destroy() {
        for (int i = 0; i < n; ++i) (void)hipEventDestroy(ev[i]);
        n = 0;
    }
};

// Number of (query, document) pairs above which round r of R is cheaper as one corpus pass
// shared by all queries than as per-pair gathers.  Time model (seconds), with the rates these
// kernels reach on an MI355X: a corpus pass costs the larger of streaming the tokens once
// (~3.5 TB/s) and the matrix work of all query rows against them (~1.15 PFLOP/s); a gathered
// pair streams its document once (~4.5 TB/s) and nothing is shared between queries.  A
// gathered visit also caches the document's cells for the remaining rounds when the query fits
// the cache, so the gather is preferred up to twice the cost of the pass and, where every list
// fits, of a round's other launches (~18 us): there a gathered round is the last one to launch,
// which also saves those of all rounds after it.  Lists beyond the cache are launched round after round
// either way, and where even full ones are gathered for no more than twice a pass and a round's
// launches the pass is left out (~0): its empty launch is 4 us in every round (3 queries x 19,583 documents of
// 48 tokens, T = 53 in rounds of 2, d = 32, a full gather 40 us and a pass 17: 762 us with it, 732 without).
unsigned long long dense_pairs_threshold(const Problem& P, int G, bool codes, int r, int R, bool lists_fit, double* t_gather) {
    // int8 codes: half the bytes of bf16 and twice the rate
    const double row_bytes = (codes ? 1.0 : P.dt == DT_BF16 ? 2.0 : 4.0) * P.d;
    const double rate = codes ? 2.3e15 : 1.15e15;
    const double rows = (double)(((int64_t)P.nq * G + 15) / 16 * 16);
    double per_token = fmax(row_bytes / 3.5e12, 2.0 * rows * P.d / rate);
    const double t_round = 18e-6;
    const double doc_tokens = (double)P.total / (double)P.N;
    double t_pass = (double)P.total * per_token;
    double t_pair = doc_tokens * row_bytes / 4.5e12;
    double passes = 2.0;
    if (!codes && P.dt == DT_F32) {
        // The matrix work of both weighs too (terms as in score_by_gather; a round's kernels are a little slower): all T tokens of a pair
        // at once against a batch in each pass, so where the lists fit the cache the one visit is weighed
        // against a pass in every round left.  A pass takes no less than a mean document's blocks one
        // after the other in a workgroup.
        const int tq = (P.T + 15) / 16;
        const bool two = rows <= 128.0;
        const double tiles = rows <= 64.0 ? 4.0 : two ? 8.0 : ceil(rows / 256.0) * 16.0;
        const double groups = two ? 1.0 : tiles / 16.0;
        per_token = fmax(row_bytes / 4.5e12, (tiles * (two || P.d >= 96 ? 15.4 : 14.2) + 25.0 * groups) * 1e-12 * P.d / 128.0);
        t_pass = (double)P.total * per_token;
        t_pass = fmax(t_pass, doc_tokens / 16.0 * (0.13e-6 + (two ? 0.006e-6 : 0.012e-6) * P.d));
        const int tile = tq <= 1 ? 1 : tq <= 2 ? 2 : 4;
        if ((double)P.total * row_bytes <= 256e6) t_pair = doc_tokens * row_bytes / 7.2e12;   // in the last-level cache
        t_pair = fmax(t_pair, doc_tokens * (16.5 + 13.5 * tile + (tile == 4 && P.d >= 96 ? 19.0 : 0.0)) * 1e-12 * (P.d + 12) / 128.0);
        if (lists_fit) passes = R - r + 1;
    }
    if (!lists_fit && (double)P.nq * (double)P.N * t_pair < passes * (t_pass + t_round)) return ~0ull;
    const double worth = passes * t_pass + (lists_fit ? (passes + R - r) * t_round : 0.0);
    // Queries that share a corpus of the last-level cache's size gather faster, and where lists fit and even full
    // ones cost no more to read than what the gather saves, none of the later rounds is launched (7 queries x 6,007
    // documents, d = 64, T = 21: 144 -> 109 us; 16 x 6,000 164 -> 107, with alpha 1.0, where they stay full, 339 -> 294).
    // fp32 as well by its bytes, though its matrix work can make full lists cost 1.4 times as much: lists are seldom full,
    // and a threshold brings the empty launches back (5,000 documents, d = 128, 64 queries of 64 tokens: 511 us so
    // and 782 by t_pair's price, with alpha 1.0 593 and 869; of 40 calls between the two prices only one was slower:
    // 10,000 documents, d = 32, 120 queries, alpha 1.0 1,459 and 1,297).
    if (lists_fit && (double)P.total * row_bytes <= 256e6 &&
        (double)P.nq * (double)P.total * row_bytes / 7.5e12 <= worth) return ~0ull;
    const double thr = worth / t_pair;
    *t_gather = t_pair;
    return thr >= 1.8e19 ? ~0ull - 1 : (unsigned long long)thr;
}

// Scratch of colbandit_topk_static: part of the device image, one copy per GPU.  Host code
// never uses this name as an address; it asks the runtime for the copy of the current device.
__device__ __align__(256) unsigned char scratch[COLBANDIT_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];          // device address of `scratch` on each GPU, once known
std::mutex g_scratch_mutex;

// Address of the current device's copy of `scratch` (looked up once per device).
hipError_t static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

double rho_n(int n, int T) {
    // finite-population correction, Appendix A
    if (2 * n <= T) return 1.0 - (double)(n - 1) / (double)T;
    return (1.0 - (double)n / (double)T) * (1.0 + 1.0 / (double)n);
}

}  // namespace

extern "C" {

const char* colbandit_strerror(int code) {
    switch (code) {
        case COLBANDIT_OK: return "ok";
        case COLBANDIT_ERR_NULL: return "a required pointer is NULL";
        case COLBANDIT_ERR_SHAPE: return "invalid size (n_queries, T, d, N, total_tokens, K or dtype)";
        case COLBANDIT_ERR_KNOB: return "knob out of range (alpha_ef, delta, M, B or support [a,b])";
        case COLBANDIT_ERR_UNSUPPORTED: return "request outside what this build's kernels cover";
        case COLBANDIT_ERR_WORKSPACE: return "workspace or trace buffer too small";
        case COLBANDIT_ERR_ALIGNMENT: return "pointer not aligned as required";
        case COLBANDIT_ERR_HIP: return "HIP runtime error";
        case COLBANDIT_ERR_BAD_OFFSETS: return "doc_offsets violates its preconditions";
        case COLBANDIT_ERR_TOO_LARGE:
            return "sizes need more scratch than the library's built-in buffer "
                   "(COLBANDIT_STATIC_SCRATCH_BYTES): use colbandit_topk with a workspace";
        default: return "unknown error code";
    }
}

int colbandit_permutation(uint64_t seed, int64_t query_index, int T, int32_t* pi) {
    if (!pi) return COLBANDIT_ERR_NULL;
    if (T < 1 || query_index < 0) return COLBANDIT_ERR_SHAPE;
    uint64_t s = seed + ((uint64_t)query_index + 1ull) * 0x9E3779B97F4A7C15ull;
    for (int t = 0; t < T; ++t) pi[t] = t;
    for (int i = T - 1; i >= 1; --i) {
        s += 0x9E3779B97F4A7C15ull;
        uint64_t z = s;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        const int j = (int)(z % (uint64_t)(i + 1));
        const int32_t tmp = pi[i];
        pi[i] = pi[j];
        pi[j] = tmp;
    }
    return COLBANDIT_OK;
}

double colbandit_radius_prefactor(float alpha_ef, float delta, int T, int64_t N, int n) {
    if (n <= 1) return INFINITY;
    const double lg = log((double)N * (double)T / (double)delta);
    return (double)alpha_ef * (double)T * sqrt(2.0 * lg / (double)n) * sqrt(rho_n(n, T));
}

size_t colbandit_trace_bytes(int n_queries, int T, int B, int64_t N) {
    if (n_queries < 1 || T < 1 || B < 1 || N < 1) return 0;
    const size_t R = (size_t)((T + B - 1) / B), nq = (size_t)n_queries;
    return align_up(4 * (R + 1) * nq) + align_up(4 * R * nq) + 2 * align_up(4 * R * nq * (size_t)N) +
           align_up(R * nq * (size_t)N);
}

size_t colbandit_workspace_bytes(int n_queries, int T, int d, int64_t N, int64_t total_tokens,
                                 int K, int M) {
    (void)K; (void)M;
    if (n_queries < 1 || T < 1 || N < 1 || total_tokens < N) return 0;
    return make_layout(n_queries, T, d, N, total_tokens).total;
}

int colbandit_validate_offsets(const int64_t* doc_offsets, int64_t N, int64_t total_tokens,
                               void* workspace, size_t workspace_bytes, void* stream) {
    if (!doc_offsets) return COLBANDIT_ERR_NULL;
    if (N < 1 || total_tokens < N) return COLBANDIT_ERR_SHAPE;
    int rc = check_workspace(workspace, workspace_bytes, 256);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    int* flag = (int*)workspace;
    if (launch_validate_offsets(doc_offsets, N, total_tokens, flag, st) != hipSuccess)
        return COLBANDIT_ERR_HIP;
    int h = 0;
    if (hipMemcpyAsync(&h, flag, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess)
        return COLBANDIT_ERR_HIP;
    if (hipStreamSynchronize(st) != hipSuccess) return COLBANDIT_ERR_HIP;
    return h ? COLBANDIT_ERR_BAD_OFFSETS : COLBANDIT_OK;
}

size_t colbandit_quantize_workspace_bytes(int64_t n_segments) {
    if (n_segments < 1) return 0;
    return align_up(quantize_scratch_bytes(n_segments));
}

int colbandit_quantize_i8(const void* x, colbandit_dtype dt, int64_t n_segments,
                          int64_t rows_per_segment, int d, int permille, int8_t* codes,
                          float* scales, void* workspace, size_t workspace_bytes, void* stream) {
    if (!x || !codes || !scales) return COLBANDIT_ERR_NULL;
    if (n_segments < 1 || n_segments > 65535 || rows_per_segment < 1 || d < 1)
        return COLBANDIT_ERR_SHAPE;
    if (dt != COLBANDIT_F32 && dt != COLBANDIT_BF16) return COLBANDIT_ERR_SHAPE;
    if (permille < 1 || permille > 1000) return COLBANDIT_ERR_KNOB;
    if (rows_per_segment > (int64_t)0x7fffffffffffLL / d) return COLBANDIT_ERR_UNSUPPORTED;
    if (((uintptr_t)x & 15) || ((uintptr_t)scales & 3)) return COLBANDIT_ERR_ALIGNMENT;
    int rc = check_workspace(workspace, workspace_bytes, colbandit_quantize_workspace_bytes(n_segments));
    if (rc) return rc;
    const hipError_t e = launch_quantize_i8(x, (int)dt, n_segments, rows_per_segment * d, permille,
                                            codes, scales, workspace, (hipStream_t)stream);
    return e == hipSuccess ? COLBANDIT_OK : COLBANDIT_ERR_HIP;
}

int colbandit_coarse_maxsim(const void* Q, int n_queries, int T, int d, colbandit_dtype dt,
                            const int8_t* docs_i8, const float* docs_scale,
                            const int64_t* doc_offsets, int64_t N, int64_t total_tokens,
                            int permille, float* scores, float* cells, int8_t* q_codes,
                            float* q_scales, void* workspace, size_t workspace_bytes,
                            void* stream) {
    int rc = check_shapes(Q, n_queries, T, d, (int)dt, docs_i8, doc_offsets, N, total_tokens);
    if (rc) return rc;
    if (!docs_scale || !scores) return COLBANDIT_ERR_NULL;
    if (permille < 1 || permille > 1000) return COLBANDIT_ERR_KNOB;
    const Layout L = make_layout(n_queries, T, d, N, total_tokens);
    rc = check_workspace(workspace, workspace_bytes, L.total);
    if (rc) return rc;
    Work W = carve(workspace, L);
    const Problem P{Q, n_queries, T, d, (int)dt, docs_i8, doc_offsets, N, total_tokens};
    const ScoreShape s = score_shape(P, true);
    choose_chunks(W, P, s.tiles, true, s.nt == 4 && !s.split && in_pairs(P, s.tiles, true));
    hipStream_t st = (hipStream_t)stream;
    Coarse co{docs_i8, docs_scale, W.q8, W.qscale};
    if (!dense_supported(P, &co)) return COLBANDIT_ERR_UNSUPPORTED;
    hipError_t e = launch_quantize_i8(Q, (int)dt, n_queries, (int64_t)T * d, permille, W.q8,
                                      W.qscale, W.qscratch, st);
    int n_chunks = 0;
    if (e == hipSuccess) e = launch_dense_prepare(P, W, &n_chunks, st);
    if (e == hipSuccess) e = launch_dense_score(P, W, n_chunks, scores, cells, &co, st);
    if (e == hipSuccess && q_codes)
        e = hipMemcpyAsync(q_codes, W.q8, (size_t)n_queries * T * d, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && q_scales)
        e = hipMemcpyAsync(q_scales, W.qscale, sizeof(float) * n_queries, hipMemcpyDeviceToDevice, st);
    return e == hipSuccess ? COLBANDIT_OK : COLBANDIT_ERR_HIP;
}

// ---- the two non-adaptive baselines (appendix "Compared Methods")

namespace {
struct UniformLayout { size_t base, cells, total; };
UniformLayout uniform_layout(int nq, int T, int d, int64_t N, int64_t total_tokens) {
    UniformLayout U{};
    U.base = make_layout(nq, T, d, N, total_tokens).total;
    U.cells = U.base;
    U.total = U.cells + align_up(4 * (size_t)nq * (size_t)N * (size_t)T);
    return U;
}
struct BallLayout { size_t base, Cz, kq, labels, goff, Qg, ident, part, total; int TG; };
BallLayout ball_layout(int nq, int T, int d, int dt, int64_t N, int64_t total_tokens) {
    BallLayout B{};
    size_t o = make_layout(nq, T, d, N, total_tokens).total;
    B.base = o;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    const size_t elem = dt == COLBANDIT_BF16 ? 2 : 4;
    B.TG = (T + 3) / 4;
    B.Cz = take(elem * (size_t)nq * T * d);
    B.kq = take(4 * (size_t)nq);
    B.labels = take(4 * (size_t)nq * T);
    B.goff = take(4 * ((size_t)nq + 1));
    if (dt == COLBANDIT_BF16) {
        B.Qg = take(2 * (size_t)nq * B.TG * 4 * d);
        B.ident = take(4 * (size_t)nq * B.TG * 4);
        B.part = take(8 * (size_t)nq * B.TG * (size_t)N);
    }
    B.total = o;
    return B;
}
}  // namespace

size_t colbandit_doc_uniform_workspace_bytes(int n_queries, int T, int d, int64_t N,
                                             int64_t total_tokens) {
    if (n_queries < 1 || T < 1 || N < 1 || total_tokens < N) return 0;
    return uniform_layout(n_queries, T, d, N, total_tokens).total;
}

int colbandit_cells_per_doc(double gamma, int T) {
    if (T < 1) return COLBANDIT_ERR_SHAPE;
    if (!(gamma > 0.0) || !(gamma <= 1.0)) return COLBANDIT_ERR_KNOB;
    const double m = ceil(gamma * (double)T - 1e-9);
    return m < 1.0 ? 1 : (m > (double)T ? T : (int)m);
}

int colbandit_doc_uniform(const void* Q, int n_queries, int T, int d, colbandit_dtype dt,
                          const void* doc_tokens, const int64_t* doc_offsets, int64_t N,
                          int64_t total_tokens, int K, int cells_per_doc, uint64_t seed,
                          float* scores, uint64_t* masks, int64_t* topk_ids, float* topk_scores,
                          void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_shapes(Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens);
    if (rc) return rc;
    if (K < 0 || K > N) return COLBANDIT_ERR_SHAPE;
    if (K > COLBANDIT_MAX_K || T > 64) return COLBANDIT_ERR_UNSUPPORTED;
    if (cells_per_doc < 1 || cells_per_doc > T) return COLBANDIT_ERR_KNOB;
    if (K == 0 && !scores) return COLBANDIT_ERR_NULL;
    if (K > 0 && (!topk_ids || !topk_scores)) return COLBANDIT_ERR_NULL;
    if ((uintptr_t)masks & 7) return COLBANDIT_ERR_ALIGNMENT;
    const UniformLayout U = uniform_layout(n_queries, T, d, N, total_tokens);
    rc = check_workspace(workspace, workspace_bytes, U.total);
    if (rc) return rc;
    Work W = carve(workspace, make_layout(n_queries, T, d, N, total_tokens));
    const Problem P{Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens};
    hipStream_t st = (hipStream_t)stream;
    float* cells = (float*)((char*)workspace + U.cells);
    float* out = scores ? scores : W.scores;
    // the whole MaxSim matrix (exhaustive row sums go to a scratch array), then the subset sums
    hipError_t e = hipSuccess;
    if (score_by_gather(W, P)) {
        e = launch_gather_all(P, W, W.rescored, cells, st);
    } else {
        int n_chunks = 0;
        e = launch_dense_prepare(P, W, &n_chunks, st);
        if (e == hipSuccess) e = launch_dense_score(P, W, n_chunks, W.rescored, cells, nullptr, st);
    }
    if (e == hipSuccess)
        e = launch_uniform_score(cells, n_queries, N, T, cells_per_doc, seed, out, masks, st);
    if (e == hipSuccess && K > 0) e = launch_topk(P, W, false, false, false, out, K, topk_ids, topk_scores, st);
    return e == hipSuccess ? COLBANDIT_OK : COLBANDIT_ERR_HIP;
}

size_t colbandit_ball_carving_workspace_bytes(int n_queries, int T, int d, colbandit_dtype dt,
                                              int64_t N, int64_t total_tokens) {
    if (n_queries < 1 || T < 1 || N < 1 || total_tokens < N) return 0;
    if (dt != COLBANDIT_F32 && dt != COLBANDIT_BF16) return 0;
    return ball_layout(n_queries, T, d, (int)dt, N, total_tokens).total;
}

int colbandit_ball_carving(const void* Q, int n_queries, int T, int d, colbandit_dtype dt,
                           const void* doc_tokens, const int64_t* doc_offsets, int64_t N,
                           int64_t total_tokens, int K, float tau, int32_t* n_clusters,
                           int32_t* labels, void* centroids, float* scores, int64_t* topk_ids,
                           float* topk_scores, void* workspace, size_t workspace_bytes,
                           void* stream) {
    int rc = check_shapes(Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens);
    if (rc) return rc;
    if (K < 0 || K > N) return COLBANDIT_ERR_SHAPE;
    if (K > COLBANDIT_MAX_K || T > 64) return COLBANDIT_ERR_UNSUPPORTED;
    if (!(tau > 0.f) || !(tau <= 1.f)) return COLBANDIT_ERR_KNOB;
    if (K == 0 && !scores) return COLBANDIT_ERR_NULL;
    if (K > 0 && (!topk_ids || !topk_scores)) return COLBANDIT_ERR_NULL;
    if (((uintptr_t)n_clusters & 3) || ((uintptr_t)labels & 3) || ((uintptr_t)centroids & 15))
        return COLBANDIT_ERR_ALIGNMENT;
    const BallLayout B = ball_layout(n_queries, T, d, (int)dt, N, total_tokens);
    rc = check_workspace(workspace, workspace_bytes, B.total);
    if (rc) return rc;
    Work W = carve(workspace, make_layout(n_queries, T, d, N, total_tokens));
    const Problem P{Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens};
    hipStream_t st = (hipStream_t)stream;
    char* b = (char*)workspace;
    void* Cz = b + B.Cz;
    int32_t* kq = (int32_t*)(b + B.kq);
    int32_t* lab = (int32_t*)(b + B.labels);
    int32_t* goff = (int32_t*)(b + B.goff);
    float* out = scores ? scores : W.scores;
    const size_t elem = dt == COLBANDIT_BF16 ? 2 : 4;

    hipError_t e = launch_ball_carve(P, tau, Cz, lab, kq, st);
    if (e == hipSuccess && dt == COLBANDIT_BF16 && (d == 64 || d == 128)) {
        // centroids of the batch, four to a group, through the corpus-streaming reveal kernel:
        // its work follows the number of query columns, i.e. the number of centroids
        void* Qg = b + B.Qg;
        int32_t* ident = (int32_t*)(b + B.ident);
        float2* part = (float2*)(b + B.part);
        e = launch_ball_groups(P, Cz, kq, goff, Qg, ident, st);
        int32_t ng = 0;
        if (e == hipSuccess)
            e = hipMemcpyAsync(&ng, goff + n_queries, sizeof(int32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e == hipSuccess && (ng < n_queries || (int64_t)ng > (int64_t)n_queries * B.TG))
            e = hipErrorUnknown;
        int n_chunks = 0;
        if (e == hipSuccess) {                       // else ng has not arrived
            choose_chunks(W, P, ((int64_t)ng * 4 + 15) / 16);
            e = launch_dense_prepare(P, W, &n_chunks, st);
        }
        if (e == hipSuccess) {
            const Problem P2{Qg, ng, 4, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens};
            Work W2 = W;
            W2.pi = ident;
            W2.stat = part;
            RevealRound rr{};
            rr.r = 1;
            rr.lo = 0;
            rr.nb = 4;
            rr.n = 4;
            rr.dense = kNeverDense;
            e = launch_dense_reveal(P2, W2, n_chunks, rr, 4, nullptr, st);
        }
        if (e == hipSuccess) e = launch_ball_reduce((const float*)part, 2, goff, n_queries, N, out, st);
    } else if (e == hipSuccess) {
        // fp32, and widths without a group pass: exhaustive scoring of the zero-padded centroid
        // matrix (a zero row's cell is 0)
        const Problem P3{Cz, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens};
        e = launch_gather_all(P3, W, out, nullptr, st);
    }
    if (e == hipSuccess && n_clusters)
        e = hipMemcpyAsync(n_clusters, kq, 4 * (size_t)n_queries, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && labels)
        e = hipMemcpyAsync(labels, lab, 4 * (size_t)n_queries * T, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && centroids)
        e = hipMemcpyAsync(centroids, Cz, elem * (size_t)n_queries * T * d, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && K > 0) e = launch_topk(P, W, false, false, false, out, K, topk_ids, topk_scores, st);
    return e == hipSuccess ? COLBANDIT_OK : COLBANDIT_ERR_HIP;
}

size_t colbandit_sizeof_opts(void) { return sizeof(colbandit_opts); }
size_t colbandit_sizeof_stats(void) { return sizeof(colbandit_stats); }

int colbandit_full_maxsim(const void* Q, int n_queries, int T, int d, colbandit_dtype dt,
                          const void* doc_tokens, const int64_t* doc_offsets, int64_t N,
                          int64_t total_tokens, int K, float* scores, int64_t* topk_ids,
                          float* topk_scores, float* cells, float* phase_ms, void* workspace,
                          size_t workspace_bytes, void* stream) {
    int rc = check_shapes(Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens);
    if (rc) return rc;
    if (K < 0 || K > N) return COLBANDIT_ERR_SHAPE;
    if (K > COLBANDIT_MAX_K) return COLBANDIT_ERR_UNSUPPORTED;
    if (K == 0 && !scores) return COLBANDIT_ERR_NULL;
    if (K > 0 && (!topk_ids || !topk_scores)) return COLBANDIT_ERR_NULL;
    const Layout L = make_layout(n_queries, T, d, N, total_tokens);
    rc = check_workspace(workspace, workspace_bytes, L.total);
    if (rc) return rc;

    Work W = carve(workspace, L);
    const Problem P{Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens};
    hipStream_t st = (hipStream_t)stream;
    float* out = scores ? scores : W.scores;

    // phase_ms: event 0 | chunk table | event 1 | scoring kernel | event 2 | top-K | event 3
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    int n_ev = 0;
    auto mark = [&]() {
        if (phase_ms && n_ev < 4 && hipEventCreate(&ev[n_ev]) == hipSuccess) (void)hipEventRecord(ev[n_ev++], st);
    };
    hipError_t e = hipSuccess;
    mark();
    if (score_by_gather(W, P)) {
        mark();
        e = launch_gather_all(P, W, out, cells, st);
    } else {
        int n_chunks = 0;
        e = launch_dense_prepare(P, W, &n_chunks, st);
        mark();
        if (e == hipSuccess) e = launch_dense_score(P, W, n_chunks, out, cells, nullptr, st);
    }
    mark();
    if (e == hipSuccess && K > 0) e = launch_topk(P, W, false, false, false, out, K, topk_ids, topk_scores, st);
    mark();
    if (phase_ms) {
        phase_ms[0] = phase_ms[1] = 0.f;
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e == hipSuccess && n_ev == 4) {
            (void)hipEventElapsedTime(&phase_ms[0], ev[1], ev[2]);
            (void)hipEventElapsedTime(&phase_ms[1], ev[2], ev[3]);
        } else if (e == hipSuccess) {
            e = hipErrorUnknown;
        }
        for (int i = 0; i < n_ev; ++i) (void)hipEventDestroy(ev[i]);
    }
    return e == hipSuccess ? COLBANDIT_OK : COLBANDIT_ERR_HIP;
}

// Body of colbandit_topk and colbandit_topk_static.  builtin_scratch: the workspace is the
// current device's copy of `scratch` (looked up only after every argument has passed).
static int topk_impl(const void* Q, int n_queries, int T, int d, colbandit_dtype dt,
                     const void* doc_tokens, const int64_t* doc_offsets, int64_t N,
                     int64_t total_tokens, int K, float alpha_ef, float delta, int M, uint64_t seed,
                     const colbandit_opts* opts, int64_t* topk_ids, float* topk_scores,
                     colbandit_stats* stats, void* workspace, size_t workspace_bytes,
                     bool builtin_scratch, void* stream) {
    int rc = check_shapes(Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens);
    if (rc) return rc;
    if (!topk_ids || !topk_scores) return COLBANDIT_ERR_NULL;
    if (K < 1 || K > N) return COLBANDIT_ERR_SHAPE;
    if (K > COLBANDIT_MAX_K) return COLBANDIT_ERR_UNSUPPORTED;
    if (!(alpha_ef > 0.f) || !(alpha_ef <= 1.f) || !(delta > 0.f) || !(delta < 1.f) || M < 0)
        return COLBANDIT_ERR_KNOB;
    Knobs kn{K, M, 4, -1.f, 1.f, alpha_ef <= 0.25f};
    const int32_t* user_pi = nullptr;
    void* trace = nullptr;
    size_t trace_bytes = 0;
    bool force_gather = false, no_cache = false;
    int later_rounds = 0;
    Coarse coarse{};
    int q_permille = 999;
    if (opts) {
        if (opts->B < 0) return COLBANDIT_ERR_KNOB;
        if (opts->B > 0) kn.B = opts->B;
        if (!(opts->a == 0.f && opts->b == 0.f)) {
            if (!(opts->a < opts->b)) return COLBANDIT_ERR_KNOB;
            kn.a = opts->a;
            kn.b = opts->b;
        }
        user_pi = opts->pi;
        trace = opts->trace;
        trace_bytes = opts->trace_bytes;
        force_gather = opts->force_gather != 0;
        no_cache = opts->no_cell_cache != 0;
        if (opts->later_rounds < 0 || opts->later_rounds > 2) return COLBANDIT_ERR_KNOB;
        later_rounds = opts->later_rounds;
        if (opts->docs_i8) {
            if (!opts->docs_scale) return COLBANDIT_ERR_NULL;
            if (d % 64 != 0) return COLBANDIT_ERR_UNSUPPORTED;   // int8 MFMA contracts 64 at a time
            if (((uintptr_t)opts->docs_i8 & 15) || ((uintptr_t)opts->docs_scale & 3))
                return COLBANDIT_ERR_ALIGNMENT;
            if (opts->coarse_permille < 0 || opts->coarse_permille > 1000) return COLBANDIT_ERR_KNOB;
            if (opts->coarse_permille > 0) q_permille = opts->coarse_permille;
            coarse.docs8 = opts->docs_i8;
            coarse.dscale = opts->docs_scale;
        }
    }
    if (kn.B > COLBANDIT_MAX_B) return COLBANDIT_ERR_UNSUPPORTED;
    const int R = (T + kn.B - 1) / kn.B;
    if (R > COLBANDIT_MAX_ROUNDS) return COLBANDIT_ERR_UNSUPPORTED;
    const Layout L = make_layout(n_queries, T, d, N, total_tokens);
    if (builtin_scratch) {
        if (L.total > (size_t)COLBANDIT_STATIC_SCRATCH_BYTES) return COLBANDIT_ERR_TOO_LARGE;
        workspace_bytes = (size_t)COLBANDIT_STATIC_SCRATCH_BYTES;
    } else {
        rc = check_workspace(workspace, workspace_bytes, L.total);
        if (rc) return rc;
    }

    Trace tr{};
    if (trace) {
        if ((uintptr_t)trace & 255) return COLBANDIT_ERR_ALIGNMENT;
        if (trace_bytes < colbandit_trace_bytes(n_queries, T, kn.B, N)) return COLBANDIT_ERR_WORKSPACE;
        char* b = (char*)trace;
        const size_t nq = (size_t)n_queries, Rn = (size_t)R;
        tr.count = (int32_t*)b;
        b += align_up(4 * (Rn + 1) * nq);
        tr.tau = (float*)b;
        b += align_up(4 * Rn * nq);
        tr.lcb = (float*)b;
        b += align_up(4 * Rn * nq * (size_t)N);
        tr.ucb = (float*)b;
        b += align_up(4 * Rn * nq * (size_t)N);
        tr.alive = (uint8_t*)b;
    }

    if (builtin_scratch && static_scratch(&workspace) != hipSuccess) return COLBANDIT_ERR_HIP;
    Work W = carve(workspace, L);
    if (no_cache) W.cache_cap = 0;
    // The work items lie over rows of tau_hist that no round of this call writes (rows R and up; two
    // rows of nq floats, at an even number of floats).
    static_assert(COLBANDIT_MAX_ROUNDS % 2 == 0, "the last pair of spare rows starts at an even one");
    W.work = (unsigned long long*)(W.tau_hist + (size_t)(R + ((R & 1) && (n_queries & 1) ? 1 : 0)) * n_queries);
    const Problem P{Q, n_queries, T, d, (int)dt, doc_tokens, doc_offsets, N, total_tokens};
    hipStream_t st = (hipStream_t)stream;

    PhaseTimer pt;
    if (stats && !pt.start(st)) return COLBANDIT_ERR_HIP;

    hipError_t e = hipSuccess;
    const bool loop = N > (int64_t)K + M;    // |A_1| > K + M, else the loop body never runs
    // coarse pass: code the queries (per query) and reveal from the int8 codes
    const Coarse* co = nullptr;
    if (coarse.docs8) {
        coarse.Q8 = W.q8;
        coarse.qscale = W.qscale;
        co = &coarse;
        if (e == hipSuccess && loop)
            e = launch_quantize_i8(Q, (int)dt, n_queries, (int64_t)T * d, q_permille, W.q8,
                                   W.qscale, W.qscratch, st);
    }
    const bool dense = dense_supported(P, co) && !force_gather && !(small_call(P) && later_rounds != 1);
    int G_max = 1;                                   // columns of a full batch
    while (G_max < kn.B) G_max <<= 1;
    const int64_t reveal_tiles = ((int64_t)n_queries * G_max + 15) / 16;
    choose_chunks(W, P, reveal_tiles, co != nullptr, in_pairs(P, reveal_tiles, co != nullptr));
    const int n_chunks = loop && dense ? dense_chunks(P, W) : 0;
    // the smallest calls visit every document once: round 1 caches all cells of all documents
    const bool cache_all = loop && !dense && !force_gather && later_rounds == 0 && small_call(P) &&
                           N <= (int64_t)W.cache_cap;
    if (e == hipSuccess) e = cache_all ? launch_cache_all(P, W, kn, R, seed, user_pi, tr, co, st)
                                       : launch_init(P, W, kn, R, seed, user_pi, tr, co, n_chunks, st);
    float kappa[COLBANDIT_MAX_ROUNDS + 1] = {};      // radius per unit sigma_hat of each round
    for (int r = 1; r <= R; ++r) {
        const double kap = colbandit_radius_prefactor(alpha_ef, delta, T, N, r * kn.B < T ? r * kn.B : T);
        kappa[r] = isinf(kap) ? 0.f : (float)kap;    // unused by the kernels when n <= 1
    }
    DenseRule round_rule[COLBANDIT_MAX_ROUNDS + 2];
    for (int r = 0; r <= R + 1; ++r) round_rule[r] = kNeverDense;
    const bool share = loop && !cache_all && shares_documents(P, W, co);
    auto round_of = [&](int r) {
        RevealRound rr{};
        rr.r = r;
        rr.lo = (r - 1) * kn.B;
        rr.nb = (r * kn.B < T ? r * kn.B : T) - rr.lo;
        rr.n_prev = rr.lo;
        rr.n = rr.lo + rr.nb;
        rr.dense = kNeverDense;
        if (r == 1 || cache_all) return rr;
        if (dense && later_rounds != 2) {
            double t_pair = 0.0;
            int G = 1;
            while (G < rr.nb) G <<= 1;
            const unsigned long long thr = later_rounds == 1 ? 0ull
                : dense_pairs_threshold(P, G, co != nullptr, r, R, N <= (int64_t)W.cache_cap, &t_pair);
            if (thr < (unsigned long long)n_queries * (unsigned long long)N) rr.dense.thr = thr;
            // Round 2 by document: the corpus at 5.5 TB/s, and the documents again, from the last-level cache, for every
            // group of queries.
            if (r == 2 && share) {
                if (t_pair > 0.0) rr.dense.base = (uint32_t)fmin((double)P.total * P.d * (co ? 1.0 : 2.0) / 5.5e12 / t_pair, 4e9);
                rr.dense.lg_per = (uint16_t)(1 + share_group_lg(T));
                // Lists that fit the cache, and cost no more even if they are full (and those that are not entered by
                // document hold N pairs): it is the last round to launch.
                if (later_rounds != 1 && N <= (int64_t)W.cache_cap &&
                    rr.dense.base + (((unsigned long long)N * (unsigned)n_queries) >> rr.dense.lg_per) + (unsigned long long)N <= rr.dense.thr)
                    rr.dense.thr = NEVER_DENSE;
            }
        }
        if (r == 2 && share) {
            rr.dense.shared_at = (uint16_t)(2 * (R + 2) - 2);
            rr.dense.enough = share_enough(P);
        }
        return rr;
    };
    // A gathered round in which every list fits the cell cache is the last one to launch: k_select_prune runs all rounds
    // of a cached query.
    auto last_launched = [&](const RevealRound& rr) {
        return cache_all || (rr.r >= 2 && rr.dense.thr == NEVER_DENSE && N <= (int64_t)W.cache_cap);
    };
    // ... and, with exact cells, goes on to the top-K (cache_all: in round 1)
    const bool finish = !co && (cache_all || (loop && R >= 2 && last_launched(round_of(2))));
    for (int r = 1; e == hipSuccess && loop && r <= R; ++r) {
        const RevealRound rr = round_of(r);
        int G = 1;
        while (G < rr.nb) G <<= 1;
        round_rule[r] = rr.dense;
        if (r == 1 && dense) {
            e = launch_dense_reveal(P, W, n_chunks, rr, G, co, st);
        } else if (!cache_all) {
            e = launch_dense_reveal_later(P, W, n_chunks, rr, G, co, st);
            if (e == hipSuccess) e = launch_gather_round(P, W, rr, co, st);
        }
        pt.mark(r == 1 ? PH_FIRST_REVEAL : (r == 2 ? PH_ROUND2_REVEAL : PH_LATER_REVEAL));
        const bool last = last_launched(rr);
        const DenseRule next = share && r == 1 && R >= 2 ? round_of(2).dense : kNeverDense;
        if (e == hipSuccess) e = launch_select_prune(P, W, kn, rr, R, kappa, cache_all, cache_all && !cache_all_reveals(P, co), stats != nullptr, next,
                                                     finish && !last, tr, finish && last ? topk_ids : nullptr, topk_scores, st);
        pt.mark(PH_SELECT);
        if (last) break;
    }
    // exact rescore from the stored embeddings; cached cells give it only when they are exact
    // (where the last launched round has gathered every query's survivors, k_select_prune has gone on to the top-K).  Where no
    // round ran, all documents survive: shared by wavefronts only if they are few (296 documents of 18
    // tokens x 74 queries 86 -> 44 us a call)
    if (e == hipSuccess && !loop) e = launch_gather_all(P, W, W.rescored, nullptr, st);    // no round: all documents
    else if (e == hipSuccess && !finish) e = launch_gather_survivors(P, W, kn, W.rescored, co != nullptr, cache_all, st);
    if (e == hipSuccess && !finish) e = launch_topk(P, W, true, !co, cache_all, W.rescored, K, topk_ids, topk_scores, st);
    pt.mark(PH_RESCORE);
    if (e != hipSuccess) {
        pt.destroy();
        return COLBANDIT_ERR_HIP;
    }
    if (!stats) return COLBANDIT_OK;

    // statistics: the per-round survivor counts come back in one copy after the last kernel
    const size_t nh = (size_t)(R + 1) * n_queries;
    int32_t* hist = (int32_t*)malloc(sizeof(int32_t) * nh);
    if (!hist) { pt.destroy(); return COLBANDIT_ERR_HIP; }
    hipError_t ce = hipMemcpyAsync(hist, W.cnt_hist, sizeof(int32_t) * nh, hipMemcpyDeviceToHost, st);
    unsigned long long pairs_h[2 * (COLBANDIT_MAX_ROUNDS + 2) + 2];
    if (ce == hipSuccess)
        ce = hipMemcpyAsync(pairs_h, W.pairs, sizeof(unsigned long long) * (2 * (size_t)(R + 2) + 2),
                            hipMemcpyDeviceToHost, st);
    if (ce == hipSuccess) ce = hipStreamSynchronize(st);
    // the rounds whose device-side test took the corpus pass (the same test as the kernels')
    uint64_t corpus_rounds = 0;
    for (int r = 2; ce == hipSuccess && loop && r <= R; ++r)
        if (round_rule[r].pass(pairs_h[r], r == 2 ? pairs_h[2 * (R + 2)] : 0ull)) corpus_rounds |= 1ull << (r - 1);
    float ms = 0.f, phase_ms[PH_COUNT] = {0.f, 0.f, 0.f, 0.f, 0.f};
    if (ce == hipSuccess) pt.collect(phase_ms, ms);
    pt.destroy();
    if (ce != hipSuccess) { free(hist); return COLBANDIT_ERR_HIP; }
    for (int q = 0; q < n_queries; ++q) {
        colbandit_stats& s = stats[q];
        memset(&s, 0, sizeof(s));
        s.survivors[0] = (int32_t)N;
        int64_t count = N;
        int n = 0, r = 0;
        bool cached = false;        // the query's list holds cache slots (its cells are cached)
        while (loop && count > (int64_t)K + M && r * kn.B < T) {   // the loop condition of Algorithm 1
            const int lo = r * kn.B, hi = (r + 1) * kn.B < T ? (r + 1) * kn.B : T;
            s.cells_elim += (int64_t)(hi - lo) * count;
            // cells COMPUTED for this round: a corpus pass (round 1 always covers all N documents)
            // computes the batch for every document; the first gathered round of a list that fits
            // the cache computes all T cells of its documents once, later rounds read them back
            const bool pass = r == 0 || ((corpus_rounds >> r) & 1ull);
            if (!cached) {
                if (cache_all) {                      // round 1 computed all cells of all documents
                    s.cells_computed += (int64_t)T * N;
                    cached = true;
                } else if (pass) s.cells_computed += (int64_t)(hi - lo) * N;
                else if (W.cache_cap > 0 && count <= W.cache_cap) {
                    s.cells_computed += (int64_t)T * count;
                    cached = true;
                } else s.cells_computed += (int64_t)(hi - lo) * count;
            }
            n = hi;
            ++r;
            count = hist[(size_t)r * n_queries + q];
            s.survivors[r] = (int32_t)count;
        }
        s.rounds = r;
        s.cells_rescore = (int64_t)T * count;
        s.cells_unique = s.cells_elim + (int64_t)(T - n) * count;
        if (!cached || co) s.cells_computed += (int64_t)T * count;   // the rescore gathers the survivors
        s.ms_total = ms;
        s.ms_first_reveal = phase_ms[PH_FIRST_REVEAL];
        s.ms_later_reveals = phase_ms[PH_LATER_REVEAL] + phase_ms[PH_ROUND2_REVEAL];
        s.ms_reveal_round2 = phase_ms[PH_ROUND2_REVEAL];
        s.ms_select_prune = phase_ms[PH_SELECT];
        s.ms_rescore_topk = phase_ms[PH_RESCORE];
        s.corpus_pass_rounds = corpus_rounds;
        s.pairs_round2 = R >= 2 ? pair_count(pairs_h[2]) + pair_count(pairs_h[2 * (R + 2)]) - pairs_h[2 * (R + 2) + 1] : 0ull;
        s.tokens_round2 = R >= 2 ? pairs_h[(R + 2) + 2] : 0ull;
    }
    free(hist);
    return COLBANDIT_OK;
}

int colbandit_topk(const void* Q, int n_queries, int T, int d, colbandit_dtype dt,
                   const void* doc_tokens, const int64_t* doc_offsets, int64_t N,
                   int64_t total_tokens, int K, float alpha_ef, float delta, int M, uint64_t seed,
                   const colbandit_opts* opts, int64_t* topk_ids, float* topk_scores,
                   colbandit_stats* stats, void* workspace, size_t workspace_bytes,
                   void* stream) {
    return topk_impl(Q, n_queries, T, d, dt, doc_tokens, doc_offsets, N, total_tokens, K, alpha_ef,
                     delta, M, seed, opts, topk_ids, topk_scores, stats, workspace, workspace_bytes,
                     false, stream);
}

int colbandit_topk_static(const void* Q, int n_queries, int T, int d, colbandit_dtype dt,
                          const void* doc_tokens, const int64_t* doc_offsets, int64_t N,
                          int64_t total_tokens, int K, float alpha_ef, float delta, int M,
                          uint64_t seed, const colbandit_opts* opts, int64_t* topk_ids,
                          float* topk_scores, void* stream) {
    // stats == NULL: kernel launches only (no events, no host allocation, no read-back)
    return topk_impl(Q, n_queries, T, d, dt, doc_tokens, doc_offsets, N, total_tokens, K, alpha_ef,
                     delta, M, seed, opts, topk_ids, topk_scores, nullptr, nullptr, 0, true, stream);
}

}  // extern "C"
