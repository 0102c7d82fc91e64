// Gather-reveal / rescore kernel, bound-driven selection and pruning, top-K, and the
// small control kernels.  gfx950 only.
#include <type_traits>

#include "../../include/colbandit.h"
#include "cb_launch.h"
#include "cb_segments.h"

namespace cb {

// =====================================================================================
// init: per-query control, reveal permutations, history and trace fill
// =====================================================================================
__device__ __forceinline__ uint64_t splitmix64_next(uint64_t& s) {
    s += 0x9E3779B97F4A7C15ull;
    uint64_t z = s;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Round 2's lists by document: held[id] queries hold document id, at holders[id * nq ..] in any order, as query and list
// place.  They lie over stat2, two words a pair, which else only corpus passes of later rounds use.
__device__ __host__ __forceinline__ const int* held_of(const float2* stat2, int nq, int64_t N) {
    return (const int*)stat2 + (size_t)nq * (size_t)N;
}

struct InitArgs {
    QueryCtl* ctl;
    int32_t* pi;
    const int32_t* user_pi;
    int32_t* cnt_hist;
    float* tau_hist;
    int nq, T, R, KM;
    int64_t N;
    uint64_t seed;
    int32_t* tr_count;
    float* tr_tau;
    unsigned long long* pairs;
    int init_blocks;          // workgroups of four queries; those after them fill the chunk table
    const int64_t* off;
    int chunk_tokens, n_chunks;
    int32_t* chunk_doc;
    int chunk_blocks;         // workgroups of the chunk table; those after them clear `held`
    int* held;
};

// The reveal order of query q, a Fisher-Yates shuffle driven by SplitMix64 (Sec. 4.2: one seeded uniform permutation per
// query): lane x gets the tokens at places x and x + 64.  The generator's state after s steps is known in closed form, so
// the lanes draw the T - 1 positions side by side; a place's token is found by following the place back through the
// exchanges, five instructions each.  (One thread drawing and exchanging them in turn took 14 us, T = 32.)
// What the draws need of the lane alone is worked out in place: the compiler would keep it, some 18 registers, over a
// caller's loop, which k_cache_all has not (fp32, d = 128, T = 32 two wavefronts a SIMD fell to one: 1 query x 4,000
// documents of 17 tokens 59 us so and 47, 8 x 1,000 of 9 80 and 60).
__device__ __forceinline__ void reveal_order(uint64_t seed, int q, int T, int& p0, int& p1) {
    int lane = threadIdx.x & 63;
    asm("" : "+v"(lane) : "s"(q));
    const uint64_t s0 = seed + ((uint64_t)q + 1ull) * 0x9E3779B97F4A7C15ull;
    auto draw = [&](int i) -> int {                 // the position that i is exchanged with: step T - i
        uint64_t s = s0 + (uint64_t)(T - 1 - i) * 0x9E3779B97F4A7C15ull;
        const uint64_t z = splitmix64_next(s);
        const uint32_t m = (uint32_t)i + 1u;        // z mod m, at most 128: in halves
        const uint32_t high = (uint32_t)(z >> 32) % m * ((0u - m) % m);
        return (int)((high + (uint32_t)z % m) % m);
    };
    int j0 = 0, j1 = 0;
    if (lane >= 1 && lane < T) j0 = draw(lane);
    if (lane + 64 < T) j1 = draw(lane + 64);
    p0 = lane;
    p1 = lane + 64;
    for (int i = 1; i < T && i < 64; ++i) {
        const int j = __builtin_amdgcn_readlane(j0, i);
        p0 = p0 == i ? j : p0 == j ? i : p0;        // (places from 64 on are not reached yet)
    }
    for (int i = 64; i < T; ++i) {
        const int j = __builtin_amdgcn_readlane(j1, i - 64);
        p0 = p0 == i ? j : p0 == j ? i : p0;
        p1 = p1 == i ? j : p1 == j ? i : p1;
    }
}

// A wavefront per query, the chunk table of the corpus passes by other workgroups.
__device__ __forceinline__ void init_queries(const InitArgs& A, int block) {
    const int lane = threadIdx.x & 63;
    const int q = block * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (q == 0)                                     // pair counts, their token counts, shared and finished pairs
        for (int r = lane; r < 2 * (A.R + 2) + 2; r += 64) A.pairs[r] = 0ull;
    if (q >= A.nq) return;
    const int T = A.T;
    if (lane == 0) {
        QueryCtl c;
        c.count = (int)A.N;
        c.cur = 0;
        c.implicit = 1;
        c.active = A.N > (int64_t)A.KM;
        c.mode = 0;
        c.bound = c.done = c.pad = 0;
        A.ctl[q] = c;
    }
    for (int r = lane; r <= A.R; r += 64) {
        A.cnt_hist[r * A.nq + q] = (int)A.N;
        if (A.tr_count) A.tr_count[r * A.nq + q] = (int)A.N;
        if (r < A.R) {
            A.tau_hist[r * A.nq + q] = __uint_as_float(0x7fc00000u);   // quiet NaN: "round not run"
            if (A.tr_tau) A.tr_tau[r * A.nq + q] = __uint_as_float(0x7fc00000u);
        }
    }
    int32_t* p = A.pi + (size_t)q * T;
    if (A.user_pi) {
        for (int t = lane; t < T; t += 64) {        // clamped: a bad table must not steer a read out of Q
            const int32_t v = A.user_pi[(size_t)q * T + t];
            p[t] = v < 0 ? 0 : (v >= T ? T - 1 : v);
        }
        return;
    }
    int p0, p1;
    reveal_order(A.seed, q, T, p0, p1);
    if (lane < T) p[lane] = p0;
    if (lane + 64 < T) p[lane + 64] = p1;
}
__global__ __launch_bounds__(256) void k_init(InitArgs A) {
    const int block = (int)blockIdx.x - A.init_blocks;
    if (block < 0) init_queries(A, (int)blockIdx.x);
    else if (block < A.chunk_blocks)
        chunk_docs((int64_t)block * 256 + threadIdx.x, A.off, A.N, A.chunk_tokens, A.n_chunks, A.chunk_doc);
    else {
        const int64_t i = (int64_t)(block - A.chunk_blocks) * 256 + threadIdx.x;
        if (i < A.N) A.held[i] = 0;
    }
}

__global__ void k_fill_f32(float* p, size_t n, float v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_u8(uint8_t* p, size_t n, uint8_t v) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

static InitArgs init_args(const Problem& P, const Work& W, const Knobs& kn, int R, uint64_t seed,
                          const int32_t* user_pi, const Trace& tr, int n_chunks) {
    InitArgs A{};
    A.ctl = W.ctl;
    A.pi = W.pi;
    A.user_pi = user_pi;
    A.cnt_hist = W.cnt_hist;
    A.tau_hist = W.tau_hist;
    A.nq = P.nq;
    A.T = P.T;
    A.R = R;
    A.KM = kn.K + kn.M;
    A.N = P.N;
    A.seed = seed;
    A.tr_count = tr.count;
    A.tr_tau = tr.tau;
    A.pairs = W.pairs;
    A.init_blocks = (P.nq + 3) / 4;
    A.off = P.off;
    A.chunk_tokens = W.chunk_tokens;
    A.n_chunks = n_chunks;
    A.chunk_doc = W.chunk_doc;
    return A;
}
static void fill_trace(const Problem& P, int R, const Trace& tr, hipStream_t st) {
    if (!tr.lcb) return;
    const size_t n = (size_t)R * P.nq * P.N;
    const int g = (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    k_fill_f32<<<g, 256, 0, st>>>(tr.lcb, n, __builtin_nanf(""));
    k_fill_f32<<<g, 256, 0, st>>>(tr.ucb, n, __builtin_nanf(""));
    k_fill_u8<<<g, 256, 0, st>>>(tr.alive, n, 0);
}

constexpr int SHARE_TOKENS = 256;
bool shares_documents(const Problem& P, const Work& W, const Coarse* co) {
    return (co || P.dt == DT_BF16) && W.cache_cap > 0 && P.nq >= 4 && P.total >= SHARE_TOKENS * P.N;
}
// Half as many as documents; 4,096 for a corpus of few, whose pairs fill the chip better than its documents.
unsigned share_enough(const Problem& P) { return (unsigned)(P.N > 8192 ? P.N / 2 : 4096); }
int share_group_lg(int T) { return T <= 16 ? 3 : T <= 32 ? 2 : T <= 64 ? 1 : 0; }
hipError_t launch_init(const Problem& P, const Work& W, const Knobs& kn, int R, uint64_t seed,
                       const int32_t* user_pi, const Trace& tr, const Coarse* co, int n_chunks, hipStream_t st) {
    InitArgs A = init_args(P, W, kn, R, seed, user_pi, tr, n_chunks);
    A.chunk_blocks = n_chunks > 0 ? (int)((P.N + 1 + 255) / 256) : 0;
    int64_t blocks = A.init_blocks + A.chunk_blocks;
    if (shares_documents(P, W, co)) {
        A.held = (int*)held_of(W.stat2, P.nq, P.N);
        blocks += (P.N + 255) / 256;
    }
    k_init<<<(unsigned)blocks, 256, 0, st>>>(A);
    fill_trace(P, R, tr, st);
    return hipGetLastError();
}

// =====================================================================================
// gather kernels: (query, document) pairs, each document read from memory for its own query.
//
// A wavefront keeps the query rows it needs as B operands in registers, streams document tokens
// from global memory in blocks of 16 rows (A operand, rows past the end of the document repeat its
// last token, which cannot change a max), runs the MFMA chain over d and folds the 16x16 result
// into a running per-column maximum.
//   k_gather_round     the reveal of one round (Algorithm 1, reveal step), see there
//   k_gather_docs      the same, a document for several queries at once
//   k_gather_survivors exact scores of the survivors (Eq. (2); rescore)
//   k_gather_all       all documents of all queries: the smallest calls, fp32 where it beats the corpus
//                      pass, Ball-carving in fp32 and in the widths without a group pass
// =====================================================================================
struct GatherArgs {
    const void* Q;
    const void* docs;
    const int64_t* off;
    int64_t N, total;
    int nq, T;
    const QueryCtl* ctl;
    int32_t* list0;
    int32_t* list1;
    // reveal
    const int32_t* pi;
    int lo, nb, n_prev, G;
    float2* stat;
    const unsigned long long* pairs_r;   // pairs of the round (pair_count); nullptr: all N documents of
                                         // every query
    const unsigned long long* work;      // its queries (work_item)
    DenseRule dense;
    // cell cache
    int cache_all;            // slots are documents (k_cache_all)
    int cache_cap, TP;
    int32_t* cid;
    float2* cstat;
    float* ccell;
    // k_gather_docs: stat2 (hold_documents)
    const float2* holders;
    // score
    float* out;
    float* cells;
    int shared;               // k_gather_all: the wavefronts of a workgroup share a document (gather_shares)
    int score_slots;          // also serve queries whose list holds cache slots
    // int8 codes: a cell is the integer maximum times qscale[q] * dscale[0]
    const float* qscale;
    const float* dscale;
};

// Registers of a gather kernel with NT tiles of query rows and one block at work, and wavefronts per
// SIMD that leaves.
template <int NT, class F> constexpr int gather_regs(bool ahead) {
    return (NT + 1) * ((int)sizeof(F) / 4) + (ahead ? (int)sizeof(typename F::Raw) / 4 + 8 * NT : 36);
}
constexpr int waves_of(int regs) { return 512 / regs < 4 ? 512 / regs : 4; }
// fp32: a block is cut into its pieces after it was read
template <class F> constexpr bool cuts() { return !__is_same(typename F::Raw, F); }
// Whether a second block of a document is in flight.  bf16 and codes: where its registers do not cost a wavefront
// per SIMD.
// fp32: in the kernels that only score, always, held to the wavefronts that its registers leave (one query x
// 200 documents of 1,030 tokens in d = 96, T = 32: 28.5 -> 24.0 us, T = 48 35.3 -> 30.0; d = 64 23.9 -> 19.2); in those of
// a round, which need 48 more, where that costs no wavefront: d = 128 and T <= 16 took 197, two
// wavefronts (20,000 documents x 4 queries, Col-Bandit, 267 -> 257 us; held to three they spill), while one block in flight
// cost 5,000 documents x 60 queries of 32 tokens 491 us in the place of 488, of 64 tokens 515 and 512.
template <int NT, class F> constexpr bool score_ahead() { return cuts<F>() || gather_regs<NT, F>(true) <= 112; }
template <int NT, class F> constexpr bool round_ahead() {
    return cuts<F>() ? waves_of(gather_regs<NT, F>(true) + 48) >= waves_of(gather_regs<NT, F>(false) + 16)
                     : gather_regs<NT, F>(true) <= 112;
}
template <int TQ, class F> constexpr int score_waves() { return cuts<F>() ? waves_of(gather_regs<TQ, F>(true)) : 1; }
// Wavefronts per SIMD of k_gather_round, which serves two kinds of list and without a bound takes a few
// registers too many for the four (or what the query rows leave) that a kernel with one block in
// flight needs (T = 48, 50,000 documents x 16 queries 1,645 -> 1,546 us a call, T = 100 and d = 96, 20,000
// x 16 1,005 -> 908).
// fp32 needs some for a block on its way from what was read to its pieces.
template <int TQ, class F> constexpr int round_waves() {
    return round_ahead<TQ, F>() ? 1 : waves_of(gather_regs<TQ, F>(false) + (cuts<F>() ? 16 : 0));
}

// Folds the blocks first, first + stride, ... of the document [o0, o1) into h.
template <int ROWB, bool AHEAD, int NT, class F>
__device__ __forceinline__ void fold_doc(const char* docs, int64_t o0, int64_t o1, int first, int stride,
                                         int col, int kg, const F (&bq)[NT], bool query_wild,
                                         typename F::val_t (&h)[NT]) {
    int64_t r0 = o0 + 16 * first;
    if (r0 >= o1) return;
    using R = typename F::Raw;
    auto load = [&](R& a, int64_t r) {
        int64_t row = r + col;
        row = row < o1 ? row : o1 - 1;
        a.load(docs + (size_t)row * ROWB, kg);
    };
    R raw;
    load(raw, r0);
    for (;;) {
        const int64_t r1 = r0 + 16 * stride;
        const bool more = r1 < o1;
        F a;
        const bool wild = __ballot(a.from(raw)) != 0ull || query_wild;
        R next;
        if (AHEAD && more) load(next, r1);
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
            typename F::acc_t acc = {0, 0, 0, 0};
            F::mma(acc, a, bq[tt], wild);
            h[tt] = fold_max(h[tt], acc);
        }
        if (!more) return;
        if (AHEAD) raw = next;
        else load(raw, r1);
        r0 = r1;
    }
}

// Cross-lane column maxima of one document, decoded to float cells.  parts > 1: the four
// wavefronts of the workgroup hold maxima of different blocks of it, which are combined through
// `ex`; then only wavefront 0's result counts.  Two barriers (parts > 1 is uniform).
constexpr int EX_FLOATS = 3 * 2 * 64;
template <int NT, class V>
__device__ __forceinline__ void doc_cells(const V (&h)[NT], int parts, float scale, int* ex,
                                          float (&w)[Pack<NT>::NW]) {
    using P = Pack<NT>;
    V wi[P::NW];
    P::colmax(h, wi);
    if (parts > 1) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (wave > 0) {
#pragma unroll
            for (int j = 0; j < P::NW; ++j) ex[((wave - 1) * P::NW + j) * 64 + lane] = __builtin_bit_cast(int, wi[j]);
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int j = 0; j < P::NW; ++j)
                    wi[j] = vmax(wi[j], __builtin_bit_cast(V, ex[(s * P::NW + j) * 64 + lane]));
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < P::NW; ++j) {
        if constexpr (__is_same(V, float)) w[j] = wi[j];
        else w[j] = (float)wi[j] * scale;
    }
}

__device__ __forceinline__ void doc_range(const GatherArgs& A, int id, int64_t& o0, int64_t& o1) {
    o0 = A.off[id];
    o1 = A.off[id + 1];
    o0 = o0 < 0 ? 0 : (o0 > A.total ? A.total : o0);
    o1 = o1 < o0 ? o0 : (o1 > A.total ? A.total : o1);
}

// the T rows of a query as the B operands of TQ column tiles; whether any of their values is wild (Frag)
template <class F, int ROWB, int TQ>
__device__ __forceinline__ bool load_query(const GatherArgs& A, int q, int col, int kg, F (&bq)[TQ]) {
    const char* Qq = (const char*)A.Q + (size_t)q * A.T * ROWB;
    bool wild = false;
#pragma unroll
    for (int tt = 0; tt < TQ; ++tt) {
        const int t = tt * 16 + col;
        wild |= bq[tt].load(Qq + (size_t)(t < A.T ? t : 0) * ROWB, kg);
    }
    return __ballot(wild) != 0ull;
}

// Inclusive sum over the wavefront's lanes, in lane order (DPP: shifts by 1, 2, 4, 8 inside the
// rows of 16 lanes, then the rows' totals are passed on).
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return v;
}

// The T cells of query q's k-th document to its cache slot.
template <int TQ>
__device__ __forceinline__ void store_cells(const GatherArgs& A, int q, int k, const float (&w)[Pack<TQ>::NW]) {
    using P = Pack<TQ>;
    const int row = (int)(threadIdx.x & 63) >> 4, col = threadIdx.x & 15;
    float* crow = A.ccell + ((size_t)q * A.cache_cap + k) * A.TP;
#pragma unroll
    for (int j = 0; j < P::NW; ++j)
        if (P::row_is_primary(row)) crow[P::tile_of_row(j, row) * 16 + col] = w[j];
}
// This round's batch of the same cells, merged into the pair's statistics, which go to the slot.  t: the batch's
// query token of this lane; slot s of the batch (lane s of row 0) fetches its cell from its owner.  NAMED: slots are places
// of a list; else documents, before round 1, so that there are no statistics yet.
template <int TQ, bool NAMED = true>
__device__ __forceinline__ void reveal_cached(const GatherArgs& A, int q, int k, int id, int t, const float (&w)[Pack<TQ>::NW]) {
    using P = Pack<TQ>;
    const int lane = threadIdx.x & 63;
    const int tile = t >> 4;
    const int src = P::row_of_tile(tile) * 16 + (t & 15);
    float v = __shfl(w[0], src);
    if constexpr (P::NW > 1) {
        const float v1 = __shfl(w[1], src);
        v = tile >= 4 ? v1 : v;
    }
    float sb, m2b;
    batch_stats(v, (lane & 15) % A.G, A.nb, A.G, sb, m2b);
    if (lane == 0) {
        const size_t slot = (size_t)q * A.cache_cap + k;
        float2 st = make_float2(sb, m2b);
        if constexpr (NAMED) {
            st = make_float2(0.f, 0.f);
            if (A.n_prev > 0) st = A.stat[(size_t)q * A.N + id];
            merge_stats(st.x, st.y, A.n_prev, sb, m2b, A.nb);
            A.cid[slot] = id;
        }
        A.cstat[slot] = st;
    }
}

constexpr int64_t ALL_DOCS = 64;

// One round's reveal.  The round's pairs (over all queries that hold ids) are spread evenly over
// the grid whatever the lengths of the lists: worker w of W takes pairs [w * per, (w + 1) * per).  Up
// to one pair per workgroup, the four wavefronts share the pair's blocks (few pairs: the
// time is the latency of one document: 64 queries x 9 pairs of 106 tokens 30 -> 9 us); beyond, each
// wavefront takes pairs of its own.  Workers of more than one pair take their places in as many
// streams as there are queries, so that lists that share documents, ascending all, read them at about
// the same time: 8 queries x 100,000 documents of 106 tokens, alpha 0.5, 5,530 -> 5,090 us a call,
// 4 x 16,048 of 1,000 3,450 -> 3,080; with a pair each nothing is divided, which the rounds without
// pairs feel most (7 queries x 6,007 documents 150 -> 143 us a call).
// What happens to a pair depends on its query:
//   list longer than the cell cache   one 16-column tile, column c < nb is query token pi[lo+c]; the
//                  epilogue merges the batch into the pair's (sum, M2).
//   list that fits the cell cache     TQ tiles = all T tokens; the epilogue stores the pair's T
//                  cells in the query's cell cache (slot = place in the list) and merges this round's batch
//                  from them.  A gathered reveal is bound by the bytes of the
//                  document, not by the cells computed from them, so a document is visited once
//                  and the later rounds (and the rescore) read its cells back; the order in which
//                  cells are REVEALED to the bounds is unchanged.  cache_all: the smallest calls visit all
//                  documents so before round 1, which takes its batch from the cells as well; the
//                  launch also sets the queries up, which nothing in it needs, and two launches make
//                  the call (1 query x 1,000 documents of 48 fp32 tokens: 45 -> 39 us; 25 to 33, by the inputs, since
//                  round 1 is revealed there, cache_all_reveals).
// batch_token(q): this lane's token of the round's batch (REVEAL).
template <typename Tag, int D, int TQ, bool CACHE_ALL, bool REVEAL, class TokenFn>
__device__ __forceinline__ void gather_round(const GatherArgs& A, int n_blocks, TokenFn batch_token) {
    using F = Frag<Tag, D>;
    using V = typename F::val_t;
    constexpr int ROWB = D * F::ELEM_BYTES;
    __shared__ int ex[EX_FLOATS];
    // The round's items: those of pairs_r, then, from the end of the array, those entered by document if k_gather_docs
    // does not serve them.
    unsigned long long head = (unsigned long long)A.nq * (unsigned long long)A.N, shared = 0ull;
    if (!CACHE_ALL && A.pairs_r) {
        head = *A.pairs_r;
        if (A.dense.enough) shared = A.pairs_r[A.dense.shared_at];
        if ((head | shared) == 0ull || A.dense.pass(head, shared)) return;   // no pairs, or the corpus pass serves the round
        if (A.dense.enough && A.dense.by_document(shared)) shared = 0ull;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15;
    const int kg = lane >> 4;

    const int n_own = (int)work_count(head);
    const long long total = (long long)(A.pairs_r ? pair_count(head) + pair_count(shared) : head);
    const int n_work = A.pairs_r ? n_own + (int)work_count(shared) : A.nq;
    auto item_at = [&](int i) {
        return i < n_own ? A.work[i] : A.work[A.nq - 1 - (i - n_own)] + (pair_count(head) << 16);
    };
    const bool coop = total <= (long long)n_blocks;
    const int parts = coop ? 4 : 1;
    const long long workers = coop ? n_blocks : 4ll * n_blocks;
    int me = coop ? (int)blockIdx.x : (int)blockIdx.x * 4 + wave;
    if (me >= total) return;                        // in shared mode the same for the whole workgroup
    long long per = 1;
    if (total > workers) {
        per = (total + workers - 1) / workers;
        if (A.pairs_r) {
            const int rows = (int)((total + per - 1) / per) / n_work;
            if (me < rows * n_work) me = me % n_work * rows + me / n_work;
        }
    }
    long long x = me * per;
    const long long x_end = x + per < total ? x + per : total;
    if (x >= x_end) return;

    // the last query whose first pair is not beyond x: 64 probes at a time
    int item = 0;
    if (A.pairs_r) {
        int n = n_work;
        while (n > 1) {
            const int step = (n + 63) / 64;
            const bool in = lane * step < n;
            const long long s = in ? (long long)work_start(item_at(item + lane * step)) : 0;
            const int hit = __popcll(__ballot(in && s <= x));       // >= 1: the item at hand starts at or before x
            item += (hit - 1) * step;
            n -= (hit - 1) * step;
            n = n < step ? n : step;
        }
    }
    // round 1: all documents of all queries, ALL_DOCS of them for every query in turn, so that the
    // queries that read a document do so at about the same time
    int64_t block = 0, block_docs = 0;
    auto at_block = [&](int64_t b) {
        block = b;
        block_docs = A.N - b * ALL_DOCS < ALL_DOCS ? A.N - b * ALL_DOCS : ALL_DOCS;
    };
    if (!A.pairs_r) {
        at_block(x / (ALL_DOCS * A.nq));
        item = (int)((x - block * ALL_DOCS * A.nq) / block_docs);
    }

    for (; x < x_end; ++item) {
        int q, k, k_end;
        if (A.pairs_r) {
            const unsigned long long it = item_at(item);
            q = work_query(it);
            const long long first = (long long)work_start(it);
            const int n = A.ctl[q].count;
            k = (int)(x - first);
            k_end = x_end - first < n ? (int)(x_end - first) : n;
        } else {
            if (item == A.nq) {
                at_block(block + 1);
                item = 0;
            }
            q = item;
            const long long first = block * ALL_DOCS * A.nq + item * block_docs;   // pair of the block's first document
            const int64_t d0 = block * ALL_DOCS;
            k = (int)(d0 + (x - first));
            k_end = (int)(d0 + (x_end - first < block_docs ? x_end - first : block_docs));
        }
        x += k_end - k;
        int count = 0;
        int32_t* list = nullptr;
        if (!CACHE_ALL) {
            const QueryCtl c = A.ctl[q];
            count = c.count;
            if (!c.implicit) list = (c.cur ? A.list1 : A.list0) + (size_t)q * A.N;
        }
        const float scale = A.qscale ? A.qscale[q] * A.dscale[0] : 1.f;
        if (!CACHE_ALL && (!list || count > A.cache_cap)) {
            F bq[1];
            const int trow = A.pi[(size_t)q * A.T + A.lo + (col < A.nb ? col : 0)];
            const bool query_wild = __ballot(bq[0].load((const char*)A.Q + ((size_t)q * A.T + trow) * ROWB, kg)) != 0ull;
            for (; k < k_end; ++k) {
                const int id = list ? list[k] : k;
                int64_t o0, o1;
                doc_range(A, id, o0, o1);
                V h[1] = {lowest_val<V>()};
                fold_doc<ROWB, round_ahead<1, F>()>((const char*)A.docs, o0, o1, coop ? wave : 0, parts, col, kg, bq, query_wild, h);
                float w[1];
                doc_cells(h, parts, scale, ex, w);
                float sb, m2b;
                batch_stats(w[0], col % A.G, A.nb, A.G, sb, m2b);
                if (lane == 0 && (!coop || wave == 0)) {
                    const size_t at = (size_t)q * A.N + id;
                    float2 st = make_float2(0.f, 0.f);
                    if (A.n_prev > 0) st = A.stat[at];
                    merge_stats(st.x, st.y, A.n_prev, sb, m2b, A.nb);
                    A.stat[at] = st;
                }
            }
        } else {
            F bq[TQ];
            const bool query_wild = load_query<F, ROWB, TQ>(A, q, col, kg, bq);
            const int t = REVEAL ? batch_token(q) : 0;
            for (; k < k_end; ++k) {
                const int id = list ? list[k] : k;
                int64_t o0, o1;
                doc_range(A, id, o0, o1);
                V h[TQ];
#pragma unroll
                for (int tt = 0; tt < TQ; ++tt) h[tt] = lowest_val<V>();
                fold_doc<ROWB, round_ahead<TQ, F>()>((const char*)A.docs, o0, o1, coop ? wave : 0, parts, col, kg, bq, query_wild, h);
                float w[Pack<TQ>::NW];
                doc_cells(h, parts, scale, ex, w);
                if (coop && wave > 0) continue;
                store_cells<TQ>(A, q, k, w);
                if (REVEAL) reveal_cached<TQ, !CACHE_ALL>(A, q, k, id, t, w);
            }
        }
    }
}

// The same reveal of round 2, document by document, where many documents are long and held by several queries: a
// wavefront (a workgroup of its own: they take different times) takes a document, reads once the list of the queries
// that hold it (k_select_prune has entered them, hold_documents) and multiplies it with the rows of up to NQ of them at a
// time, so that it is read once for those.  Bound by memory: 64 queries of T = 24 x 20,000 pages of 1,030 tokens, 62,900
// pairs on some 19,200 documents: 1.07 ms for 5.1 GB of documents, 6.3 with those read again for a fifth query on, of
// which HBM delivers all (by its counters, 5.9 TB/s; 1.05 to 1.25 ms on other machines and inputs), in the place of a second
// corpus pass of 1.15 and gathers of 0.5.  (A workgroup of four wavefronts per run of documents,
// two queries and one block ahead each: 1.57; each wavefront searching the lists for its document: 1.29; three blocks in
// flight as four; tokens with the non-temporal hint: 1.45, the documents read again miss the caches.)  The query rows of
// eight tiles and the blocks fill the 256 registers of two wavefronts a SIMD: in bf16 at d = 128, queries of 33 to 64
// tokens put 3 in scratch memory and longer ones 11, outside the loop over a document's blocks.
template <int TQ> constexpr int share_queries() { return 8 / TQ; }
// blocks in flight: 64 registers
template <class F> constexpr int share_depth() { return 64 / ((int)sizeof(F) / 4) < 8 ? 64 / ((int)sizeof(F) / 4) : 8; }

// Folds the document [o0, o1) into h, DEPTH blocks in flight.  The last block is repeated up to a multiple of DEPTH.
template <int ROWB, int DEPTH, int NT, class F>
__device__ __forceinline__ void fold_long_doc(const char* docs, int64_t o0, int64_t o1, int col, int kg,
                                              const F (&bq)[NT], typename F::val_t (&h)[NT]) {
    const int n = (int)((o1 - o0 + 15) >> 4);
    if (n <= 0) return;
    F a[DEPTH];
    auto load = [&](F& x, int b) {
        b = b < n ? b : n - 1;
        int64_t row = o0 + 16 * (int64_t)b + col;
        row = row < o1 ? row : o1 - 1;
        x.load(docs + (size_t)row * ROWB, kg);
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) {               // the order of the loads is that in which they are waited for
        __builtin_amdgcn_sched_barrier(0);
        load(a[i], i);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int b = 0; b < n; b += DEPTH) {
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            block_mma<NT>(a[i], bq, h, false);
            load(a[i], b + i + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("" ::: "memory");              // else the compiler moves the loads into the next turn, to their use
    }
}

template <typename Tag, int D, int TQ>
__global__ __launch_bounds__(64, 2) void k_gather_docs(GatherArgs A) {
    using F = Frag<Tag, D>;
    using V = typename F::val_t;
    constexpr int ROWB = D * F::ELEM_BYTES;
    constexpr int NQ = share_queries<TQ>();
    const unsigned long long shared = A.pairs_r[A.dense.shared_at];
    if (!A.dense.by_document(shared) || A.dense.pass(*A.pairs_r, shared)) return;
    const int lane = threadIdx.x;
    const int col = lane & 15;
    const int kg = lane >> 4;
    for (int id = (int)blockIdx.x; id < (int)A.N; id += (int)gridDim.x) {
        const uint32_t* holders = (const uint32_t*)A.holders + (size_t)id * A.nq;
        const int m = (int)held_of(A.holders, A.nq, A.N)[id];
        int64_t o0, o1;
        doc_range(A, id, o0, o1);
        for (int at = 0; at < m; at += NQ) {
            const int left = m - at;
            auto visit = [&](auto queries) {        // that many queries; past `left` the last one again
                constexpr int M = decltype(queries)::value;
                int q[M], k[M], t[M];
                F bq[M * TQ];
#pragma unroll
                for (int i = 0; i < M; ++i) {
                    const uint32_t x = holders[at + (i < left ? i : left - 1)];
                    q[i] = (int)(x >> 14);
                    k[i] = (int)(x & 16383u);
                    F rows[TQ];
                    load_query<F, ROWB, TQ>(A, q[i], col, kg, rows);
#pragma unroll
                    for (int tt = 0; tt < TQ; ++tt) bq[i * TQ + tt] = rows[tt];
                    t[i] = A.pi[(size_t)q[i] * A.T + A.lo + (lane < A.nb ? lane : 0)];
                }
                V h[M * TQ];
#pragma unroll
                for (int tt = 0; tt < M * TQ; ++tt) h[tt] = lowest_val<V>();
                fold_long_doc<ROWB, share_depth<F>()>((const char*)A.docs, o0, o1, col, kg, bq, h);
#pragma unroll
                for (int i = 0; i < M; ++i)
                    if (i < left) {
                        V hq[TQ];
#pragma unroll
                        for (int tt = 0; tt < TQ; ++tt) hq[tt] = h[i * TQ + tt];
                        float w[Pack<TQ>::NW];
                        doc_cells(hq, 1, A.qscale ? A.qscale[q[i]] * A.dscale[0] : 1.f, nullptr, w);
                        store_cells<TQ>(A, q[i], k[i], w);
                        reveal_cached<TQ>(A, q[i], k[i], id, t[i], w);
                    }
            };
            if (NQ >= 8 && left > 4) visit(std::integral_constant<int, NQ < 8 ? 1 : 8>{});
            else if (NQ >= 4 && left > 2) visit(std::integral_constant<int, NQ < 4 ? 1 : 4>{});
            else if (NQ >= 2 && left > 1) visit(std::integral_constant<int, NQ < 2 ? 1 : 2>{});
            else visit(std::integral_constant<int, 1>{});
        }
    }
}

template <typename Tag, int D, int TQ>
__global__ __launch_bounds__(256, (round_waves<TQ, Frag<Tag, D>>())) void k_gather_round(GatherArgs A) {
    gather_round<Tag, D, TQ, false, true>(A, (int)gridDim.x, [&](int q) {
        const int lane = threadIdx.x & 63;
        return A.pi[(size_t)q * A.T + A.lo + (lane < A.nb ? lane : 0)];
    });
}
// (a kernel of its own: the longer argument list cost every launch of a round 1 us)
template <typename Tag, int D, int TQ, bool REVEAL>
__global__ __launch_bounds__(256, (round_waves<TQ, Frag<Tag, D>>())) void k_cache_all(GatherArgs A, InitArgs I) {
    const int n_blocks = (int)gridDim.x - I.init_blocks;
    if ((int)blockIdx.x < n_blocks) gather_round<Tag, D, TQ, true, REVEAL>(A, n_blocks, [&](int q) {
        const int lane = threadIdx.x & 63;
        int p0, p1;
        if (I.user_pi) {
            p0 = I.user_pi[(size_t)q * A.T + (lane < A.nb ? lane : 0)];
            return p0 < 0 ? 0 : (p0 >= A.T ? A.T - 1 : p0);
        }
        reveal_order(I.seed, q, A.T, p0, p1);       // the table is being written by this launch
        return lane < A.nb ? p0 : __builtin_amdgcn_readfirstlane(p0);
    });
    else init_queries(I, (int)blockIdx.x - n_blocks);
}

// Exact scores of the survivors of the queries whose list holds ids (score_slots: of all), by
// list position; a workgroup per pair, its wavefronts share the document's blocks (survivors are
// few: latency).  128 queries x 10 pairs of 106 tokens that no cache holds: 87 us with a
// wavefront per pair and one block in flight, 12 us so; 64 queries x 10 pages of 1,030 tokens 81 -> 18.
template <typename Tag, int D, int TQ>
__global__ __launch_bounds__(256, (score_waves<TQ, Frag<Tag, D>>())) void k_gather_survivors(GatherArgs A) {
    using F = Frag<Tag, D>;
    using V = typename F::val_t;
    constexpr int ROWB = D * F::ELEM_BYTES;
    __shared__ int ex[EX_FLOATS];
    const int q = blockIdx.y;
    const QueryCtl c = A.ctl[q];
    if (c.mode != 0 && !A.score_slots) return;
    if ((int)blockIdx.x >= c.count) return;
    const int32_t* slot_ids = c.mode != 0 && !A.cache_all ? A.cid + (size_t)q * A.cache_cap : nullptr;
    const int32_t* list = c.implicit ? nullptr : (c.cur ? A.list1 : A.list0) + (size_t)q * A.N;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15;
    const int kg = lane >> 4;
    F bq[TQ];
    const bool query_wild = load_query<F, ROWB, TQ>(A, q, col, kg, bq);
    for (int k = blockIdx.x; k < c.count; k += gridDim.x) {
        int id = list ? list[k] : k;
        if (slot_ids) id = slot_ids[id];
        int64_t o0, o1;
        doc_range(A, id, o0, o1);
        V h[TQ];
#pragma unroll
        for (int tt = 0; tt < TQ; ++tt) h[tt] = lowest_val<V>();
        fold_doc<ROWB, score_ahead<TQ, F>()>((const char*)A.docs, o0, o1, wave, 4, col, kg, bq, query_wild, h);
        float w[Pack<TQ>::NW];
        doc_cells(h, 4, 1.f, ex, w);
        using SC = Score<TQ, TQ>;
        float sc[SC::NS];
        SC::finish(w, A.T, col, sc);
        if (lane == 0 && wave == 0) A.out[(size_t)q * A.N + k] = sc[0];
    }
}

// All documents of all queries, a wavefront per pair, or (shared) a workgroup, whose wavefronts share
// the document's blocks.
template <typename Tag, int D, int TQ>
__global__ __launch_bounds__(256, (score_waves<TQ, Frag<Tag, D>>())) void k_gather_all(GatherArgs A) {
    using F = Frag<Tag, D>;
    using V = typename F::val_t;
    constexpr int ROWB = D * F::ELEM_BYTES;
    __shared__ int ex[EX_FLOATS];
    const int q = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15;
    const int kg = lane >> 4;
    const int parts = A.shared ? 4 : 1;
    const int first = A.shared ? (int)blockIdx.x : (int)blockIdx.x * 4 + wave;
    if (first >= (int)A.N) return;                  // shared: the same for the whole workgroup
    F bq[TQ];
    const bool query_wild = load_query<F, ROWB, TQ>(A, q, col, kg, bq);
    for (int id = first; id < (int)A.N; id += (int)gridDim.x * (4 / parts)) {
        int64_t o0, o1;
        doc_range(A, id, o0, o1);
        V h[TQ];
#pragma unroll
        for (int tt = 0; tt < TQ; ++tt) h[tt] = lowest_val<V>();
        fold_doc<ROWB, score_ahead<TQ, F>()>((const char*)A.docs, o0, o1, A.shared ? wave : 0, parts, col, kg, bq, query_wild, h);
        float w[Pack<TQ>::NW];
        doc_cells(h, parts, 1.f, ex, w);
        if (A.shared && wave > 0) continue;
        using SC = Score<TQ, TQ>;
        float sc[SC::NS];
        SC::finish(w, A.T, col, sc);
        if (lane == 0) A.out[(size_t)q * A.N + id] = sc[0];
        if (A.cells) {
            const int row = lane >> 4;
#pragma unroll
            for (int j = 0; j < SC::NW; ++j) {
                const int t = Pack<TQ>::tile_of_row(j, row) * 16 + col;
                if (Pack<TQ>::row_is_primary(row) && t < A.T) A.cells[((size_t)q * A.N + id) * A.T + t] = w[j];
            }
        }
    }
}

enum { GM_ROUND = 0, GM_SURVIVORS = 1, GM_ALL = 2, GM_CACHE_ALL = 3, GM_DOCS = 4 };

template <typename Tag, int D, int TQ>
static hipError_t gather_mode(const GatherArgs& A, const InitArgs& I, int mode, dim3 grid, hipStream_t st) {
    const dim3 block(256);
    if (mode == GM_ROUND) k_gather_round<Tag, D, TQ><<<grid, block, 0, st>>>(A);
    else if (mode == GM_DOCS) {
        if constexpr (!cuts<Frag<Tag, D>>()) k_gather_docs<Tag, D, TQ><<<grid, 64, 0, st>>>(A);
        else return hipErrorInvalidValue;
    }
    else if (mode == GM_CACHE_ALL) {
        if (A.nb) k_cache_all<Tag, D, TQ, true><<<grid, block, 0, st>>>(A, I);
        else k_cache_all<Tag, D, TQ, false><<<grid, block, 0, st>>>(A, I);
    }
    else if constexpr (!__is_same(Tag, i8_tag)) {   // scores come from the stored embeddings
        if (mode == GM_SURVIVORS) k_gather_survivors<Tag, D, TQ><<<grid, block, 0, st>>>(A);
        else k_gather_all<Tag, D, TQ><<<grid, block, 0, st>>>(A);
    } else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <typename Tag, int D>
static hipError_t gather_tq(const GatherArgs& A, const InitArgs& I, int mode, dim3 grid, hipStream_t st) {
    const int tq = (A.T + 15) / 16;
    if (tq <= 1) return gather_mode<Tag, D, 1>(A, I, mode, grid, st);
    if (tq <= 2) return gather_mode<Tag, D, 2>(A, I, mode, grid, st);
    if (tq <= 4) return gather_mode<Tag, D, 4>(A, I, mode, grid, st);
    if constexpr (Tag::wide) return gather_mode<Tag, D, 8>(A, I, mode, grid, st);
    return hipErrorInvalidValue;
}

template <typename Tag>
static hipError_t gather_by_d(const GatherArgs& A, const InitArgs& I, int mode, int d, dim3 grid, hipStream_t st) {
    if (d == 128) return gather_tq<Tag, 128>(A, I, mode, grid, st);
    if (d == 64) return gather_tq<Tag, 64>(A, I, mode, grid, st);
    // no codes in these widths: the int8 MFMA contracts 64 elements at a time
    if constexpr (!__is_same(Tag, i8_tag)) {
        if (d == 96) return gather_tq<Tag, 96>(A, I, mode, grid, st);
        if (d == 32) return gather_tq<Tag, 32>(A, I, mode, grid, st);
    }
    return hipErrorInvalidValue;
}

// co != nullptr: the reveal reads the int8 codes instead of the stored embeddings
static hipError_t gather_any(GatherArgs& A, const InitArgs& I, int mode, const Problem& P, const Work& W, dim3 grid,
                             const Coarse* co, hipStream_t st) {
    A.Q = P.Q;
    A.docs = P.docs;
    A.off = P.off;
    A.N = P.N;
    A.total = P.total;
    A.nq = P.nq;
    A.T = P.T;
    A.list0 = W.list[0];
    A.list1 = W.list[1];
    A.pi = W.pi;
    A.stat = W.stat;
    A.cache_cap = W.cache_cap;
    A.TP = W.TP;
    A.cid = W.cid;
    A.cstat = W.cstat;
    A.ccell = W.ccell;
    if (co) {
        A.Q = co->Q8;
        A.docs = co->docs8;
        A.qscale = co->qscale;
        A.dscale = co->dscale;
        return gather_by_d<i8_tag>(A, I, mode, P.d, grid, st);
    }
    return P.dt == DT_BF16 ? gather_by_d<bf16_tag>(A, I, mode, P.d, grid, st)
                           : gather_by_d<f32_tag>(A, I, mode, P.d, grid, st);
}

// Workgroups of a round's gather: enough that the hardware's dispatch evens out documents of
// different lengths (eight or more per CU and several turns of them), few enough that a round
// without pairs ends at once (8,192: 4.7 us; 256 per query at 128 queries: 9 us).
constexpr long long GATHER_BLOCKS = 8192;
hipError_t launch_gather_round(const Problem& P, const Work& W, const RevealRound& rr, const Coarse* co, hipStream_t st) {
    GatherArgs A{};
    A.ctl = W.ctl;
    A.lo = rr.lo;
    A.nb = rr.nb;
    A.n_prev = rr.n_prev;
    A.G = 1;
    while (A.G < rr.nb) A.G <<= 1;
    A.pairs_r = rr.r == 1 ? nullptr : W.pairs + rr.r;
    A.work = W.work;
    A.dense = rr.dense;
    const long long blocks = (long long)P.nq * P.N;
    if (rr.dense.enough) {
        A.holders = W.stat2;
        const hipError_t e = gather_any(A, InitArgs{}, GM_DOCS, P, W, dim3((unsigned)(P.N < 32768 ? P.N : 32768)), co, st);
        if (e != hipSuccess) return e;
    }
    return gather_any(A, InitArgs{}, GM_ROUND, P, W, dim3((unsigned)(blocks < GATHER_BLOCKS ? blocks : GATHER_BLOCKS)), co, st);
}

// k_cache_all takes round 1's batch from the cells as it computes them: each wavefront works out the reveal order, while
// its loads are under way, and k_select_prune reads 8 bytes a document side by side instead of cells from as many lines
// (1 query x 1,000 documents: 13 us from its start to the threshold with cells, 7 so; 37.0 -> 31.5 us a call, 2 x 487
// 25.0 -> 22.5).  A query's list gains some ns a document, a pair costs as many, shared by the wavefronts that the query
// rows leave on a SIMD: four or three of them 9 x 709 46.9 -> 43.1, 12 x 522 39.8 -> 37.2; two (96 registers of query rows
// or more: fp32 from 17 tokens in d = 128 and from 33 in d = 64 on, bf16 of more than 64 in d = 96 and 128) 4 x 1,000
// of 32 fp32 tokens in d = 128 53.6 -> 50.5, but 8 x 1,400 61.9 -> 66.6, 12 x 400 50.6 -> 52.2; one (fp32 from 33 tokens in d = 128
// on) 1 x 4,000 93.4 -> 87.6, 3 x 1,000 76.4 -> 73.5, but 3 x 2,700 108.6 -> 112.8, 8 x 1,400 112.4 -> 128.9.
bool cache_all_reveals(const Problem& P, const Coarse* co) {
    const int tq = (P.T + 15) / 16;
    const int row_regs = (tq <= 1 ? 1 : tq <= 2 ? 2 : tq <= 4 ? 4 : 8) * P.d * (co ? 2 : P.dt == DT_BF16 ? 4 : 12) / 32;
    const int64_t pairs = (int64_t)P.nq * P.N;
    if (row_regs >= 192) return P.nq <= 1 || (P.nq <= 3 && pairs <= 4096);
    if (row_regs >= 96) return P.nq <= 5;
    return P.nq <= 8 || pairs <= 12288;
}

hipError_t launch_cache_all(const Problem& P, const Work& W, const Knobs& kn, int R, uint64_t seed,
                            const int32_t* user_pi, const Trace& tr, const Coarse* co, hipStream_t st) {
    GatherArgs A{};
    A.dense = kNeverDense;
    const InitArgs I = init_args(P, W, kn, R, seed, user_pi, tr, 0);
    if (cache_all_reveals(P, co)) A.nb = kn.B < P.T ? kn.B : P.T;
    A.G = 1;
    while (A.G < A.nb) A.G <<= 1;
    long long blocks = (long long)P.nq * P.N;
    // A document shared by four wavefronts loads the query four times.  From some three pairs a CU a
    // wavefront per pair is faster (us a call: 1,000 pairs of 48 fp32 tokens 112 -> 104, 2,000 of bf16 56 -> 50),
    // below shared documents are (250 pairs 35 and 38, 250 of 500 tokens 38 and 51).
    if (blocks >= 768) blocks = (blocks + 3) / 4;
    blocks = blocks < GATHER_BLOCKS ? blocks : GATHER_BLOCKS;
    fill_trace(P, R, tr, st);
    return gather_any(A, I, GM_CACHE_ALL, P, W, dim3((unsigned)(blocks + I.init_blocks)), co, st);
}

hipError_t launch_gather_survivors(const Problem& P, const Work& W, const Knobs& kn, float* out,
                                   bool score_slots, bool cache_all, hipStream_t st) {
    GatherArgs A{};
    A.ctl = W.ctl;
    A.out = out;
    A.score_slots = score_slots ? 1 : 0;
    A.cache_all = cache_all ? 1 : 0;
    // most queries end with at most K + M survivors
    const int64_t want = (int64_t)kn.K + kn.M < 256 ? (int64_t)kn.K + kn.M : 256;
    return gather_any(A, InitArgs{}, GM_SURVIVORS, P, W, dim3((unsigned)(P.N < want ? P.N : want), P.nq), nullptr, st);
}

// A workgroup per pair where wavefronts would be few, or where their last turn (1,024 SIMDs) would
// be emptier and the documents are long enough for four: 10 documents of 15,000 tokens 459 us with a
// wavefront each and 123 shared (bf16, one query), 200 of 1,030 x 6 fp32 queries 186 and 124; 1,000 pairs
// of 1,030 196 and 207, 1,000 of 48 13 and 16.
bool gather_shares(const Problem& P) {
    const int64_t pairs = (int64_t)P.nq * P.N;
    return pairs < 768 || (pairs < 4096 && P.total >= 512 * P.N && 4 * ((pairs + 1023) / 1024) > (pairs + 255) / 256);
}

hipError_t launch_gather_all(const Problem& P, const Work& W, float* out, float* cells, hipStream_t st) {
    GatherArgs A{};
    A.out = out;
    A.cells = cells;
    A.shared = gather_shares(P) ? 1 : 0;
    const int64_t gx = A.shared ? P.N : (P.N + 3) / 4;
    int64_t most = P.nq >= 4 ? 256 : 1024 / P.nq;   // four workgroups a CU over all queries
    // fp32 with a wavefront per document: as many as the registers hold and no more, or fewer.  (us, two queries x
    // 20,000 documents of 100 tokens: d = 128, T = 16 with 512 workgroups 285, 768 304, 1,024 372; d = 96, T = 32 237, 240, 278;
    // d = 64, T = 48 223, 209, 232; d = 32, T = 16 89, 75, 74; 16 x 5,000 of d = 32, T = 32, 1,024 132, 4,096 156.)
    if (P.dt == DT_F32 && !A.shared) most = (P.d >= 96 ? 512 : P.d == 64 ? 768 : 1024) / P.nq;
    if (most < 1) most = 1;
    return gather_any(A, InitArgs{}, GM_ALL, P, W, dim3((unsigned)(gx < most ? gx : most), P.nq), nullptr, st);
}

// Exact score of a survivor from its cached cells: the T cells of a slot are laid out as the
// column maxima of TQ tiles and summed by the same routine as everywhere else (same bits).
template <int TQ>
__device__ __forceinline__ float cached_score(const float* crow, int T) {
    const int col = threadIdx.x & 15;
    using SC = Score<TQ, TQ>;
    float h[TQ], w[SC::NW], sc[SC::NS];
#pragma unroll
    for (int tt = 0; tt < TQ; ++tt) h[tt] = crow[tt * 16 + col];
    SC::run(h, T, col, w, sc);
    return sc[0];
}

// =====================================================================================
// block-wide helpers for the one-workgroup-per-query kernels (1024 threads)
// =====================================================================================
constexpr int SEL_THREADS = 1024;
constexpr int SEL_WAVES = SEL_THREADS / 64;
constexpr int SEL_ITEMS = 4;                       // consecutive entries per thread per chunk (long lists)
constexpr int SEL_CHUNK = SEL_THREADS * SEL_ITEMS;
constexpr int SEL_RUN = 16;                        // samples are taken in runs of adjacent entries
// Lists longer than SEL_TILE are first cut down tile by tile (k_select_segments,
// k_topk_segments).  k_topk holds what is left in registers, SEL_E entries per thread; k_select_prune,
// which needs more registers per entry, SEL_REGS, and takes longer lists from memory.
constexpr int SEL_E = 16;
constexpr int SEL_TILE = SEL_E * SEL_THREADS;
static_assert(SEL_TILE == 16384, "the cell cache's slots per query must fit one tile");
constexpr int SEG_E = SEG_TILE / SEL_THREADS;      // pre-filter kernels: entries per thread and tile
// (8: topk 1,000 x 1 62 -> 70 us.  k_select_prune holds three ways through a list and needs more than the
// 128 registers that 1,024 threads leave: with 4, 13 of them and 56 bytes of scratch a lane spill.)
constexpr int SEL_REGS = 4;
constexpr int SEL_BINS = 2048;
constexpr int SEL_FEW = 1024;

struct SelShared {
    uint32_t hist[SEL_BINS];
    int wtot[SEL_WAVES];
    int pick[2];
    int cnt[SEL_WAVES];                            // kept entries per wavefront
    uint32_t group[64];                            // largest key of each 16 lanes
    uint32_t few[SEL_FEW];                         // keys that reach the lower bound, in any order
    int n_few;
    int round_count[COLBANDIT_MAX_ROUNDS];         // survivors and threshold of the rounds run
    float round_tau[COLBANDIT_MAX_ROUNDS];
};

// wave_incl_scan inside each row of 16 lanes
__device__ __forceinline__ int row_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    return v;
}
// this thread's wavefront, as a scalar
__device__ __forceinline__ int my_wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
// sum of the wavefronts' totals before this wavefront, and of all (wtot: LDS, one per wavefront)
__device__ __forceinline__ int waves_before(const int* wtot, int& total) {
    const int x = wtot[threadIdx.x & (SEL_WAVES - 1)];
    const int incl = row_incl_scan(x);
    const int wave = my_wave();
    total = __builtin_amdgcn_readlane(incl, SEL_WAVES - 1);
    return __builtin_amdgcn_readlane(incl, wave) - __builtin_amdgcn_readlane(x, wave);
}

// Exclusive scan of v over the block in thread order; returns the thread's offset and the
// block total.  wtot: LDS int[SEL_WAVES].  Two barriers.
__device__ __forceinline__ int block_excl_scan(int v, int* wtot, int& total) {
    const int incl = wave_incl_scan(v);
    if ((threadIdx.x & 63) == 63) wtot[threadIdx.x >> 6] = incl;
    __syncthreads();
    const int base = waves_before(wtot, total);
    __syncthreads();
    return base + incl - v;
}

// hist[bin] += 1 for every lane with `on`.  Keys of similar magnitude share their leading
// digit, so plain LDS atomics of a wavefront would pile onto one address: up to four rounds of
// "first pending lane's bin, one add for all lanes that share it" come first, the rest (spread
// digits) go as ordinary atomics.
__device__ __forceinline__ void hist_add(uint32_t* hist, int bin, bool on) {
    unsigned long long pending = __ballot(on);
#pragma unroll 1
    for (int it = 0; it < 4 && pending != 0ull; ++it) {
        const int leader = __ffsll((long long)pending) - 1;
        const int lbin = __builtin_amdgcn_readlane(bin, leader);
        const unsigned long long same = __ballot(on && bin == lbin) & pending;
        if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[lbin], (uint32_t)__popcll(same));
        pending &= ~same;
    }
    if ((pending >> (threadIdx.x & 63)) & 1ull) atomicAdd(&hist[bin], 1u);
}

// One digit of the radix selection.  The histogram of the digit is complete (the caller's
// barrier): finds the bin, counted from the highest down, that holds the kk-th entry, moves kk to
// the rank inside that bin, and leaves the histogram cleared.  Every thread takes its two
// neighbouring bins (one for 1,024), so that no two lanes of a read share a bank beyond the
// two-word stride; one wavefront reading 32 bins per lane was a 32-way conflict and took
// longer than the histogram itself.  Two barriers.
__device__ __forceinline__ int pick_digit(SelShared& sh, int nbins, int& kk) {
    const int per = nbins / SEL_THREADS;
    const int hi = nbins - 1 - (int)threadIdx.x * per;
    const int c0 = (int)sh.hist[hi];
    sh.hist[hi] = 0u;
    int c1 = 0;
    if (per == 2) {
        c1 = (int)sh.hist[hi - 1];
        sh.hist[hi - 1] = 0u;
    }
    const int local = c0 + c1;
    const int incl = wave_incl_scan(local);
    if ((threadIdx.x & 63) == 63) sh.wtot[threadIdx.x >> 6] = incl;
    __syncthreads();
    int all;
    const int excl = waves_before(sh.wtot, all) + incl - local;
    if (excl < kk && kk <= excl + local) {          // exactly one thread
        const bool first = excl + c0 >= kk;
        sh.pick[0] = first ? hi : hi - 1;
        sh.pick[1] = first ? kk - excl : kk - excl - c0;
    }
    __syncthreads();
    kk = sh.pick[1];
    return sh.pick[0];
}

// clears the histogram (pick_digit leaves it clear afterwards); the caller's next barrier publishes
__device__ __forceinline__ void clear_hist(SelShared& sh) {
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) sh.hist[i] = 0u;
    if (threadIdx.x == 0) {
        sh.pick[0] = 0;
        sh.pick[1] = 1;
        sh.n_few = 0;
    }
    __syncthreads();
}

// K-th largest (K >= 1) of the 64 lanes' keys, bit by bit from the top: a step is one comparison
// and a count of its mask.  BITS < 32: only the leading bits, i.e. a lower bound.  (Two bits a step with three masks, a
// loop of one or four steps, or ranks of few lanes: no faster, 1 query x 1,000 documents 28.5 us so and 28.3 to 30.3.)
template <int BITS>
__device__ __forceinline__ uint32_t wave_kth_largest(uint32_t v, int K) {
    uint32_t best = 0;
#pragma unroll
    for (int bit = 31; bit > 31 - BITS; --bit) {
        const uint32_t test = best | (1u << bit);
        if (__popcll(__ballot(v >= test)) >= K) best = test;
    }
    return best;
}

// Radix selection of the K-th largest (1 <= K <= number of set bits over the block) of the keys
// whose bit in `on` is set: three passes (11+11+10 bits), any distribution of keys.
template <int NK>
__device__ __forceinline__ uint32_t kth_largest_radix(const uint32_t (&key)[NK], unsigned on, int K, SelShared& sh) {
    uint32_t prefix = 0, pmask = 0;
    int kk = K;
#pragma unroll 1
    for (int p = 0; p < 3; ++p) {
        const int shift = p == 0 ? 21 : (p == 1 ? 10 : 0);
        const int nbins = p == 2 ? 1024 : 2048;
#pragma unroll
        for (int u = 0; u < NK; ++u)
            hist_add(sh.hist, (int)((key[u] >> shift) & (nbins - 1)),
                     ((on >> u) & 1u) && (key[u] & pmask) == prefix);
        __syncthreads();
        prefix |= (uint32_t)pick_digit(sh, nbins, kk) << shift;
        pmask |= (uint32_t)(nbins - 1) << shift;
    }
    return prefix;
}

// A lower bound of the K-th largest key over the block, given each thread's largest (0: it has
// none): the K-th largest of a set of maxima, which are keys of K different entries.  0 when the
// set is smaller than K.  The few largest keys seldom share a group, so the bound is close.
// K <= 32: 64 groups of 16 lanes, one barrier; else the threads themselves.
__device__ __forceinline__ uint32_t lower_bound_key(uint32_t top, int K, SelShared& sh) {
    if (K > 32) {
        const uint32_t k1[1] = {top};
        return kth_largest_radix<1>(k1, 1u, K, sh);
    }
    auto ror_max = [](uint32_t v, auto ctrl) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, false);
        return o > v ? o : v;
    };
    top = ror_max(top, std::integral_constant<int, DPP_ROW_ROR + 8>{});
    top = ror_max(top, std::integral_constant<int, DPP_ROW_ROR + 4>{});
    top = ror_max(top, std::integral_constant<int, DPP_ROW_ROR + 2>{});
    top = ror_max(top, std::integral_constant<int, DPP_ROW_ROR + 1>{});
    if ((threadIdx.x & 15) == 0) sh.group[threadIdx.x >> 4] = top;
    __syncthreads();
    return wave_kth_largest<22>(sh.group[threadIdx.x & 63], K);
}

// appends the lanes' keys to the collected ones (n_few counts on beyond SEL_FEW)
__device__ __forceinline__ void collect_few(uint32_t key, bool hit, SelShared& sh) {
    const int lane = threadIdx.x & 63;
    const unsigned long long m = __ballot(hit);
    if (m != 0ull) {                                // uniform over the wavefront
        int at = 0;
        if (lane == 0) at = atomicAdd(&sh.n_few, __popcll(m));
        at = __builtin_amdgcn_readlane(at, 0) + __popcll(m & ((1ull << lane) - 1ull));
        if (hit && at < SEL_FEW) sh.few[at] = key;
    }
}
// K-th largest of the collected keys (at least K of them), which are cleared; false if there were
// too many to keep.  Two barriers.
__device__ __forceinline__ bool kth_of_few(int K, uint32_t& kth, SelShared& sh) {
    const int lane = threadIdx.x & 63;
    __syncthreads();
    const int n = sh.n_few;
    if (n <= 64) {
        kth = wave_kth_largest<32>(lane < n ? sh.few[lane] : 0u, K);
    } else if (n <= SEL_FEW && (int)threadIdx.x < n) {
        const uint32_t mine = sh.few[threadIdx.x];
        int above = 0, equal = 0;
        for (int j = 0; j < n; ++j) {
            const uint32_t x = sh.few[j];
            above += x > mine;
            equal += x == mine;
        }
        if (above < K && K <= above + equal) sh.pick[0] = (int)mine;   // all writers hold the same key
    }
    __syncthreads();                                // n_few and few have been read
    if (threadIdx.x == 0) sh.n_few = 0;             // the next use is behind a barrier of its own
    if (n > 64) kth = (uint32_t)sh.pick[0];
    return n <= SEL_FEW;
}

// Key of the K-th largest (1 <= K <= number of set bits over the block) of the keys whose bit in
// `on` is set, NK per thread.  The keys that reach a lower bound of it, a little more than K, are
// collected and ranked; only when they are many (ties, or K near the size of the list) does the
// radix selection run over all keys.  A histogram pass of that costs about 100 instructions per
// key of a thread, this selection about 100 in all: threshold and prune of round 1 at
// 128 queries x 500,000 documents 76 -> 34 us, seven cached rounds of lists of 1,800 entries
// 7 launches of 31 us -> one of 99 us.
template <int NK>
__device__ __forceinline__ uint32_t kth_largest_regs(const uint32_t (&key)[NK], unsigned on, int K, SelShared& sh) {
    uint32_t top = 0;
#pragma unroll
    for (int u = 0; u < NK; ++u) {
        const uint32_t k = (on >> u) & 1u ? key[u] : 0u;
        top = k > top ? k : top;
    }
    const uint32_t bound = lower_bound_key(top, K, sh);
#pragma unroll
    for (int u = 0; u < NK; ++u) collect_few(key[u], ((on >> u) & 1u) && key[u] >= bound, sh);
    uint32_t kth;
    if (!kth_of_few(K, kth, sh)) kth = kth_largest_radix<NK>(key, on, K, sh);
    return kth;
}

// The same over key_of(0..count-1) of a list of any length: the keys are evaluated again in each
// pass, SEL_ITEMS strided entries per thread and trip so that several loads are in flight.
template <class KeyFn>
__device__ uint32_t kth_largest_list(int count, int K, KeyFn key_of, SelShared& sh) {
    uint32_t prefix = 0, pmask = 0;
    int kk = K;
#pragma unroll 1
    for (int p = 0; p < 3; ++p) {
        const int shift = p == 0 ? 21 : (p == 1 ? 10 : 0);
        const int nbins = p == 2 ? 1024 : 2048;
        for (int base = 0; base < count; base += SEL_CHUNK) {
            uint32_t key[SEL_ITEMS];
#pragma unroll
            for (int u = 0; u < SEL_ITEMS; ++u) {
                const int idx = base + u * SEL_THREADS + threadIdx.x;
                key[u] = idx < count ? key_of(idx) : 0u;
            }
#pragma unroll
            for (int u = 0; u < SEL_ITEMS; ++u) {
                const int idx = base + u * SEL_THREADS + threadIdx.x;
                hist_add(sh.hist, (int)((key[u] >> shift) & (nbins - 1)),
                         idx < count && (key[u] & pmask) == prefix);
            }
        }
        __syncthreads();
        prefix |= (uint32_t)pick_digit(sh, nbins, kk) << shift;
        pmask |= (uint32_t)(nbins - 1) << shift;
    }
    return prefix;
}

// Layout of n <= E * SEL_THREADS list entries over the block: each wavefront takes `span`
// consecutive ones (whole groups of 64, the same for all wavefronts), thread `lane` the entries
// u * 64 + lane of them.  Entry order is then (wavefront, u, lane), and the places of kept entries
// need one exchange of 16 counts.
struct Spread {
    int first, n, span;      // this thread's first entry; entries in all; entries per wavefront
    __device__ __forceinline__ explicit Spread(int n_) : n(n_) {
        span = (n_ + SEL_THREADS - 1) / SEL_THREADS * 64;
        first = my_wave() * span + (int)(threadIdx.x & 63);
    }
    // list position of the thread's u-th entry (past the end: the last one again)
    __device__ __forceinline__ int at(int u) const {
        const int i = first + u * 64;
        return i < n ? i : n - 1;
    }
    // which of the thread's E entries exist
    template <int E> __device__ __forceinline__ unsigned mask() const {
        unsigned m = 0;
#pragma unroll
        for (int u = 0; u < E; ++u) m |= (u * 64 < span && first + u * 64 < n ? 1u : 0u) << u;
        return m;
    }
};

// Places of the kept entries of such a list, in entry order: place(u) is the number of kept
// entries before this thread's u-th, total their number.  One barrier; the caller puts another
// between two uses.
template <int E> struct Places {
    unsigned long long m[E];
    int base[E], total;
    __device__ __forceinline__ Places(unsigned keep, SelShared& sh) {
        int n = 0;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            m[u] = __ballot((keep >> u) & 1u);
            base[u] = n;
            n += __popcll(m[u]);
        }
        if ((threadIdx.x & 63) == 0) sh.cnt[threadIdx.x >> 6] = n;
        __syncthreads();
        const int before = waves_before(sh.cnt, total);
#pragma unroll
        for (int u = 0; u < E; ++u) base[u] += before;
    }
    __device__ __forceinline__ int place(int u) const {
        return base[u] + __builtin_amdgcn_mbcnt_hi((unsigned)(m[u] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m[u], 0u));
    }
};

// The 16 slot values of a reveal batch, summed in the order of the cross-lane form
// (batch_stats_g): zero slots past nb make the order of every group size a case of this one.
__device__ __forceinline__ float slot_sum(const float (&v)[16]) {
    const float u0 = (v[0] + v[15]) + (v[7] + v[8]), u1 = (v[1] + v[14]) + (v[6] + v[9]);
    const float u2 = (v[2] + v[13]) + (v[5] + v[10]), u3 = (v[3] + v[12]) + (v[4] + v[11]);
    return (u0 + u2) + (u1 + u3);
}
// The batch statistics of batch_stats_g evaluated by ONE thread (same additions, same bits).
// cell(i): the batch's i-th cell.
template <class CellFn>
__device__ __forceinline__ void batch_stats_thread(CellFn cell, int nb, float& s, float& m2) {
    if (nb <= 4) {                                  // uniform
        float c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = i < nb ? cell(i) : 0.f;
        s = (c[0] + c[2]) + (c[1] + c[3]);
        const float mean = div_count(s, nb);
        float d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float x = i < nb ? c[i] - mean : 0.f;
            d[i] = x * x;
        }
        m2 = (d[0] + d[2]) + (d[1] + d[3]);
        return;
    }
    float c[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = i < nb ? cell(i) : 0.f;
    s = slot_sum(c);
    const float mean = div_count(s, nb);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const float x = i < nb ? c[i] - mean : 0.f;
        c[i] = x * x;
    }
    m2 = slot_sum(c);
}

// =====================================================================================
// threshold + prune: tau_r = K-th largest LCB over the active set, A_{r+1} = {UCB >= tau_r}
// (Algorithm 1, threshold and elimination steps), one workgroup per query, stable.
// A query whose cells are cached needs nothing but this kernel any more: its remaining rounds run
// here one after the other, each entry's (sum, M2) taking the batch pi[lo..lo+nb) from its
// cached cells.
// =====================================================================================
struct SelArgs {
    QueryCtl* ctl;
    int32_t* list0;
    int32_t* list1;
    float2* stat;
    float2* stat2;
    unsigned long long* pairs;           // [R+2] pairs, then [R+2] document tokens of those pairs
    unsigned long long* work;            // [nq] queries of the next round
    const int64_t* off;                  // document offsets (token counts of the kept pairs)
    int R;
    DenseRule dense;
    int64_t N;
    int nq, T, B, K, KM;
    int r, n, n_prev, nb;                // this launch's round
    float a, b;
    const int32_t* pi;
    int cache_all;                       // round 1 has cached the cells of all documents
    int fold_cells;                      // ... and not revealed them
    int finish_next;                     // round 1: round 2 ends with the top-K of all queries
    int note_pairs;                      // cache_all: then the pairs going on to round 2 are counted for the statistics
    int cache_cap, TP;
    const int32_t* cid;
    float2* cstat;
    const float* ccell;
    int32_t* cnt_hist;
    float* tau_hist;
    int32_t* tr_count;
    float* tr_tau;
    float* tr_lcb;
    float* tr_ucb;
    uint8_t* tr_alive;
    int32_t* seg_cnt;                    // [nq][SEG_MAX]: candidates per segment (k_select_segments)
    float kappa;                         // radius per unit sigma_hat of the round
    unsigned enough;                     // round 1, where round 2 may gather by document (DenseRule); else 0
    unsigned long long certain;          // ... from how many pairs on it is sure to be a corpus pass (DenseRule::certain)
};
// ... of every round.  A parameter of its own: indexed at run time, it would keep the whole of SelArgs, which
// the compiler otherwise takes apart, in scratch memory.
struct Kappas {
    float of[COLBANDIT_MAX_ROUNDS + 1];
};

// Candidates that the segment workgroups left at the segment starts of `buf` -> one contiguous
// run at the front, order kept.  A destination never lies beyond its source, and a chunk is read
// completely before it is written.
__device__ int merge_segments(int32_t* buf, const int32_t* cnt, int count) {
    const int len = seg_len(count);
    const int n_seg = seg_count(count);
    int base = 0;
    for (int sg = 0; sg < n_seg; ++sg) {
        const int c = cnt[sg];
        const int src = sg * len;
        if (src != base) {
            for (int k0 = 0; k0 < c; k0 += SEL_THREADS) {
                const int k = k0 + (int)threadIdx.x;
                const int v = k < c ? buf[src + k] : 0;
                __syncthreads();
                if (k < c) buf[base + k] = v;
                __syncthreads();
            }
        }
        base += c;
    }
    __syncthreads();
    return base;
}

// Where candidate i of a segmented list lies.  first: LDS int[SEG_MAX + 1], the number of
// candidates before each segment (segment_starts).
__device__ __forceinline__ int segment_starts(const int32_t* cnt, int count, int* first) {
    const int n_seg = seg_count(count);
    if (threadIdx.x < 64) {
        const int c = (int)threadIdx.x < n_seg ? cnt[threadIdx.x] : 0;
        const int incl = wave_incl_scan(c);
        first[threadIdx.x + 1] = incl;
        if (threadIdx.x == 0) first[0] = 0;
    }
    __syncthreads();
    return first[SEG_MAX];
}
__device__ __forceinline__ int segment_place(int i, int len, const int* first) {
    int s = 0;
#pragma unroll
    for (int step = SEG_MAX / 2; step >= 1; step >>= 1)
        if (first[s + step] <= i) s += step;
    return s * len + (i - first[s]);
}

// Survivor count and threshold of a round, kept in LDS until the query's rounds of this launch
// are over: a store to memory in the round would be waited for at its next barrier.
__device__ __forceinline__ void note_round(SelShared& sh, int r, int count, float tau) {
    sh.round_count[r - 1] = count;
    sh.round_tau[r - 1] = tau;
}

// Enters a query's list (in the buffer nc.cur) with its documents (held_of).  Once what is entered costs more than the corpus
// pass, the round is one and nobody reads the table: the last queries, for which the others wait, need not fill it in (alpha
// 1.0, pages, us longer than a call without any table: 229 queries x 4,778 of 292 tokens 6 -> 4 of 1,740, 166 x 1,113 2.5 -> 1.6
// of 876, 64 x 20,000 of 1,030 55 -> 0 of 6,870).  The number only grows, so each thread asks for itself, here, out of the way of the
// calls that enter nothing: asked once for the workgroup, after a barrier at the end of the prune, it took k_select_prune
// from 14.1 to 15.2 us wherever that runs (67,406 documents x 30).
__device__ __forceinline__ void hold_documents(const SelArgs& A, int q, const QueryCtl& nc) {
    if (pair_count(__hip_atomic_load(A.pairs + 2 * (A.R + 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >= A.certain) return;
    const int32_t* list = (nc.cur ? A.list1 : A.list0) + (size_t)q * A.N;
    uint32_t* holders = (uint32_t*)A.stat2;
    int* held = (int*)held_of(A.stat2, A.nq, A.N);
    for (int k = (int)threadIdx.x; k < nc.count; k += SEL_THREADS) {
        const int id = list[k];
        holders[(size_t)id * A.nq + atomicAdd(held + id, 1)] = (uint32_t)q << 14 | (uint32_t)k;
    }
}

// The end of a query's rounds in this launch: its state, and the documents (pairs and tokens) that
// the next round would have to gather if the list holds ids.
// Also writes the history of the rounds run, and of those that the query will not take part in.
__device__ __forceinline__ void end_rounds(const SelArgs& A, int q, const QueryCtl& nc, int r, bool slots,
                                           long long my_tokens, SelShared& sh,
                                           unsigned long long* kept_tokens) {
    if (!slots) {                                   // uniform over the workgroup
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) my_tokens += __shfl_down(my_tokens, o);
        if ((threadIdx.x & 63) == 0 && my_tokens != 0) atomicAdd(kept_tokens, (unsigned long long)my_tokens);
    }
    __syncthreads();
    // Lists that may make a round worth gathering by document, if others are like them (DenseRule::enough).
    const bool entered = A.enough != 0u && nc.active && nc.count <= A.cache_cap && 4ll * nc.count * A.nq >= (long long)A.enough;
    const int x = A.r + (int)threadIdx.x;           // round
    if (x <= (nc.active ? r : A.R)) {
        const int count = x <= r ? sh.round_count[x - 1] : nc.count;
        A.cnt_hist[x * A.nq + q] = count;
        if (A.tr_count) A.tr_count[x * A.nq + q] = count;
        if (x <= r) {
            A.tau_hist[(x - 1) * A.nq + q] = sh.round_tau[x - 1];
            if (A.tr_tau) A.tr_tau[(x - 1) * A.nq + q] = sh.round_tau[x - 1];
        }
    }
    if (threadIdx.x == 0) {
        A.ctl[q] = nc;
        if (nc.active || A.finish_next) {           // (finished: the round's gather is to cache its survivors' cells)
            // pairs and work item in one step: starts ascend with the items
            const unsigned long long at = atomicAdd(entered ? A.pairs + 2 * (A.R + 2) : A.pairs + r + 1, work_add(nc.count));
            const int place = (int)work_count(at);
            A.work[entered ? A.nq - 1 - place : place] = work_item(q, pair_count(at));
            if (nc.active) atomicAdd(A.pairs + (A.R + 2) + r + 1, *kept_tokens);
            else atomicAdd(A.pairs + 2 * (A.R + 2) + 1, (unsigned long long)nc.count);
        }
    }
    if (entered) hold_documents(A, q, nc);
}

// Round 1 of a query all of whose cells are cached: the pairs that go on, and their tokens, for the
// statistics (no kernel reads them).  entry(u): the thread's u-th entry, a document id here.
template <int E, class EntryFn>
__device__ __forceinline__ void note_pairs(const SelArgs& A, int count, unsigned keep, EntryFn entry) {
    long long tokens = 0;
#pragma unroll
    for (int u = 0; u < E; ++u)
        if ((keep >> u) & 1u) {
            const int e = entry(u);
            tokens += A.off[e + 1] - A.off[e];
        }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) tokens += __shfl_down(tokens, o);
    if ((threadIdx.x & 63) == 0 && tokens != 0) atomicAdd(A.pairs + (A.R + 2) + 2, (unsigned long long)tokens);
    if (threadIdx.x == 0) atomicAdd(A.pairs + 2, (unsigned long long)count);
}

// The remaining rounds of a cached list of at most WAVE_LIST entries, by one wavefront: entry u * 64 + lane.
// A round of sixteen wavefronts takes 10 us however short its list (13 entries: 4.2 us for the batch's tokens
// and then its cells, 4.4 for the selection and its three barriers); here the tokens are in registers, the
// next round's cells are on their way during this one's selection, and nothing waits for another wavefront
// (1 query x 1,000 documents, eight rounds of 13: 100 -> 45 us a call; 7 x 6,007, lists of 59: 110 -> 90).
// Leaves the list in `out`, its length and the last round in sh.pick.
constexpr int WAVE_E = 4;
constexpr int WAVE_LIST = 64 * WAVE_E;
__device__ __forceinline__ void prune_wave(const SelArgs& A, const Kappas& kappas, int q, const int32_t* in, int32_t* out,
                                           const float2* stat, int ncand, int r, bool from_cells, SelShared& sh) {
    constexpr int E = WAVE_E;
    const int lane = threadIdx.x & 63;
    const int T = A.T;
    const int32_t* pi = A.pi + (size_t)q * T;
    const int p0 = pi[lane < T ? lane : T - 1], p1 = pi[lane + 64 < T ? lane + 64 : T - 1];
    auto token = [&](int p) { return p < 64 ? __builtin_amdgcn_readlane(p0, p) : __builtin_amdgcn_readlane(p1, p - 64); };
    int parts = (ncand + 63) >> 6;                  // places of a lane in use
    int e[E];
    float2 st[E];
    unsigned live = 0;
#pragma unroll
    for (int u = 0; u < E; ++u) {
        const int i = u * 64 + lane;
        live |= (i < ncand ? 1u : 0u) << u;
        const int at = i < ncand ? i : ncand - 1;
        e[u] = in ? in[at] : at;
    }
#pragma unroll
    for (int u = 0; u < E; ++u) st[u] = stat[e[u]];
    const float* rows = A.ccell + (size_t)q * A.cache_cap * A.TP;
    float cv[E][4];
    // A batch of at most four: its tokens first, then one branch for each entry (716 documents in rounds of two 62 -> 59 us).
    auto fetch = [&](int round) {
        const int lo = (round - 1) * A.B, nb = lo + A.B < T ? A.B : T - lo;
        int t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = token(lo + (i < nb ? i : 0));
#pragma unroll
        for (int u = 0; u < E; ++u)
            if (u < parts) {
                const unsigned at = (unsigned)(e[u] * A.TP);
#pragma unroll
                for (int i = 0; i < 4; ++i) cv[u][i] = rows[at + (unsigned)t[i]];
            }
    };
    if (A.B <= 4 && from_cells) fetch(r);
    int count;
    for (;; ++r, from_cells = true) {
        const int lo = (r - 1) * A.B;
        const int n = lo + A.B < T ? lo + A.B : T;
        const int nb = n - lo;
        if (from_cells) {
#pragma unroll
            for (int u = 0; u < E; ++u)
                if (u < parts) {
                    float sb, m2b;
                    if (A.B <= 4) {
                        batch_stats_thread([&](int i) { return cv[u][i & 3]; }, nb, sb, m2b);
                    } else {
                        const float* crow = rows + (unsigned)(e[u] * A.TP);
                        batch_stats_thread([&](int i) { return crow[token(lo + i)]; }, nb, sb, m2b);
                    }
                    merge_stats(st[u].x, st[u].y, lo, sb, m2b, nb);
                }
        }
        if (A.B <= 4 && r < A.R) fetch(r + 1);
        const float kappa = kappas.of[r];
        uint32_t key[E];
        float low[E], hi[E];
#pragma unroll
        for (int u = 0; u < E; ++u) {
            key[u] = 0u;
            low[u] = hi[u] = 0.f;
            if (u < parts) {
                interval(st[u].x, st[u].y, n, T, kappa, A.a, A.b, low[u], hi[u]);
                if ((live >> u) & 1u) key[u] = float_key(low[u]);
            }
        }
        uint32_t best = 0;                          // the K-th largest key, bit by bit
        if (parts == 1) {
            best = wave_kth_largest<32>(key[0], A.K);
        } else {
#pragma unroll 4
            for (int bit = 31; bit >= 0; --bit) {
                const uint32_t test = best | (1u << bit);
                int reach = 0;
#pragma unroll
                for (int u = 0; u < E; ++u) reach += __popcll(__ballot(key[u] >= test));
                if (reach >= A.K) best = test;
            }
        }
        const float tau = key_float(best);
        unsigned keep = 0;
#pragma unroll
        for (int u = 0; u < E; ++u) keep |= (hi[u] >= tau ? 1u : 0u) << u;
        keep &= live;
        if (A.tr_lcb) {
            const size_t tro = ((size_t)(r - 1) * A.nq + q) * A.N;
            const int32_t* cid = A.cid + (size_t)q * A.cache_cap;
#pragma unroll
            for (int u = 0; u < E; ++u)
                if ((live >> u) & 1u) {
                    const int id = A.cache_all ? e[u] : cid[e[u]];
                    A.tr_lcb[tro + id] = low[u];
                    A.tr_ucb[tro + id] = hi[u];
                    A.tr_alive[tro + id] = (keep >> u) & 1u;
                }
        }
        live = keep;
        unsigned long long m[E];
        count = 0;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            m[u] = __ballot((live >> u) & 1u);
            count += __popcll(m[u]);
        }
        if (lane == 0) note_round(sh, r, count, tau);
        const bool more = count > A.KM && r < A.R;
        if (more && r == 1 && A.note_pairs) note_pairs<E>(A, count, live, [&](int u) { return e[u]; });
        if (more && (count + 63) >> 6 == parts) continue;
        // the list's end, or fewer places are enough: entries move up, statistics through LDS
        int base = 0;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int at = base + __builtin_amdgcn_mbcnt_hi((unsigned)(m[u] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m[u], 0u));
            if ((live >> u) & 1u) {
                if (!more) out[at] = e[u];
                sh.few[at] = (uint32_t)e[u];
                sh.hist[2 * at] = __float_as_uint(st[u].x);
                sh.hist[2 * at + 1] = __float_as_uint(st[u].y);
            }
            base += __popcll(m[u]);
        }
        if (!more) break;
        __builtin_amdgcn_wave_barrier();            // a wavefront's LDS accesses are performed in order
        asm volatile("" ::: "memory");
        parts = (count + 63) >> 6;
        live = 0;
#pragma unroll
        for (int u = 0; u < E; ++u) {
            const int i = u * 64 + lane;
            live |= (i < count ? 1u : 0u) << u;
            const int at = i < count ? i : count - 1;
            e[u] = (int)sh.few[at];
            st[u] = make_float2(__uint_as_float(sh.hist[2 * at]), __uint_as_float(sh.hist[2 * at + 1]));
        }
        asm volatile("" ::: "memory");
        if (A.B <= 4) fetch(r + 1);
    }
    if (lane == 0) {
        sh.pick[0] = count;
        sh.pick[1] = r;
    }
}

// The rounds of a query whose ncand <= SEL_REGS * SEL_THREADS candidates fit the registers, from
// round r on.  Returns true when they are done; false when cached rounds remain and at most half of the
// places that the list takes in each thread are still needed, or a wavefront is enough (prune_wave): then r is the next round, ncand the
// length of the list in `out`, and the statistics are stored.
__device__ __forceinline__ bool prune_regs(const SelArgs& A, const Kappas& kappas, int q, int count, QueryCtl nc,
                                           const int32_t* in, int32_t* out, float2* stat, const float2* bat,
                                           bool slots, bool fold_dense, bool segmented, int& ncand,
                                           int& r, bool from_cells, SelShared& sh, const int* seg_first,
                                           unsigned long long* kept_tokens) {
    constexpr int E = SEL_REGS;
    const int T = A.T;
    const float a = A.a, b = A.b;
    // Loads are unconditional: places past the end repeat the last entry, entries that have been
    // dropped are carried along, and only `live` decides.  Places that no thread has (a short
    // list) are skipped by scalar branches.
    const Spread sp(ncand);
    unsigned live = sp.mask<E>();
    auto used = [&](int u) { return u * 64 < sp.span; };   // uniform
    // the reveal order, one token a lane: a round's tokens from memory would be waited for before its cells
    const int32_t* pi = A.pi + (size_t)q * T;
    const int lane = threadIdx.x & 63;
    const int p0 = pi[lane < T ? lane : T - 1], p1 = pi[lane + 64 < T ? lane + 64 : T - 1];
    auto token = [&](int p) { return p < 64 ? __builtin_amdgcn_readlane(p0, p) : __builtin_amdgcn_readlane(p1, p - 64); };
    int e[E];
    float2 st[E];
    if (segmented) {
        const int len = seg_len(count);
#pragma unroll
        for (int u = 0; u < E; ++u) e[u] = out[segment_place(sp.at(u), len, seg_first)];
    } else if (in) {
#pragma unroll
        for (int u = 0; u < E; ++u) e[u] = in[sp.at(u)];
    } else {
#pragma unroll
        for (int u = 0; u < E; ++u) e[u] = sp.at(u);
    }
#pragma unroll
    for (int u = 0; u < E; ++u) st[u] = stat[e[u]];
    if (fold_dense) {
        float2 bb[E];
#pragma unroll
        for (int u = 0; u < E; ++u) bb[u] = bat[e[u]];
#pragma unroll
        for (int u = 0; u < E; ++u)
            if (used(u)) merge_stats(st[u].x, st[u].y, A.n_prev, bb[u].x, bb[u].y, A.nb);
    }
    for (;; ++r, from_cells = true) {
        const int lo = (r - 1) * A.B;
        const int n = lo + A.B < T ? lo + A.B : T;
        const int nb = n - lo;
        if (from_cells) {
            const float* cells = A.ccell + (size_t)q * A.cache_cap * A.TP;
            if (nb <= 4) {                          // four entries' cells in flight
#pragma unroll
                for (int g = 0; g < E; g += 4)
                    if (used(g)) {
                        float cv[4][4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int t = token(lo + (i < nb ? i : 0));
#pragma unroll
                            for (int w = 0; w < 4; ++w) cv[w][i] = cells[(unsigned)(e[g + w] * A.TP + t)];
                        }
#pragma unroll
                        for (int w = 0; w < 4; ++w)
                            if (used(g + w)) {
                                float sb, m2b;
                                batch_stats_thread([&](int i) { return cv[w][i & 3]; }, nb, sb, m2b);
                                merge_stats(st[g + w].x, st[g + w].y, lo, sb, m2b, nb);
                            }
                    }
            } else {
#pragma unroll
                for (int u = 0; u < E; ++u)
                    if (used(u)) {
                        const float* crow = cells + (unsigned)(e[u] * A.TP);
                        float sb, m2b;
                        batch_stats_thread([&](int i) { return crow[token(lo + i)]; }, nb, sb, m2b);
                        merge_stats(st[u].x, st[u].y, lo, sb, m2b, nb);
                    }
            }
        }
        const float kappa = kappas.of[r];
        uint32_t key[E];
        float hi[E];
#pragma unroll
        for (int u = 0; u < E; ++u) {
            key[u] = 0u;
            hi[u] = 0.f;
            if (used(u)) {
                float lcb;
                interval(st[u].x, st[u].y, n, T, kappa, a, b, lcb, hi[u]);
                key[u] = float_key(lcb);
            }
        }
        const float tau = key_float(kth_largest_regs<E>(key, live, A.K, sh));
        unsigned keep = 0;
#pragma unroll
        for (int u = 0; u < E; ++u) keep |= (hi[u] >= tau ? 1u : 0u) << u;
        keep &= live;
        if (A.tr_lcb) {
            const size_t tro = ((size_t)(r - 1) * A.nq + q) * A.N;
            const int32_t* cid = A.cid + (size_t)q * A.cache_cap;
#pragma unroll
            for (int u = 0; u < E; ++u)
                if ((live >> u) & 1u) {
                    const int id = slots && !A.cache_all ? cid[e[u]] : e[u];
                    float lcb, ucb;
                    interval(st[u].x, st[u].y, n, T, kappa, a, b, lcb, ucb);
                    A.tr_lcb[tro + id] = lcb;
                    A.tr_ucb[tro + id] = ucb;
                    A.tr_alive[tro + id] = (keep >> u) & 1u;
                }
        }
        live = keep;
        const Places<E> pl(live, sh);
        nc.count = pl.total;
        if (threadIdx.x == 0) note_round(sh, r, nc.count, tau);
        const bool more = slots && nc.count > A.KM && r < A.R;
        if (more && r == 1 && A.note_pairs) note_pairs<E>(A, nc.count, live, [&](int u) { return e[u]; });
        if (more && nc.count > WAVE_LIST && Spread(nc.count).span * 2 > sp.span) continue;
#pragma unroll
        for (int u = 0; u < E; ++u)
            if ((live >> u) & 1u) {
                out[pl.place(u)] = e[u];
                if (more) stat[e[u]] = st[u];
            }
        if (more) {
            ncand = nc.count;
            ++r;
            __syncthreads();                        // list and statistics are read by other threads next
            return false;
        }
        break;
    }
    nc.active = !slots && nc.count > A.KM;
    long long my_tokens = 0;                        // tokens of the documents this thread keeps
    if (!slots) {
#pragma unroll
        for (int u = 0; u < E; ++u)
            if ((live >> u) & 1u) {                 // what a gather of the survivors would have to read
                my_tokens += A.off[e[u] + 1] - A.off[e[u]];
                if (fold_dense) stat[e[u]] = st[u];
            }
    }
    end_rounds(A, q, nc, r, slots, my_tokens, sh, kept_tokens);
    return true;
}

// One round of a query whose list fits a tile but not, with its statistics, the registers: keys
// and upper bounds are held there, entries and statistics are read again.  Returns true when the
// query's rounds are done; false when cached rounds remain: then r is the next round and ncand the
// length of the list in `out`.
__device__ __forceinline__ bool prune_tile(const SelArgs& A, const Kappas& kappas, int q, int count, QueryCtl nc,
                                           const int32_t* in, int32_t* out, float2* stat, const float2* bat,
                                           bool slots, bool fold_dense, bool segmented, int& ncand,
                                           int& r, bool from_cells, SelShared& sh, const int* seg_first,
                                           unsigned long long* kept_tokens) {
    constexpr int E = SEL_E;
    const int T = A.T;
    const float a = A.a, b = A.b;
    const int lo = (r - 1) * A.B;
    const int n = lo + A.B < T ? lo + A.B : T;
    const int nb = n - lo;
    const float kappa = kappas.of[r];
    const int32_t* pq = A.pi + (size_t)q * T + lo;
    const float* cells = A.ccell + (size_t)q * A.cache_cap * A.TP;
    const int len = seg_len(count);
    const Spread sp(ncand);
    const unsigned live = sp.mask<E>();
    auto entry = [&](int u) {
        const int i = sp.at(u);
        return segmented ? out[segment_place(i, len, seg_first)] : (in ? in[i] : i);
    };
    // statistics after this round's batch; `store`: for the rounds after it
    auto stat_of = [&](int e, bool store) {
        float2 st = stat[e];
        if (from_cells) {
            const float* crow = cells + (unsigned)(e * A.TP);
            float sb, m2b;
            batch_stats_thread([&](int i) { return crow[pq[i]]; }, nb, sb, m2b);
            merge_stats(st.x, st.y, lo, sb, m2b, nb);
        } else if (fold_dense) {
            const float2 bb = bat[e];
            merge_stats(st.x, st.y, lo, bb.x, bb.y, nb);
        }
        if (store && (from_cells || fold_dense)) stat[e] = st;
        return st;
    };
    uint32_t key[E];
    float hi[E];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        key[u] = 0u;
        hi[u] = 0.f;
        if (u * 64 < sp.span) {                     // uniform
            const float2 st = stat_of(entry(u), (live >> u) & 1u);
            float lcb;
            interval(st.x, st.y, n, T, kappa, a, b, lcb, hi[u]);
            key[u] = float_key(lcb);
        }
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    const float tau = key_float(kth_largest_regs<E>(key, live, A.K, sh));
    unsigned keep = 0;
#pragma unroll
    for (int u = 0; u < E; ++u) keep |= (hi[u] >= tau ? 1u : 0u) << u;
    keep &= live;
    const Places<E> pl(keep, sh);
    nc.count = pl.total;
    if (threadIdx.x == 0) note_round(sh, r, nc.count, tau);
    if (A.tr_lcb) {
        const size_t tro = ((size_t)(r - 1) * A.nq + q) * A.N;
        const int32_t* cid = A.cid + (size_t)q * A.cache_cap;
#pragma unroll 1
        for (int u = 0; u < E; ++u)
            if ((live >> u) & 1u) {
                const int e = entry(u);
                const int id = slots && !A.cache_all ? cid[e] : e;
                const float2 st = stat[e];          // stored above
                float lcb, ucb;
                interval(st.x, st.y, n, T, kappa, a, b, lcb, ucb);
                A.tr_lcb[tro + id] = lcb;
                A.tr_ucb[tro + id] = ucb;
                A.tr_alive[tro + id] = (keep >> u) & 1u;
            }
    }
    int mine[E];                                    // read before anything is written: the list may be in `out`
#pragma unroll
    for (int u = 0; u < E; ++u) mine[u] = entry(u);
    __syncthreads();
    long long my_tokens = 0;
#pragma unroll
    for (int u = 0; u < E; ++u) {
        if ((keep >> u) & 1u) {
            out[pl.place(u)] = mine[u];
            if (!slots) my_tokens += A.off[mine[u] + 1] - A.off[mine[u]];
        }
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if (slots && nc.count > A.KM && r < A.R) {
        if (r == 1 && A.note_pairs) note_pairs<E>(A, nc.count, keep, [&](int u) { return mine[u]; });
        ncand = nc.count;
        ++r;
        __syncthreads();                            // the list is read by other threads next
        return false;
    }
    nc.active = !slots && nc.count > A.KM;
    end_rounds(A, q, nc, r, slots, my_tokens, sh, kept_tokens);
    return true;
}

constexpr int LIST_ITEMS = 8;                      // entries per thread and trip: loads in flight
constexpr int LIST_CHUNK = SEL_THREADS * LIST_ITEMS;
// A round of a longer list (document ids: cached lists fit a tile; cut down by k_select_segments),
// from memory: the statistics of an entry are read three times (bound, keys above it, prune).
__device__ __forceinline__ void prune_list(const SelArgs& A, int q, int count, QueryCtl nc,
                                           int32_t* out, float2* stat, const float2* bat, bool fold_dense,
                                           int ncand, int r, SelShared& sh, unsigned long long* kept_tokens) {
    const int T = A.T;
    const float a = A.a, b = A.b;
    const int lo = (r - 1) * A.B;
    const int n = lo + A.B < T ? lo + A.B : T;
    const int nb = n - lo;
    const float kappa = A.kappa;                    // (r is the launch's round)
    long long my_tokens = 0;
    merge_segments(out, A.seg_cnt + (size_t)q * SEG_MAX, count);
    if (fold_dense) {                        // the candidates' statistics take the round's batch
#pragma unroll 4
        for (int idx = threadIdx.x; idx < ncand; idx += SEL_THREADS) {
            const int e = out[idx];
            float2 st = stat[e];
            const float2 bb = bat[e];
            merge_stats(st.x, st.y, lo, bb.x, bb.y, nb);
            stat[e] = st;
        }
        __syncthreads();
    }
    auto key_of = [&](int idx) -> uint32_t {
        float lcb, ucb;
        const float2 st = stat[out[idx]];
        interval(st.x, st.y, n, T, kappa, a, b, lcb, ucb);
        return float_key(lcb);
    };
    // A lower bound from a sample of evenly spaced runs, then the K-th largest of the entries that reach
    // it, about ncand / SEL_TILE * K: their keys in LDS, or, where those are too many, the entries in the
    // list buffer that this round no longer reads (3 queries, lists of 39,000 to 82,000, K = 1,000: four
    // rounds 1,010 us, 1,370 by three passes over the whole list).
    const int run_stride = ncand / (SEL_TILE / SEL_RUN);
    uint32_t tkey;
    if ((long long)ncand * A.K > (long long)SEL_TILE * SEL_FEW) {
        int32_t* some = (nc.cur ? A.list0 : A.list1) + (size_t)q * A.N;
        uint32_t bound;
        {
            uint32_t key[SEL_E];
#pragma unroll
            for (int u = 0; u < SEL_E; ++u) {
                const int j = u * SEL_THREADS + (int)threadIdx.x;
                key[u] = key_of((j / SEL_RUN) * run_stride + (j % SEL_RUN));
                if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
            bound = kth_largest_regs<SEL_E>(key, 0xffffu, A.K, sh);
        }
        __syncthreads();                            // n_few is 0
        const int lane = threadIdx.x & 63;
        for (int base = 0; base < ncand; base += LIST_CHUNK) {
            int e[LIST_ITEMS];
            uint32_t key[LIST_ITEMS];
#pragma unroll
            for (int u = 0; u < LIST_ITEMS; ++u) {
                const int idx = base + u * SEL_THREADS + (int)threadIdx.x;
                e[u] = out[idx < ncand ? idx : ncand - 1];
            }
#pragma unroll
            for (int u = 0; u < LIST_ITEMS; ++u) {
                float lcb, ucb;
                const float2 st = stat[e[u]];
                interval(st.x, st.y, n, T, kappa, a, b, lcb, ucb);
                key[u] = float_key(lcb);
            }
#pragma unroll
            for (int u = 0; u < LIST_ITEMS; ++u) {
                const bool hit = base + u * SEL_THREADS + (int)threadIdx.x < ncand && key[u] >= bound;
                const unsigned long long m = __ballot(hit);
                if (m != 0ull) {                    // uniform over the wavefront
                    int at = 0;
                    if (lane == 0) at = atomicAdd(&sh.n_few, __popcll(m));
                    at = __builtin_amdgcn_readlane(at, 0) + __popcll(m & ((1ull << lane) - 1ull));
                    if (hit) some[at] = e[u];
                }
            }
        }
        __syncthreads();
        const int n_some = sh.n_few;
        auto key_some = [&](int idx) -> uint32_t {
            float lcb, ucb;
            const float2 st = stat[some[idx]];
            interval(st.x, st.y, n, T, kappa, a, b, lcb, ucb);
            return float_key(lcb);
        };
        tkey = kth_largest_list(n_some, A.K, key_some, sh);
    } else {
        uint32_t top = 0u;
        for (int base = 0; base < SEL_TILE; base += LIST_CHUNK) {
#pragma unroll
            for (int u = 0; u < LIST_ITEMS; ++u) {
                const int j = base + u * SEL_THREADS + (int)threadIdx.x;
                const uint32_t k = key_of((j / SEL_RUN) * run_stride + (j % SEL_RUN));
                top = k > top ? k : top;
            }
        }
        const uint32_t bound = lower_bound_key(top, A.K, sh);
        // the keys that reach it, then the K-th largest of those
        for (int base = 0; base < ncand; base += LIST_CHUNK) {
            uint32_t key[LIST_ITEMS];
#pragma unroll
            for (int u = 0; u < LIST_ITEMS; ++u) {
                const int idx = base + u * SEL_THREADS + (int)threadIdx.x;
                key[u] = idx < ncand ? key_of(idx) : 0u;
            }
#pragma unroll
            for (int u = 0; u < LIST_ITEMS; ++u)
                collect_few(key[u], base + u * SEL_THREADS + (int)threadIdx.x < ncand && key[u] >= bound, sh);
        }
        if (!kth_of_few(A.K, tkey, sh)) tkey = kth_largest_list(ncand, A.K, key_of, sh);
    }
    const float tau = key_float(tkey);
    // Stable compaction of {entry : UCB >= tau} in place: a chunk is read completely
    // before anything is written, and writes stay below the next chunk.  Software pipeline over
    // chunks: the entries are fetched two chunks ahead and their statistics one chunk ahead,
    // so the loads are in flight across this chunk's scan and its barriers.
    const size_t tro = ((size_t)(r - 1) * A.nq + q) * A.N;
    const int t0 = threadIdx.x * LIST_ITEMS;         // LIST_ITEMS consecutive entries
    int kept = 0;
    auto load_e = [&](int start, int (&e)[LIST_ITEMS]) {
#pragma unroll
        for (int u = 0; u < LIST_ITEMS; ++u) {
            const int idx = start + t0 + u;
            e[u] = idx < ncand ? out[idx] : 0;
        }
    };
    auto load_s = [&](int start, const int (&e)[LIST_ITEMS], float2 (&st)[LIST_ITEMS]) {
#pragma unroll
        for (int u = 0; u < LIST_ITEMS; ++u)
            st[u] = (start + t0 + u < ncand) ? stat[e[u]] : make_float2(0.f, 0.f);
    };
    int e[LIST_ITEMS], e_next[LIST_ITEMS];
    float2 st[LIST_ITEMS];
    load_e(0, e);
    load_s(0, e, st);
    load_e(LIST_CHUNK, e_next);
    for (int start = 0; start < ncand; start += LIST_CHUNK) {
        const int i0 = start + t0;
        int e_next2[LIST_ITEMS];
        float2 st_next[LIST_ITEMS];
        load_s(start + LIST_CHUNK, e_next, st_next);
        load_e(start + 2 * LIST_CHUNK, e_next2);
        unsigned keep = 0;
#pragma unroll
        for (int u = 0; u < LIST_ITEMS; ++u) {
            if (i0 + u < ncand) {
                float lcb, ucb;
                interval(st[u].x, st[u].y, n, T, kappa, a, b, lcb, ucb);
                const bool kp = ucb >= tau;
                keep |= (kp ? 1u : 0u) << u;
                if (A.tr_lcb) {
                    A.tr_lcb[tro + e[u]] = lcb;
                    A.tr_ucb[tro + e[u]] = ucb;
                    A.tr_alive[tro + e[u]] = kp ? 1 : 0;
                }
            }
        }
        if (__syncthreads_or(keep != 0)) {
            int total;
            int pos = kept + block_excl_scan(__popc(keep), sh.wtot, total);
#pragma unroll
            for (int u = 0; u < LIST_ITEMS; ++u)
                if (keep & (1u << u)) {
                    out[pos++] = e[u];
                    my_tokens += A.off[e[u] + 1] - A.off[e[u]];
                }
            kept += total;
        }
#pragma unroll
        for (int u = 0; u < LIST_ITEMS; ++u) {
            e[u] = e_next[u];
            st[u] = st_next[u];
            e_next[u] = e_next2[u];
        }
    }
    nc.count = kept;
    if (threadIdx.x == 0) note_round(sh, r, kept, tau);
    nc.active = kept > A.KM;
    end_rounds(A, q, nc, r, false, my_tokens, sh, kept_tokens);
}

struct TopkArgs {
    const QueryCtl* ctl;   // nullptr: all N documents, vals indexed by id
    int32_t* list0;        // the list that is not the query's current one doubles as scratch
    int32_t* list1;        // for candidate positions of long inputs
    const int32_t* cid;
    int cache_cap;
    float* vals;           // [nq][N]; written here for survivors with exact cached cells
    const float* ccell;    // nullptr: every value is there already
    int T, TP;
    int64_t N;
    int K;
    int64_t* out_ids;
    float* out_scores;
    int32_t* seg_cnt;      // [nq][SEG_MAX]
};

// The winners of at most E * SEL_THREADS candidates, held in registers: into cs / ci, in no order.
template <int E>
__device__ __forceinline__ void topk_regs(const float* vals, const int32_t* list, const int32_t* cid,
                                          const int32_t* scratch, bool segmented, int count, int ncand, int Kq,
                                          float* cs, int* ci, int* n_above, const int* seg_first, SelShared& sh) {
    const Spread sp(ncand);
    const unsigned on = sp.mask<E>();
    int p[E];
    float v[E];
    uint32_t key[E];
    if (segmented) {
        const int len = seg_len(count);
#pragma unroll
        for (int u = 0; u < E; ++u) p[u] = scratch[segment_place(sp.at(u), len, seg_first)];
    } else {
#pragma unroll
        for (int u = 0; u < E; ++u) p[u] = sp.at(u);
    }
#pragma unroll
    for (int u = 0; u < E; ++u) v[u] = vals[p[u]];
#pragma unroll
    for (int u = 0; u < E; ++u) key[u] = float_key(v[u]);
    const uint32_t tkey = kth_largest_regs<E>(key, on, Kq, sh);
    // winners above the K-th value in any order (they are ranked below), those equal to
    // it in index order as far as there is room
    unsigned eq = 0;
    auto put = [&](int slot, int u) {
        const int e = list ? list[p[u]] : p[u];
        cs[slot] = v[u];
        ci[slot] = cid ? cid[e] : e;
    };
#pragma unroll
    for (int u = 0; u < E; ++u)
        if ((on >> u) & 1u) {
            if (key[u] > tkey) put(atomicAdd(n_above, 1), u);
            else if (key[u] == tkey) eq |= 1u << u;
        }
    const Places<E> pl(eq, sh);         // its barrier completes n_above
    const int n_gt = *n_above;
#pragma unroll
    for (int u = 0; u < E; ++u)
        if (((eq >> u) & 1u) && n_gt + pl.place(u) < Kq) put(n_gt + pl.place(u), u);
}

// Scores of a query's survivors from its cached cells, a wavefront each, by list position (no list: the slots themselves).
__device__ __forceinline__ void score_cached(const TopkArgs& A, int q, int count, const int32_t* list) {
    float* v = A.vals + (size_t)q * A.N;
    const float* rows = A.ccell + (size_t)q * A.cache_cap * A.TP;
    for (int k = my_wave(); k < count; k += SEL_WAVES) {
        const float* crow = rows + (size_t)(list ? list[k] : k) * A.TP;
        const float x = A.TP == 16 ? cached_score<1>(crow, A.T)
                      : A.TP == 32 ? cached_score<2>(crow, A.T)
                      : A.TP == 64 ? cached_score<4>(crow, A.T) : cached_score<8>(crow, A.T);
        if ((threadIdx.x & 63) == 0) v[k] = x;
    }
    __syncthreads();
}

// The top-K of a query: candidates 0..count-1 (list: the entries they stand for, cid: whose documents these
// are; nullptr: themselves).  segmented: what k_topk_segments left of them in `scratch`.
struct TopkShared {
    float cs[1024];
    int ci[1024];
    int n_above;
};
__device__ __forceinline__ void topk_query(const TopkArgs& A, int q, int count, const int32_t* list, const int32_t* cid,
                                           int32_t* scratch, bool segmented, SelShared& sh, int* seg_first, TopkShared& tk) {
    float* cs = tk.cs;
    int* ci = tk.ci;
    const float* vals = A.vals + (size_t)q * A.N;
    const int Kq = A.K < count ? A.K : count;
    // few candidates, as after most elimination: one wavefront ranks them (k_topk 8 -> 5 us)
    if (count <= 64 && !segmented) {
        if (my_wave() == 0 && count > 0) {
            const int lane = threadIdx.x & 63;
            const int at = lane < count ? lane : count - 1;
            const float v = vals[at];
            int id = list ? list[at] : at;
            if (cid) id = cid[id];
            const uint32_t key = float_key(v);
            int rank = 0;
            for (int j = 0; j < count; ++j) {
                const uint32_t other = __builtin_amdgcn_readlane(key, j);
                rank += other > key || (other == key && __builtin_amdgcn_readlane(id, j) < id);
            }
            if (lane < count && rank < Kq) {
                A.out_ids[(size_t)q * A.K + rank] = id;
                A.out_scores[(size_t)q * A.K + rank] = v;
            }
        }
    } else if (Kq > 0) {
        if (threadIdx.x == 0) tk.n_above = 0;
        clear_hist(sh);
        // candidate positions: all of 0..count-1, or what the pre-filter left of a long input
        // (survivors are few: a longer list of them is scanned whole)
        int ncand = count;
        if (segmented) ncand = segment_starts(A.seg_cnt + (size_t)q * SEG_MAX, count, seg_first);
        if (ncand <= 4 * SEL_THREADS) {
            topk_regs<4>(vals, list, cid, scratch, segmented, count, ncand, Kq, cs, ci, &tk.n_above, seg_first, sh);
        } else if (ncand <= SEL_TILE) {
            topk_regs<SEL_E>(vals, list, cid, scratch, segmented, count, ncand, Kq, cs, ci, &tk.n_above, seg_first, sh);
        } else {
            const int32_t* cand = nullptr;
            if (segmented) {
                ncand = merge_segments(scratch, A.seg_cnt + (size_t)q * SEG_MAX, count);
                cand = scratch;
            }
            auto key_of = [&](int j) -> uint32_t { return float_key(vals[cand ? cand[j] : j]); };
            const uint32_t tkey = kth_largest_list(ncand, Kq, key_of, sh);
            // how many are strictly above the K-th value
            int gt_local = 0;
            for (int j = threadIdx.x; j < ncand; j += SEL_THREADS) gt_local += key_of(j) > tkey;
            int n_gt;
            block_excl_scan(gt_local, sh.wtot, n_gt);
            const int need_eq = Kq - n_gt;
            int base_gt = 0, base_eq = 0;
            for (int start = 0; start < ncand; start += SEL_CHUNK) {
                const int i0 = start + threadIdx.x * SEL_ITEMS;
                float v[SEL_ITEMS];
                int p[SEL_ITEMS];
                unsigned gt = 0, eq = 0;
#pragma unroll
                for (int u = 0; u < SEL_ITEMS; ++u) {
                    p[u] = (i0 + u < ncand) ? (cand ? cand[i0 + u] : i0 + u) : 0;
                    v[u] = (i0 + u < ncand) ? vals[p[u]] : 0.f;
                }
#pragma unroll
                for (int u = 0; u < SEL_ITEMS; ++u) {
                    if (i0 + u < ncand) {
                        const uint32_t key = float_key(v[u]);
                        gt |= (key > tkey ? 1u : 0u) << u;
                        eq |= (key == tkey ? 1u : 0u) << u;
                    }
                }
                if (__syncthreads_or((gt | eq) != 0)) {      // most chunks hold no winner
                    int tot;
                    const int pos = block_excl_scan(__popc(gt) | (__popc(eq) << 16), sh.wtot, tot);
                    int pg = base_gt + (pos & 0xffff), pe = base_eq + (pos >> 16);
#pragma unroll
                    for (int u = 0; u < SEL_ITEMS; ++u) {
                        int slot = -1;
                        if (gt & (1u << u)) slot = pg++;
                        else if (eq & (1u << u)) {
                            if (pe < need_eq) slot = n_gt + pe;
                            ++pe;
                        }
                        if (slot >= 0) {
                            const int e = list ? list[p[u]] : p[u];
                            cs[slot] = v[u];
                            ci[slot] = cid ? cid[e] : e;
                        }
                    }
                    base_gt += tot & 0xffff;
                    base_eq += tot >> 16;
                }
            }
        }
        __syncthreads();
        if (threadIdx.x < Kq) {
            const float v = cs[threadIdx.x];
            const int id = ci[threadIdx.x];
            int rank = 0;
            for (int j = 0; j < Kq; ++j) {
                const float u = cs[j];
                rank += (u > v) || (u == v && ci[j] < id);
            }
            A.out_ids[(size_t)q * A.K + rank] = id;
            A.out_scores[(size_t)q * A.K + rank] = v;
        }
    }
    for (int k = Kq + threadIdx.x; k < A.K; k += SEL_THREADS) {
        A.out_ids[(size_t)q * A.K + k] = -1;
        A.out_scores[(size_t)q * A.K + k] = -__builtin_inff();
    }
}

// Bound by latency and instructions, not by bytes: a list that fits the registers is read once, and
// selection, prune and count of all its rounds run there.
// TOPK (cache_all, or lists that all fit the cell cache and are revealed by no corpus pass): every query ends in this
// launch, which goes on to its top-K; a launch for that cost 6 us of a call of 50, and one for the survivors of queries that
// ended in round 1 as much.
// LONG: lists may be longer than a tile (what they need costs the others registers).
enum { END_NONE = 0, END_CACHE_ALL = 1, END_LAST = 2 };
template <int END, bool LONG>
__device__ __forceinline__ void prune_query(const SelArgs& A, const Kappas& kappas, const TopkArgs& P, int q, SelShared& sh) {
    __shared__ int seg_first[SEG_MAX + 1];
    __shared__ unsigned long long kept_tokens;
    QueryCtl c{};
    c.count = (int)A.N;
    c.implicit = c.active = 1;
    constexpr bool TOPK = END != END_NONE;
    if constexpr (END != END_CACHE_ALL) c = A.ctl[q];   // (cache_all: round 1, all documents)
    if (!TOPK && !c.active) return;
    // what is left (TOPK): of a query that finished in round 1 all of its list, whose cells are cached since
    int left = c.count;
    const int32_t* survivors = nullptr;
    if (END != END_LAST || c.active) {
    const int count = c.count;
    const int32_t* in = c.implicit ? nullptr : (c.cur ? A.list1 : A.list0) + (size_t)q * A.N;
    const int out_sel = c.implicit ? 0 : (c.cur ^ 1);
    int32_t* out = (out_sel ? A.list1 : A.list0) + (size_t)q * A.N;
    // entries are cache slots if this round's gather has cached the cells (same rule as in
    // k_gather_round); an active query's list always came as ids, for cached rounds end here
    const bool dense = A.dense.thr != NEVER_DENSE && A.dense.pass(A.pairs + A.r);
    const bool slots = A.cache_all || (!c.implicit && count <= A.cache_cap && !dense);
    float2* stat = slots ? A.cstat + (size_t)q * A.cache_cap : A.stat + (size_t)q * A.N;
    const float2* bat = A.stat2 + (size_t)q * A.N;
    const bool fold_dense = dense && in != nullptr;   // a batch that a dense pass left in stat2
    if (slots) in = nullptr;                        // slot = place in the list of ids
    if (threadIdx.x == 0) kept_tokens = 0ull;
    clear_hist(sh);

    const bool segmented = LONG && count > SEL_TILE;        // then k_select_segments has run
    int ncand = count;
    if (segmented) ncand = segment_starts(A.seg_cnt + (size_t)q * SEG_MAX, count, seg_first);

    QueryCtl nc;
    nc.cur = out_sel;
    nc.implicit = 0;
    nc.mode = slots ? 1 : 0;
    nc.bound = nc.done = nc.pad = 0;
    int r = A.r;
    bool from_cells = A.fold_cells != 0;            // the round's batch still has to be folded in
    bool seg = segmented, fold = fold_dense;        // (of the launch's round)
    if constexpr (LONG) {
        if (ncand > SEL_TILE) {
            prune_list(A, q, count, nc, out, stat, bat, fold, ncand, r, sh, &kept_tokens);
            return;
        }
    }
    for (;;) {
        bool done = true;
        if (slots && ncand <= WAVE_LIST) {
            if (my_wave() == 0) prune_wave(A, kappas, q, in, out, stat, ncand, r, from_cells, sh);
            __syncthreads();
            nc.count = sh.pick[0];
            r = sh.pick[1];
            nc.active = 0;
            end_rounds(A, q, nc, r, true, 0, sh, &kept_tokens);
        } else done =
            ncand <= SEL_REGS * SEL_THREADS
                ? prune_regs(A, kappas, q, count, nc, in, out, stat, bat, slots, fold, seg, ncand, r, from_cells, sh, seg_first, &kept_tokens)
                : prune_tile(A, kappas, q, count, nc, in, out, stat, bat, slots, fold, seg, ncand, r, from_cells, sh, seg_first, &kept_tokens);
        if (done) {
            if constexpr (!TOPK) return;
            break;
        }
        // cached rounds remain: on from the shorter list, into the other buffer
        from_cells = true;
        seg = fold = false;
        in = out;
        nc.cur ^= 1;
        out = (nc.cur ? A.list1 : A.list0) + (size_t)q * A.N;
    }
    if constexpr (TOPK) {
        __syncthreads();                            // the list is read by other threads next
        left = sh.round_count[r - 1];
        survivors = out;
    }
    }
    if constexpr (TOPK) {
        __shared__ TopkShared tk;
        score_cached(P, q, left, survivors);
        topk_query(P, q, left, survivors, END == END_CACHE_ALL ? nullptr : A.cid + (size_t)q * A.cache_cap, nullptr, false, sh, seg_first, tk);
    }
}

template <int END, bool LONG>
__global__ __launch_bounds__(SEL_THREADS) void k_select_prune(SelArgs A, Kappas kappas, TopkArgs P) {
    __shared__ SelShared sh;
    prune_query<END, LONG>(A, kappas, P, (int)blockIdx.x, sh);
}

// Cheap outer estimate of interval() for the pre-filter: reciprocal multiplications and the
// hardware square root, each good to a few units in the last place, and an allowance of 64 such
// units of the largest term: lo <= LCB and hi >= max(LCB, UCB) (cells outside [a,b] can put the
// LCB above the UCB, and the K largest LCBs must stay); n, T, kappa, a, b are uniform.
struct FastBounds {
    float c_hat, c_sig, rest_a, rest_b, mag;
    bool hybrid;        // else the hard bounds only (n <= 1), or the exact sum (n >= T: rest = 0)
};
__device__ __forceinline__ FastBounds fast_bounds_consts(int n, int T, float kappa, float a, float b) {
    FastBounds f;
    f.hybrid = n > 1 && n < T;
    f.c_hat = f.hybrid ? (float)T / (float)n : 1.f;
    f.c_sig = f.hybrid ? kappa * kappa / (float)(n - 1) : 0.f;
    f.rest_a = (float)(T - n) * a;
    f.rest_b = (float)(T - n) * b;
    f.mag = fmaxf(fabsf(f.rest_a), fabsf(f.rest_b));
    return f;
}
__device__ __forceinline__ float fast_radius(float M2, const FastBounds& f) {
    return __builtin_amdgcn_sqrtf(fmaxf(M2, 0.f) * f.c_sig);
}
__device__ __forceinline__ float fast_hi(float S, float M2, const FastBounds& f) {
    const float est = S * f.c_hat, r = fast_radius(M2, f);
    float hi = S + f.rest_b;
    if (f.hybrid) hi = fmaxf(fminf(hi, est + r), fmaxf(S + f.rest_a, est - r));
    return hi + 8e-6f * (fabsf(est) + r + f.mag);
}
// key of the lower estimate; a document outside the contract (statistics not finite) has the
// interval [-inf, -inf]
__device__ __forceinline__ uint32_t fast_lo_key(float S, float M2, const FastBounds& f) {
    const float est = S * f.c_hat, r = fast_radius(M2, f);
    float lo = S + f.rest_a;
    if (f.hybrid) lo = fmaxf(lo, est - r);
    lo -= 8e-6f * (fabsf(est) + r + f.mag);
    const bool bad = (__float_as_uint(S) & 0x7fffffffu) >= 0x7f800000u || is_nan_bits(M2);
    return bad ? 0u : float_key(lo);
}

// Lower threshold of a long round-1 list: the K-th largest LCB of a sample of SEL_TILE entries,
// evenly spaced runs of SEL_RUN adjacent ones (whole cache lines; any subset gives a valid lower
// threshold, an even one a close one whatever the order of the corpus).  One workgroup per query.
// Left in QueryCtl::bound.
__global__ __launch_bounds__(SEL_THREADS) void k_select_sample(SelArgs A) {
    __shared__ SelShared sh;
    const int q = blockIdx.x;
    const QueryCtl c = A.ctl[q];
    if (!c.active || !c.implicit || c.count <= SEL_TILE) return;
    const float2* stat = A.stat + (size_t)q * A.N;
    const FastBounds fb = fast_bounds_consts(A.n, A.T, A.kappa, A.a, A.b);
    clear_hist(sh);
    const int run_stride = c.count / (SEL_TILE / SEL_RUN);
    float2 st[SEL_E];
    uint32_t key[SEL_E];
#pragma unroll
    for (int u = 0; u < SEL_E; ++u) {
        const int j = u * SEL_THREADS + (int)threadIdx.x;
        st[u] = stat[(j / SEL_RUN) * run_stride + (j % SEL_RUN)];
    }
#pragma unroll
    for (int u = 0; u < SEL_E; ++u) key[u] = fast_lo_key(st[u].x, st[u].y, fb);
    const uint32_t bound = kth_largest_regs<SEL_E>(key, 0xffffu, A.K, sh);
    if (threadIdx.x == 0) A.ctl[q].bound = (int)bound;
}

// Pre-filter of a long active list, a workgroup per segment (one workgroup per query cannot pull a
// multi-megabyte list from memory fast enough).  Each tile of the segment is read once into
// registers and {UCB >= threshold} is kept, in order, at the start of the segment of the output
// list.  The threshold of round 1 comes from k_select_sample; the lists of later rounds are seldom
// this long, and rather than launch the sampler in each of them every tile takes a lower bound
// of its own K-th largest LCB (that of a part of the list cannot exceed that of the whole).
// 64 M entries of 8 bytes (128 queries x 500,000): 145 us = 3.5 TB/s with a given threshold, bound by
// about 24 instructions an entry; 285 us with the tiles' own thresholds and as much when every
// workgroup sampled for itself.
// In a corpus-pass round the round's batch (stat2) is merged in registers only: k_select_prune
// stores the merged statistics of the survivors, the only entries that are ever read again.
// Workgroup `first` of `step` that share the query's segments (none, if there are fewer).  The control is a copy, and
// k_select_segments leaves the look at `first` to the loop: with a reference and a look of its own the compiled loop took
// 9.9 us in the place of 9.3 (67,406 documents x 30, round 1).
__device__ __forceinline__ void filter_segments(const SelArgs& A, int q, const QueryCtl c, int first, int step, SelShared& sh) {
    const int count = c.count;
    const int len = seg_len(count);
    const int n_seg = seg_count(count);
    const bool dense = A.dense.thr != NEVER_DENSE && A.dense.pass(A.pairs + A.r);
    const int32_t* in = c.implicit ? nullptr : (c.cur ? A.list1 : A.list0) + (size_t)q * A.N;
    const int out_sel = c.implicit ? 0 : (c.cur ^ 1);
    int32_t* out = (out_sel ? A.list1 : A.list0) + (size_t)q * A.N;
    const float2* stat = A.stat + (size_t)q * A.N;
    const float2* bat = A.stat2 + (size_t)q * A.N;
    const bool fold = dense && in != nullptr;
    const int n = A.n, T = A.T;
    const float kappa = A.kappa, a = A.a, b = A.b;
    const FastBounds fb = fast_bounds_consts(n, T, kappa, a, b);
    const size_t tro = ((size_t)(A.r - 1) * A.nq + q) * A.N;
    clear_hist(sh);
    for (int sg = first; sg < n_seg; sg += step) {
        const int lo = sg * len;
        const int hi = seg_end(lo, len, count);
        int base = lo;
        for (int start = lo; start < hi; start += SEG_TILE) {
            const int left = hi - start < SEG_TILE ? hi - start : SEG_TILE;
            const Spread sp(left);
            const unsigned ok = sp.mask<SEG_E>();
            float2 st[SEG_E];
            auto at = [&](int u) { return start + sp.at(u); };
            if (in) {
                int e[SEG_E];
#pragma unroll
                for (int u = 0; u < SEG_E; ++u) e[u] = in[at(u)];
#pragma unroll
                for (int u = 0; u < SEG_E; ++u) st[u] = stat[e[u]];
                if (fold) {
#pragma unroll
                    for (int u = 0; u < SEG_E; ++u) {
                        const float2 bb = bat[e[u]];
                        merge_stats(st[u].x, st[u].y, A.n_prev, bb.x, bb.y, A.nb);
                        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                }
            } else {
#pragma unroll
                for (int u = 0; u < SEG_E; ++u) st[u] = stat[at(u)];
            }
            uint32_t bound = (uint32_t)c.bound;
            if (in) {
                uint32_t top = 0u;
#pragma unroll
                for (int u = 0; u < SEG_E; ++u) {
                    const uint32_t k = (ok >> u) & 1u ? fast_lo_key(st[u].x, st[u].y, fb) : 0u;
                    top = k > top ? k : top;
                }
                bound = lower_bound_key(top, A.K, sh);
            }
            const float thr = key_float(bound);
            unsigned keep = ok;
            if (thr > -__builtin_inff()) {              // else all, also documents outside the contract
#pragma unroll
                for (int u = 0; u < SEG_E; ++u)
                    if (!(fast_hi(st[u].x, st[u].y, fb) >= thr)) keep &= ~(1u << u);
            }
            if (A.tr_lcb) {                             // the trace records every dropped entry's interval
#pragma unroll 1
                for (int u = 0; u < SEG_E; ++u) {
                    if (!(((ok & ~keep) >> u) & 1u)) continue;
                    const int e = in ? in[at(u)] : at(u);
                    float2 x = stat[e];
                    if (fold) {
                        const float2 bb = bat[e];
                        merge_stats(x.x, x.y, A.n_prev, bb.x, bb.y, A.nb);
                    }
                    float lcb, ucb;
                    interval(x.x, x.y, n, T, kappa, a, b, lcb, ucb);
                    A.tr_lcb[tro + e] = lcb;
                    A.tr_ucb[tro + e] = ucb;
                    A.tr_alive[tro + e] = 0;
                }
            }
            const Places<SEG_E> pl(keep, sh);
#pragma unroll
            for (int u = 0; u < SEG_E; ++u)
                if ((keep >> u) & 1u) out[base + pl.place(u)] = in ? in[at(u)] : at(u);
            base += pl.total;
            __syncthreads();
        }
        if (threadIdx.x == 0) A.seg_cnt[(size_t)q * SEG_MAX + sg] = base - lo;
    }
}

__global__ __launch_bounds__(SEL_THREADS, 8) void k_select_segments(SelArgs A) {
    __shared__ SelShared sh;
    const int q = blockIdx.y;
    const QueryCtl c = A.ctl[q];
    if (!c.active || c.count <= SEL_TILE) return;   // cached lists are never this long
    filter_segments(A, q, c, (int)blockIdx.x, (int)gridDim.x, sh);
}

// Pre-filter and prune of a round >= 2 in one launch, for calls whose lists are expected to be short by then
// (Knobs::narrow) and whose workgroups, which need a CU each, take two turns at most.  Of a short list the first workgroup
// prunes at once, and the launch spared is 2.6 us in every round (64 queries x 50,000 472 -> 463 us, 13 x 91,000 in rounds
// of 4 out of 123 tokens 867 -> 805).  Of a long list the last workgroup to come prunes (QueryCtl::done, which the prune
// clears); what the others wrote has to go through memory to it, some 8 us a round, so that a call gains unless its lists
// are long in a quarter of its rounds: 38 x 66,000 with alpha 0.25 479 -> 469 us, 0.3 534 -> 526, 0.5 844 -> 834, but
// 1.0 (34,000, then 22,000 entries) 1,881 -> 1,898.  K and delta lengthen lists as well, by less: alpha 0.25, K = 200, delta
// 1e-30 and rounds of 2, 3 x 130,000 (72,000 and 51,000 entries) 2,682 -> 2,655; K = 1,000 in rounds of 4, 4 x 500,000
// (264,000, 113,000, 30,000) 7,724 -> 7,759.  (With a fence by every wavefront 38 x 66,000 took 1,973.)
// The queries are the fast axis of the grid: workgroups go to the XCDs in turn, and with eight or sixteen to a query those
// that prune short lists, the first of each, all ran on one XCD of the eight (64 queries x 60,000 documents of 51 tokens, lists
// of some 500 entries in round 2: two turns on its 32 CUs, 112 us, 60 now; a call 405 -> 358, on codes of d = 128 431 -> 372).
__global__ __launch_bounds__(SEL_THREADS) void k_select_round(SelArgs A, Kappas kappas) {
    __shared__ SelShared sh;
    __shared__ int last;
    const int q = blockIdx.x;
    const QueryCtl c = A.ctl[q];
    if (!c.active) return;
    if (c.count > SEL_TILE) {
        if ((int)blockIdx.y < seg_count(c.count)) filter_segments(A, q, c, (int)blockIdx.y, (int)gridDim.y, sh);
        // Every wavefront waits until its own stores are in L2, which the barrier alone does not wait for: the write-back of
        // one thread's fence takes what is there.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        // All workgroups count, also those without a segment: none reads the control after the prune has changed it.  (One
        // thread's fences, between the barriers, serve them all; each writes a whole L2 back.)
        if (threadIdx.x == 0) {
            __threadfence();                        // the segments, for whichever workgroup prunes
            last = atomicAdd(&A.ctl[q].done, 1) == (int)gridDim.y - 1;
            if (last) __threadfence();
        }
        __syncthreads();
        if (!last) return;
    } else if (blockIdx.y > 0) return;              // (a list is never longer after a round)
    prune_query<END_NONE, true>(A, kappas, TopkArgs{}, q, sh);
}

// Segment workgroups per query: a list of any length up to N has at most this many segments
// (seg_len: one per tile up to SEG_MAX tiles, at most SEG_MAX beyond).
static unsigned segments_of(int64_t N) {
    const int64_t tiles = (N + SEG_TILE - 1) / SEG_TILE;
    return (unsigned)(tiles < SEG_MAX ? tiles : SEG_MAX);
}

static TopkArgs topk_args(const Problem& P, const Work& W, bool use_ctl, bool cached, float* vals, int K,
                          int64_t* out_ids, float* out_scores) {
    TopkArgs A{};
    A.ctl = use_ctl ? W.ctl : nullptr;
    A.list0 = W.list[0];
    A.list1 = W.list[1];
    A.cid = W.cid;
    A.cache_cap = W.cache_cap;
    A.vals = vals;
    A.ccell = cached ? W.ccell : nullptr;
    A.T = P.T;
    A.TP = W.TP;
    A.N = P.N;
    A.K = K;
    A.out_ids = out_ids;
    A.out_scores = out_scores;
    A.seg_cnt = W.seg_cnt;
    return A;
}

hipError_t launch_select_prune(const Problem& P, const Work& W, const Knobs& kn,
                               const RevealRound& rr, int R, const float* kappa, bool cache_all, bool fold_cells,
                               bool note_pairs, const DenseRule& next, bool finish_next, const Trace& tr, int64_t* topk_ids, float* topk_scores, hipStream_t st) {
    SelArgs A{};
    A.cache_all = cache_all ? 1 : 0;
    A.finish_next = finish_next ? 1 : 0;
    A.fold_cells = fold_cells ? 1 : 0;
    A.note_pairs = cache_all && note_pairs ? 1 : 0;
    TopkArgs top{};
    if (topk_ids) top = topk_args(P, W, false, true, W.rescored, kn.K, topk_ids, topk_scores);
    A.ctl = W.ctl;
    A.list0 = W.list[0];
    A.list1 = W.list[1];
    A.stat = W.stat;
    A.stat2 = W.stat2;
    A.pairs = W.pairs;
    A.work = W.work;
    A.off = P.off;
    A.R = R;
    A.dense = rr.dense;
    A.N = P.N;
    A.nq = P.nq;
    A.T = P.T;
    A.B = kn.B;
    A.K = kn.K;
    A.KM = kn.K + kn.M;
    A.r = rr.r;
    A.n = rr.n;
    A.n_prev = rr.n_prev;
    A.nb = rr.nb;
    A.a = kn.a;
    A.b = kn.b;
    A.pi = W.pi;
    A.cache_cap = W.cache_cap;
    A.TP = W.TP;
    A.cid = W.cid;
    A.cstat = W.cstat;
    A.ccell = W.ccell;
    A.cnt_hist = W.cnt_hist;
    A.tau_hist = W.tau_hist;
    A.tr_count = tr.count;
    A.tr_tau = tr.tau;
    A.tr_lcb = tr.lcb;
    A.tr_ucb = tr.ucb;
    A.tr_alive = tr.alive;
    A.seg_cnt = W.seg_cnt;
    A.kappa = kappa[rr.r];
    A.enough = next.enough;
    A.certain = next.certain();
    Kappas kappas{};
    for (int r = 0; r <= R; ++r) kappas.of[r] = kappa[r];
    // lists that do not fit one workgroup's registers are first cut down, one workgroup per tile
    if (P.N > SEL_TILE) {
        unsigned gx = segments_of(P.N);
        if (rr.r == 1) {
            k_select_sample<<<P.nq, SEL_THREADS, 0, st>>>(A);
        } else {
            // later lists are seldom long: no more workgroups than end quickly with nothing to do
            const unsigned few = (unsigned)(2048 / P.nq > 1 ? 2048 / P.nq : 1);
            gx = gx < few ? gx : few;
            if (kn.narrow && gx * (unsigned)P.nq <= 512u) {
                k_select_round<<<dim3(P.nq, gx), SEL_THREADS, 0, st>>>(A, kappas);
                return hipGetLastError();
            }
        }
        k_select_segments<<<dim3(gx, P.nq), SEL_THREADS, 0, st>>>(A);
    }
    if (P.N > SEL_TILE) k_select_prune<END_NONE, true><<<P.nq, SEL_THREADS, 0, st>>>(A, kappas, top);
    else if (topk_ids && cache_all) k_select_prune<END_CACHE_ALL, false><<<P.nq, SEL_THREADS, 0, st>>>(A, kappas, top);
    else if (topk_ids) k_select_prune<END_LAST, false><<<P.nq, SEL_THREADS, 0, st>>>(A, kappas, top);   // (lists fit the cache)
    else k_select_prune<END_NONE, false><<<P.nq, SEL_THREADS, 0, st>>>(A, kappas, top);
    return hipGetLastError();
}

// =====================================================================================
// top-K by (value descending, document index ascending), one workgroup per query
// (Eq. (3); final step of Algorithm 1).  Candidates arrive in ascending id order, so
// ties at the K-th value are resolved towards the lower index by taking them in order.
// =====================================================================================
// The pre-filter of k_topk for long all-documents inputs, a workgroup per segment: each tile is
// read once, and the positions whose value reaches a lower bound of the tile's own K-th
// largest (lower_bound_key) go, in order, to the segment's start of the scratch list.
__global__ __launch_bounds__(SEL_THREADS, 8) void k_topk_segments(TopkArgs A) {
    __shared__ SelShared sh;
    const int q = blockIdx.y, sg = blockIdx.x;
    const int count = (int)A.N;
    const int len = seg_len(count);
    if (sg >= seg_count(count)) return;
    const int lo = sg * len;
    const int hi = seg_end(lo, len, count);
    const float* vals = A.vals + (size_t)q * A.N;
    int32_t* tmp = A.list0 + (size_t)q * A.N;
    clear_hist(sh);
    int base = lo;
    for (int start = lo; start < hi; start += SEG_TILE) {
        const int left = hi - start < SEG_TILE ? hi - start : SEG_TILE;
        const Spread sp(left);
        const unsigned ok = sp.mask<SEG_E>();
        float v[SEG_E];
        uint32_t key[SEG_E], top = 0u;
#pragma unroll
        for (int u = 0; u < SEG_E; ++u) v[u] = vals[start + sp.at(u)];
#pragma unroll
        for (int u = 0; u < SEG_E; ++u) {
            key[u] = (ok >> u) & 1u ? float_key(v[u]) : 0u;
            top = key[u] > top ? key[u] : top;
        }
        const uint32_t thr = lower_bound_key(top, A.K, sh);
        unsigned keep = 0;
#pragma unroll
        for (int u = 0; u < SEG_E; ++u) keep |= (key[u] >= thr ? 1u : 0u) << u;
        const Places<SEG_E> pl(keep & ok, sh);
#pragma unroll
        for (int u = 0; u < SEG_E; ++u)
            if (((keep & ok) >> u) & 1u) tmp[base + pl.place(u)] = start + sp.at(u);
        base += pl.total;
        __syncthreads();
    }
    if (threadIdx.x == 0) A.seg_cnt[(size_t)q * SEG_MAX + sg] = base - lo;
}

__global__ __launch_bounds__(SEL_THREADS) void k_topk(TopkArgs A) {
    __shared__ SelShared sh;
    __shared__ int seg_first[SEG_MAX + 1];
    __shared__ TopkShared tk;
    const int q = blockIdx.x;
    int count = (int)A.N;
    const int32_t* list = nullptr;
    const int32_t* cid = nullptr;
    int32_t* scratch = A.list0 + (size_t)q * A.N;
    if (A.ctl) {
        const QueryCtl c = A.ctl[q];
        count = c.count;
        if (!c.implicit) {
            list = (c.cur ? A.list1 : A.list0) + (size_t)q * A.N;
            scratch = (c.cur ? A.list0 : A.list1) + (size_t)q * A.N;
        }
        if (c.mode == 1 && A.cid) cid = A.cid + (size_t)q * A.cache_cap;
        if (c.mode == 1 && A.ccell) score_cached(A, q, count, list);
    }
    topk_query(A, q, count, list, cid, scratch, !A.ctl && count > SEL_TILE, sh, seg_first, tk);
}

hipError_t launch_topk(const Problem& P, const Work& W, bool use_ctl, bool cached, bool cache_all, float* vals, int K,
                       int64_t* out_ids, float* out_scores, hipStream_t st) {
    TopkArgs A = topk_args(P, W, use_ctl, cached, vals, K, out_ids, out_scores);
    if (cache_all) A.cid = nullptr;                 // slots are documents
    if (!use_ctl && P.N > SEL_TILE)
        k_topk_segments<<<dim3(segments_of(P.N), P.nq), SEL_THREADS, 0, st>>>(A);
    k_topk<<<P.nq, SEL_THREADS, 0, st>>>(A);
    return hipGetLastError();
}

// =====================================================================================
// offsets validation
// =====================================================================================
__global__ void k_validate_offsets(const int64_t* off, int64_t N, int64_t total, int* flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x) {
        bool bad = off[i + 1] <= off[i];
        if (i == 0) bad = bad || off[0] < 0 || off[N] > total;
        if (bad) atomicOr(flag, 1);
    }
}
__global__ void k_zero_flag(int* flag) { flag[0] = 0; }

hipError_t launch_validate_offsets(const int64_t* off, int64_t N, int64_t total, int* flag,
                                   hipStream_t st) {
    k_zero_flag<<<1, 1, 0, st>>>(flag);
    int g = (int)((N + 255) / 256);
    if (g > 2048) g = 2048;
    k_validate_offsets<<<g, 256, 0, st>>>(off, N, total, flag);
    return hipGetLastError();
}

}  // namespace cb
