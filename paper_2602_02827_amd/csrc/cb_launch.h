// Host-side launch interface between the C-ABI layer and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cb_device.h"

namespace cb {

enum { DT_F32 = 0, DT_BF16 = 1 };

struct Problem {
    const void* Q;
    int nq, T, d, dt;
    const void* docs;
    const int64_t* off;
    int64_t N, total;
};

// Views into the caller's workspace (all device pointers).
struct Work {
    QueryCtl* ctl;        // [nq]
    int32_t* list[2];     // [nq][N] each: ids of the active set, ascending
    float2* stat;         // [nq][N] per (query, doc): revealed sum, centred sum of squares
    float2* stat2;        // [nq][N] batch (sum, centred squares) of a later round's dense pass
    unsigned long long* pairs;   // [R+2] pairs[r]: (query, doc) pairs round r would have to gather
                                 // and the queries that hold them (pair_count, work_count);
                                 // then [R+2]: the document tokens of those pairs; then as [2], which does not
                                 // count them, the pairs of round 2 whose lists are entered by document; then how many of
                                 // pairs[2] are the survivors of finished queries
    unsigned long long* work;    // [nq] the queries of the next round (work_item), from the end those entered by document
    int32_t* seg_cnt;     // [nq][64] candidates per segment of a segmented pre-filter
    float* rescored;      // [nq][N] exact score of the k-th survivor
    float* scores;        // [nq][N] Full-MaxSim scores when the caller keeps none
    int32_t* cnt_hist;    // [(R+1)][nq]
    float* tau_hist;      // [R][nq]
    int32_t* pi;          // [nq][T]
    int chunk_tokens;     // tokens per chunk of the dense kernel
    int32_t* chunk_doc;   // [nchunks+1] first document of each token chunk
    int* flag;            // [64] error / scratch flags
    // cell cache of queries whose active set has shrunk to <= cache_cap documents
    int cache_cap;        // slots per query (0: caching off)
    int TP;               // floats per slot: T rounded up to whole 16-column tiles
    int32_t* cid;         // [nq][cache_cap] document id of a slot
    float2* cstat;        // [nq][cache_cap] revealed sum / centred squares of a slot
    float* ccell;         // [nq][cache_cap][TP] the slot's MaxSim cells
    // coarse pass: int8 codes of the queries, written per call
    int8_t* q8;           // [nq][T][d]
    float* qscale;        // [nq]
    void* qscratch;       // quantize_scratch_bytes(nq)
};

// int8 codes for the coarse elimination pass (implementation appendix, quantized layout):
// a code c decodes to c * scale.  All device pointers.
struct Coarse {
    const int8_t* docs8;  // [total][d] codes of the document tokens
    const float* dscale;  // [1] their decode scale
    int8_t* Q8;           // [nq][T][d] codes of the queries (written by the call)
    float* qscale;        // [nq] decode scale of each query
};

struct Trace {            // all null when tracing is off
    int32_t* count;
    float* tau;
    float* lcb;
    float* ucb;
    uint8_t* alive;
};

struct RevealRound {
    int r;                // 1-based round
    int lo, nb;           // batch = pi[lo .. lo+nb)
    int n_prev, n;        // cells revealed before / after the round
    // Rounds >= 2 pick their reveal path on the device: the corpus-streaming pass if
    // pairs[r] says (DenseRule), else by gathering.  Every kernel of the round evaluates the
    // same test.  Round 1, whose path the host fixes: never.
    DenseRule dense;
};

constexpr DenseRule kNeverDense{NEVER_DENSE, 0u, 0u, 0, 0};

struct Knobs {
    int K, M, B;
    float a, b;
    bool narrow;          // the radius is small: lists are longer than a tile in few rounds (k_select_round has the figures)
};

// n_chunks > 0: also fills the chunk table of the corpus passes (launch_dense_prepare).
hipError_t launch_init(const Problem& P, const Work& W, const Knobs& kn, int R, uint64_t seed,
                       const int32_t* user_pi, const Trace& tr, const Coarse* co, int n_chunks, hipStream_t st);

// Reveal round rr by gathering the documents of every active (query, document) pair.  Queries whose
// list fits the cell cache get all T cells of their documents computed once and cached;
// k_select_prune and the rescore read them back.
hipError_t launch_gather_round(const Problem& P, const Work& W, const RevealRound& rr, const Coarse* co, hipStream_t st);
// Whether round 2 may gather documents for several queries at a time (rr.dense.enough, k_gather_docs), and the logarithm of
// how many.
bool shares_documents(const Problem& P, const Work& W, const Coarse* co);
int share_group_lg(int T);
unsigned share_enough(const Problem& P);
// The smallest calls, in the place of launch_init: all cells of all documents go to the cell cache (slot =
// document), and the queries are set up in the same launch.
hipError_t launch_cache_all(const Problem& P, const Work& W, const Knobs& kn, int R, uint64_t seed,
                            const int32_t* user_pi, const Trace& tr, const Coarse* co, hipStream_t st);
// Whether it reveals round 1 from them.
bool cache_all_reveals(const Problem& P, const Coarse* co);

// Exact scores from the stored embeddings.  Survivors: of the current active sets, written by
// list position (score_slots: including the queries whose list holds cache slots, whose cached
// cells are coarse and cannot give the exact score).  All: every document of every query, written
// by doc id into `out` ([nq][N]).
hipError_t launch_gather_survivors(const Problem& P, const Work& W, const Knobs& kn, float* out,
                                   bool score_slots, bool cache_all, hipStream_t st);
hipError_t launch_gather_all(const Problem& P, const Work& W, float* out, float* cells, hipStream_t st);
bool gather_shares(const Problem& P);   // launch_gather_all gives a pair a workgroup

// Dense (corpus-streaming) kernel: Full-MaxSim scores or the first reveal batch.
hipError_t launch_dense_prepare(const Problem& P, const Work& W, int* n_chunks,
                                hipStream_t st);
// co != nullptr: the pass runs on the int8 codes (integer matrix instructions, exact int32
// maxima decoded by the two scales) instead of the stored embeddings.
hipError_t launch_dense_score(const Problem& P, const Work& W, int n_chunks,
                              float* out, float* cells, const Coarse* co, hipStream_t st);
hipError_t launch_dense_reveal(const Problem& P, const Work& W, int n_chunks,
                               const RevealRound& rr, int G, const Coarse* co, hipStream_t st);
// The same pass for a round >= 2: runs only if the round's device-side test picks it, writes the
// batch statistics of every (active ids-mode query, document) to stat2; k_select_prune merges
// them into the running statistics of the documents still active.
hipError_t launch_dense_reveal_later(const Problem& P, const Work& W, int n_chunks, const RevealRound& rr, int G, const Coarse* co,
                                     hipStream_t st);
// How an exhaustive pass covers P's queries with column tiles of 16 query tokens.
struct ScoreShape {
    int tq;               // tiles per query: 1, 2, 4 or 8
    int64_t tiles;        // of all queries
    int nt;               // tiles per wavefront
    int split;            // > 0: wavefronts that take the same tiles and split the documents
    int groups;           // column groups (workgroups that stream the same tokens)
};
// codes: a pass on int8 codes.
ScoreShape score_shape(const Problem& P, bool codes);
// Whether a pass over that many column tiles, in one group and no split of the documents, goes to two wavefronts of eight.
bool in_pairs(const Problem& P, int64_t tiles, bool codes);
// fp32 batches that always gather, whatever the corpus (us, 100,000 documents of 100 tokens or 4,000 of 1,030: one query of
// 32 tokens 367 and 487 by a pass, of 48 in d = 64 222 and 391, two of 48 in d = 128 2,467 and 3,410, in d = 32 579 and
// 581, two of 32 in d = 96 within 6 %): there is no corpus kernel for them.
inline bool always_gathers(const ScoreShape& s, int d) {
    return s.split != 0 && (s.tq == 4 || (s.tq == 2 && (s.split == 4 || d == 96)));
}
bool dense_supported(const Problem& P, const Coarse* co);
int dense_chunks(const Problem& P, const Work& W);

// Threshold and prune of round rr; a query whose cells are cached runs all its remaining rounds in
// this launch.  R: number of rounds of the call (layout of W.pairs); kappa[r], r = 1..R: radius
// per unit sigma_hat of round r.  fold_cells: after launch_cache_all, if that has not revealed round 1.  next: in round 1 the rule of round 2, else kNeverDense.  finish_next: round 1 of a
// call whose round 2 is the last to launch and ends with the top-K: the survivors of queries that end in round 1 are
// then gathered with it.  topk_ids (after launch_cache_all, or in that round 2; exact cells): the launch ends with the
// top-K.
hipError_t launch_select_prune(const Problem& P, const Work& W, const Knobs& kn,
                               const RevealRound& rr, int R, const float* kappa, bool cache_all, bool fold_cells,
                               bool note_pairs, const DenseRule& next, bool finish_next, const Trace& tr, int64_t* topk_ids, float* topk_scores, hipStream_t st);

// Top-K of `vals` per query.  use_ctl: candidates are the active set (vals indexed by
// list position); else all N documents (vals indexed by id).  cached: the queries whose list holds
// cache slots take their survivors' scores from the cached cells (and store them in vals).  cache_all: slots
// are documents.
hipError_t launch_topk(const Problem& P, const Work& W, bool use_ctl, bool cached, bool cache_all, float* vals, int K,
                       int64_t* out_ids, float* out_scores, hipStream_t st);

// int8 codes of x ([n_segments][seg_elems] values of dtype dt): per segment, clip = the
// nearest-rank permille/1000 percentile of |x|, code = rint(x * 127 / clip) saturated to
// +-127, scales[seg] = clip / 127.  scratch: quantize_scratch_bytes(n_segments).
size_t quantize_scratch_bytes(int64_t n_segments);
hipError_t launch_quantize_i8(const void* x, int dt, int64_t n_segments, int64_t seg_elems,
                              int permille, int8_t* codes, float* scales, void* scratch,
                              hipStream_t st);

// Doc-Uniform (appendix "Compared Methods"): scores[q][i] = sum of cells[q][i][t] over the
// seeded random subset of m tokens of (q, i); masks (nullable) receives the subsets.
hipError_t launch_uniform_score(const float* cells, int nq, int64_t N, int T, int m, uint64_t seed,
                                float* scores, uint64_t* masks, hipStream_t st);
// Ball-carving (same appendix): greedy clustering of each query's tokens at cosine threshold
// tau.  Cz [nq][T][d] (storage type): centroid c of query q in row c, zero rows past the last;
// labels [nq][T] (nullable): cluster of each token; kq [nq]: clusters per query.
hipError_t launch_ball_carve(const Problem& P, float tau, void* Cz, int32_t* labels, int32_t* kq,
                             hipStream_t st);
// bf16: packs the centroids four to a group.  goff [nq+1]: first group of each query and the
// total; Qg [total groups][4][d]; ident [total groups][4] = 0,1,2,3.
hipError_t launch_ball_groups(const Problem& P, const void* Cz, const int32_t* kq, int32_t* goff,
                              void* Qg, int32_t* ident, hipStream_t st);
// scores[q][i] = sum over the groups of q, ascending, of part[(g * N + i) * stride].
hipError_t launch_ball_reduce(const float* part, int stride, const int32_t* goff, int nq, int64_t N,
                              float* scores, hipStream_t st);

hipError_t launch_validate_offsets(const int64_t* off, int64_t N, int64_t total, int* flag,
                                   hipStream_t st);

}  // namespace cb
