// Dense corpus-streaming MaxSim kernel for bf16 and fp32 embeddings and int8 codes (gfx950).
//
// Shape of the work: a [tokens x d] corpus against a few thousand query rows, d = 32/64/96/128.
// The result matrix is never written; each 16x16 MFMA tile is folded at once into a
// running per-(document, query row) maximum, and a document's maxima are summed when
// its last token has passed (paper Eq. (1)-(2), (4)-(5)).
//
// Mapping onto the machine
//   * A workgroup (4 wavefronts) owns one token chunk (whole documents whose first token
//     falls into a fixed-size token range) and one group of 64*NT query columns.
//   * Query rows are the B operand and stay in registers for the whole kernel: each
//     wavefront holds NT column tiles of 16 rows, full depth (NT*d/8 VGPRs; fp32, in three bf16
//     pieces, NT*d*3/8, hence NT <= 4).
//   * Document tokens are the A operand.  They stream through a four-slot LDS ring of
//     64-token stages (direct global -> LDS copies issued two stages ahead of the reader), so
//     a token is read from memory once per workgroup and from LDS once per wavefront.  fp32 tokens
//     pass through registers instead, are cut into their pieces once per workgroup and lie in LDS in
//     three planes (two slots of 32 tokens).
//     Rows are stored with their 16-byte pieces XOR-swizzled by the row index, which
//     spreads the 16 rows of an operand block over all banks; a row whose length is not a power
//     of two (d = 96) is padded to one in LDS.
//   * The chunk's tokens form one stream of aligned 16-token blocks, whatever the document
//     boundaries, so no token is multiplied twice.  A block inside one document folds into
//     the running maxima directly; where a document ends inside a block the fold is split
//     by accumulator row (block_mma_split_rows / block_mma_split).  Documents of any length
//     >= 1 are handled.  Runs of whole blocks inside one document go through a loop that holds
//     only operand reads and MFMAs.
//   * Workgroup ids are laid out so that the column groups of one token chunk run on the
//     same XCD and share its L2; eight consecutive chunks go to the eight XCDs in a rotating
//     order.
#include "cb_launch.h"

namespace cb {

// A workgroup covers 4 * TILES column tiles with four wavefronts.  fp32 in d = 96 and 128 spreads them
// over eight where it can (a wavefront needs all tiles of a query): four tiles of pieces would leave
// one wavefront per SIMD, and eight wavefronts share the cutting of the tokens (16 queries x 20,000
// documents of d = 128: 1,417 us with four, 1,302 with eight; 32 of 16 tokens at d = 96 1,313 and 1,030).
// PAIR: sixteen tiles of 128-byte rows (codes of d = 128, bf16 of d = 64) go to two wavefronts of eight tiles, which
// read an operand block from LDS half as often for its matrix instructions and meet half as often: Col-Bandit, 64
// queries x 20,000 pages, codes 788 -> 762 us, 36 x 500,000 in d = 64 1,999 -> 1,908, exhaustive, 8 x 50,000 in d = 64 194 -> 186.
// (Other widths lose registers or gain nothing: bf16 of d = 128 64 x 50,000 455 -> 464, 96 474 -> 604, 32 583 -> 614.)
// Their chunks take longer, so they are halved where that fills their turns better (choose_chunks), and there have to be enough (pair_pays): 4 queries of 60 tokens x 1,613
// pages 64 -> 70 us, 11 x 868 documents 21 -> 22, 4 x 17,775 pages 529 -> 512, 7 x 41,000 documents 185 -> 180.
constexpr int PAIR = -2;                           // in the place of a number of wavefronts that split the documents
template <typename Tag, int D, int TILES, int TQ, int SPLIT> constexpr int dense_waves() {
    return SPLIT == PAIR ? 2 : !Tag::wide && D >= 96 && TILES == 4 && TQ <= 2 ? 8 : 4;
}
template <typename Tag, int D> constexpr bool can_pair() { return Tag::wide && D * Frag<Tag, D>::ELEM_BYTES == 128; }
static bool pair_pays(int64_t total, int64_t N) { return total >= 2100000 && N >= 2048; }
// Ring geometry: four stages.  Kernels with few column tiles per wavefront (small query
// batches: bound by memory, little register use) take 32-row stages, so that four workgroups fit
// a CU instead of two and more wavefronts hide the latencies; the others take 64-row stages.
// A_REGS: registers of one operand block (the query rows take NT of them, two token blocks are in
// flight); four, three or two workgroups per CU by what that and the rings' LDS leave.
template <int NT, int PITCH, int A_REGS, int PLANES, int WAVES> struct RingShape {
    static constexpr int ROWS_PER_LOAD = 64 / (PITCH / 16);
    static constexpr bool SMALL = (NT <= 4 || WAVES == 2) && 32 / ROWS_PER_LOAD / WAVES >= 1;
    static constexpr int STAGE_ROWS = SMALL ? 32 : 64;
    static constexpr int RING_ROWS = 4 * STAGE_ROWS;
    static constexpr int REGS = (NT + 2) * A_REGS + 40;
    static constexpr int BY_REGS = REGS <= 128 ? 4 : (REGS <= 168 ? 3 : 2);
    static constexpr int BY_SHAPE = SMALL ? (NT <= 2 ? 4 : 3) : 2;
    static constexpr int BY_LDS = 160 * 1024 / (RING_ROWS * PITCH);
    static constexpr int FIT = BY_REGS < BY_SHAPE ? BY_REGS : BY_SHAPE;
    static constexpr int MIN_BLOCKS = FIT < BY_LDS ? FIT : BY_LDS;   // of four wavefronts: wavefronts per SIMD
    static_assert(MIN_BLOCKS >= 1 && MIN_BLOCKS * RING_ROWS * PITCH <= 160 * 1024, "the rings of a CU's workgroups");
};
// fp32: two slots of 32 rows, each row in three planes of bf16 pieces; the loads of the next stage are
// in registers (16 at most).
template <int NT, int PITCH, int A_REGS, int WAVES> struct RingShape<NT, PITCH, A_REGS, 3, WAVES> {
    static constexpr int STAGE_ROWS = 32;
    static constexpr int RING_ROWS = 2 * STAGE_ROWS;
    static constexpr int REGS = (NT + 2) * A_REGS + 60;
    static constexpr int BY_REGS = REGS <= 128 ? 4 : (REGS <= 168 ? 3 : (REGS <= 256 ? 2 : 1));
    static constexpr int BY_LDS = 160 * 1024 / (RING_ROWS * PITCH * 3);
    static constexpr int MIN_BLOCKS = BY_REGS < BY_LDS ? BY_REGS : BY_LDS;
};
// bytes of a token row, of its place in the ring (a power of two; fp32: in a plane), and how many planes
template <class F, int D> struct RowShape {
    static constexpr int BYTES = D * F::ELEM_BYTES;
    static constexpr int PLANES = F::ELEM_BYTES == 4 ? 3 : 1;
    static constexpr int PLACE = PLANES == 3 ? D * 2 : BYTES;
    static constexpr int PITCH = PLACE <= 64 ? 64 : PLACE <= 128 ? 128 : 256;
    static constexpr int A_REGS = (int)sizeof(F) / 4;
};

struct DenseArgs {
    const void* Q;
    const void* docs;
    const int64_t* off;
    const int32_t* chunk_doc;
    int64_t N, total;
    int nq, T;
    int n_chunks, n_groups;
    int hq;                  // PACKED: half tiles (8 columns) per query
    // score
    float* out;
    float* cells;
    // reveal
    const int32_t* pi;
    int lo, nb, G;
    float2* stat;
    // a round >= 2: run only if dense.pass(pairs_r); skip queries that are
    // finished or read their cells from the cache
    const unsigned long long* pairs_r;
    DenseRule dense;
    const QueryCtl* ctl;
    // int8 codes: a cell is the integer maximum times qscale[q] * dscale[0]
    const float* qscale;
    const float* dscale;
};

// PACKED: query lengths that leave a quarter or more of their column tiles empty (T = 17..24,
// 33..48, 65..96, up to 8).  A wavefront takes as many queries as eight whole tiles would hold, but at
// half tiles each, in six tiles; the maxima of a document then pass through LDS into the layout
// whose sum every other kernel takes.  A quarter of the matrix work less, and as much less to fold, in
// every width; 64 queries of 24 tokens over 20,000 pages of 1,030 tokens 6.84 -> 5.49 ms (d = 32: 1.82 ->
// 1.43), of 40 tokens over 6.4 M tokens 4.43 -> 3.49.
constexpr int PACKED_NT = 6;
template <typename Tag, int D, int TILES, int TQ, bool REVEAL, int SPLIT = 0, bool PACKED = false>
__global__ __launch_bounds__((64 * dense_waves<Tag, D, TILES, TQ, SPLIT>()),
                             (RingShape<TILES * 4 / dense_waves<Tag, D, TILES, TQ, SPLIT>(), RowShape<Frag<Tag, D>, D>::PITCH,
                                        RowShape<Frag<Tag, D>, D>::A_REGS, RowShape<Frag<Tag, D>, D>::PLANES,
                                        dense_waves<Tag, D, TILES, TQ, SPLIT>()>::MIN_BLOCKS))
void k_dense(DenseArgs A) {
    using F = Frag<Tag, D>;
    constexpr int SPLIT_DOCS = SPLIT > 0 ? SPLIT : 0;
    constexpr int WAVES = dense_waves<Tag, D, TILES, TQ, SPLIT>();
    constexpr int NT = TILES * 4 / WAVES;          // column tiles of a wavefront
    constexpr int PLANES = RowShape<F, D>::PLANES;
    using RS = RingShape<NT, RowShape<F, D>::PITCH, RowShape<F, D>::A_REGS, PLANES, WAVES>;
    constexpr int STAGE_ROWS = RS::STAGE_ROWS;
    constexpr int RING_ROWS = RS::RING_ROWS;
    using V = typename F::val_t;           // float, or int for int8 codes
    constexpr bool CODES = !__is_same(V, float);
    constexpr int ROWB = RowShape<F, D>::BYTES;    // bytes per token row in memory
    constexpr int PITCH = RowShape<F, D>::PITCH;   // ... and in the ring
    constexpr int NCH = PITCH / 16;                // 16-byte pieces per ring row
    constexpr bool F32 = __is_same(Tag, f32_tag);
    // Cache policy of the token copies (not of fp32, whose tokens pass through registers).  The reveal pass
    // normally has one column group, and the score kernels with at most four column tiles per wavefront
    // always have: a token row is read once and should not push other lines out of L2 - above all those
    // of the (sum, M2) array, which fill up over several documents; such copies carry the non-temporal
    // hint (bit 1).
    constexpr int LOAD_POLICY = (REVEAL || TILES <= 4) ? 2 : 0;
    // Swizzle key of a ring row: rows whose 16-byte pieces would fall on the same banks (row
    // stride PITCH against the 256-byte bank window) get different keys.  The key's period must
    // divide the rows of one load of all wavefronts, of fp32 those of a stage.
    constexpr int KEY_SHIFT = NCH >= 16 ? 0 : (NCH == 8 ? 1 : 2);
    constexpr int KEY_MASK = NCH - 1;
    __shared__ __attribute__((aligned(16))) char ring[PLANES * RING_ROWS * PITCH];

    if constexpr (REVEAL) {
        if (A.pairs_r && !A.dense.pass(A.pairs_r)) return;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, in an SGPR
    const int col = lane & 15;
    const int kg = lane >> 4;

    // workgroup -> (token chunk, column group); chunks of one XCD are contiguous in `slot`
    const int b = blockIdx.x;
    const int xcd = b & 7, slot = b >> 3;
    const int group = slot % A.n_groups;
    // Eight consecutive chunks go to the eight XCDs, rotated from one eight to the next by a
    // mix of its number: documents much longer than a chunk leave all but every 2^k-th chunk
    // empty, and a fixed chunk -> XCD map would then put all the work on a few XCDs.
    const int k8 = slot / A.n_groups;
    const int chunk = k8 * 8 + ((xcd + k8 + (k8 >> 3) + (k8 >> 6) + (k8 >> 9)) & 7);
    if (chunk >= A.n_chunks) return;
    int i0 = A.chunk_doc[chunk], i1 = A.chunk_doc[chunk + 1];
    i0 = i0 < 0 ? 0 : (i0 > (int)A.N ? (int)A.N : i0);
    i1 = i1 < i0 ? i0 : (i1 > (int)A.N ? (int)A.N : i1);
    if (i0 >= i1) return;
    int64_t tok_begin = A.off[i0], tok_end = A.off[i1];
    tok_begin = tok_begin < 0 ? 0 : (tok_begin > A.total ? A.total : tok_begin);
    tok_end = tok_end < tok_begin ? tok_begin : (tok_end > A.total ? A.total : tok_end);
    const int ntok = (int)(tok_end - tok_begin);
    if (ntok <= 0) return;

    const int lgG = REVEAL ? 31 - __builtin_clz(A.G > 0 ? A.G : 1) : 0;   // G is a power of two
    // ---- query rows of this wavefront's column tiles -> B fragments (registers)
    // When the column tiles of the launch fit into one or two of the four wavefronts (one or two
    // queries), the others would only repeat their work.  Instead SPLIT_DOCS (4 or 2) wavefronts
    // take the same tiles and split the chunk's DOCUMENTS among themselves: a wavefront
    // multiplies the blocks inside its own documents (every fourth, or every second) and every
    // block in which a document ends, and writes the scores of its own documents only.  All four
    // still walk the same block stream, so the stage barriers match up.  (SPLIT_DOCS: the launch
    // has one column group.)  15.9 M tokens, bf16: 1.03 -> 0.77 ms for one query of 42 tokens, 1.03 ->
    // 0.88 for two, 1.63 -> 1.29 and 1.64 -> 1.40 with 100 tokens.
    static_assert(SPLIT_DOCS == 0 || ((SPLIT_DOCS == 2 || SPLIT_DOCS == 4) && !REVEAL),
                  "document splitting is for small batches of the score kernels");
    constexpr int TILE_WAVES = SPLIT_DOCS ? 4 / SPLIT_DOCS : 4;      // wavefronts with tiles of their own
    const int tile0 = SPLIT_DOCS ? (wave % TILE_WAVES) * NT : (group * WAVES + wave) * NT;
    auto mine = [&](int doc) {
        return SPLIT_DOCS == 0 || ((doc - i0) & (SPLIT_DOCS ? SPLIT_DOCS - 1 : 0)) == wave / TILE_WAVES;
    };
    static_assert(!PACKED || (!REVEAL && SPLIT_DOCS == 0 && NT == PACKED_NT), "packed tiles: score kernels");
    constexpr int QPW = 8 / TQ;                     // PACKED: queries of a wavefront
    const int pq0 = (group * 4 + wave) * QPW;
    F bq[NT];
    bool query_wild = false;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
        const int g = tile0 + tt;
        int q, trow;
        if (PACKED) {
            const int unit = 2 * tt + (col >> 3);
            const int lq = unit / A.hq;
            const int t = (unit - lq * A.hq) * 8 + (col & 7);
            const bool ok = lq < QPW && pq0 + lq < A.nq && t < A.T;
            q = ok ? pq0 + lq : 0;
            trow = ok ? t : 0;
        } else if (REVEAL) {
            const int x = g * 16 + col;
            q = x >> lgG;
            const int sl = x & (A.G - 1);
            q = q < A.nq ? q : 0;
            trow = A.pi[(size_t)q * A.T + A.lo + (sl < A.nb ? sl : 0)];
        } else {
            q = g / TQ;
            const int t = (g % TQ) * 16 + col;
            q = q < A.nq ? q : 0;
            trow = t < A.T ? t : 0;
        }
        query_wild |= bq[tt].load((const char*)A.Q + ((size_t)q * A.T + trow) * ROWB, kg);
    }
    query_wild = __ballot(query_wild) != 0ull;

    // ---- stage loader: 64 rows x ROWB bytes, copied global -> LDS without passing through
    // registers (global_load_lds_dwordx4: every lane names its 16 global bytes, the wavefront's
    // 64 pieces land in 1 KB of consecutive LDS).  One instruction fills 64/NCH ring rows; the
    // lane at physical piece position p of LDS row r fetches the logical piece p ^ (r & (NCH-1)).
    const char* src = (const char*)A.docs + (size_t)tok_begin * ROWB;
    constexpr int ROWS_PER_LOAD = 64 / NCH;
    constexpr int LOAD_WAVES = WAVES == 2 ? 2 : 4;                    // not of fp32
    constexpr int LOADS_PER_WAVE = STAGE_ROWS / ROWS_PER_LOAD / LOAD_WAVES;
    // A lane's place inside a load does not depend on the stage or on the load's number (both
    // move the row by multiples of the swizzle period): row wave*ROWS_PER_LOAD + lane/NCH of the
    // load group, piece (lane % NCH) ^ key(row).  A complete stage therefore needs no per-lane
    // address arithmetic at all: uniform base + this constant offset.
    const int lrow0 = wave * ROWS_PER_LOAD + lane / NCH;
    // the piece that belongs at a lane's place; the padding's places repeat others
    auto piece_of = [&](int row) {
        const int c = (lane & (NCH - 1)) ^ ((row >> KEY_SHIFT) & KEY_MASK);
        return c < ROWB / 16 ? c : c - (NCH - ROWB / 16);
    };
    static_assert(F32 || LOAD_WAVES * ROWS_PER_LOAD % ((KEY_MASK + 1) << KEY_SHIFT) == 0, "the swizzle's period");
    const unsigned fetch_off = (unsigned)(lrow0 * ROWB + piece_of(lrow0) * 16);
    auto stage_fetch = [&](int s) {
        if ((s + 1) * STAGE_ROWS <= ntok) {
#pragma unroll
            for (int i = 0; i < LOADS_PER_WAVE; ++i) {
                const int r0 = s * STAGE_ROWS + i * LOAD_WAVES * ROWS_PER_LOAD;      // uniform
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)(src + (size_t)r0 * ROWB + fetch_off),
                    (__attribute__((address_space(3))) void*)(ring + ((r0 + wave * ROWS_PER_LOAD) & (RING_ROWS - 1)) * PITCH),
                    16, 0, LOAD_POLICY);
            }
            return;
        }
        // the chunk's last, incomplete stage: rows past the end are clamped (they are never read)
#pragma unroll
        for (int i = 0; i < LOADS_PER_WAVE; ++i) {
            const int rbase = s * STAGE_ROWS + (i * LOAD_WAVES + wave) * ROWS_PER_LOAD;   // wave-uniform
            if (rbase < ntok) {
                const int lrow = rbase + lane / NCH;                  // the LDS row this lane fills
                const int grow = lrow < ntok ? lrow : ntok - 1;
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)(src + (size_t)grow * ROWB + piece_of(lrow) * 16),
                    (__attribute__((address_space(3))) void*)(ring + (rbase & (RING_ROWS - 1)) * PITCH),
                    16, 0, LOAD_POLICY);
            }
        }
    };

    // ---- document walk state (identical in all four wavefronts)
    int ibase = i0;
    auto fetch_offs = [&](int base) -> int {
        int j = base + lane;
        j = j > i1 ? i1 : j;
        int64_t o = A.off[j] - tok_begin;
        o = o < 0 ? 0 : (o > ntok ? ntok : o);
        return (int)o;
    };
    int offv = fetch_offs(ibase);
    auto rel_off = [&](int i) -> int {
        if (i - ibase >= 64) {
            ibase = i;
            offv = fetch_offs(ibase);
        }
        return __builtin_amdgcn_readlane(offv, i - ibase);
    };

    V h[NT];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) h[tt] = lowest_val<V>();

    // int8 codes: decode scale of the query behind each of this lane's packed results
    float cscale[Pack<NT>::NW];
    if constexpr (CODES && PACKED) {                // row r of pass j: query 4j + r
        const float ds = A.dscale[0];
#pragma unroll
        for (int j = 0; j < (QPW + 3) / 4; ++j) {
            const int q = pq0 + 4 * j + (lane >> 4);
            cscale[j] = A.qscale[q < A.nq ? q : 0] * ds;
        }
    } else if constexpr (CODES) {
        const float ds = A.dscale[0];
#pragma unroll
        for (int j = 0; j < Pack<NT>::NW; ++j) {
            const int g = tile0 + Pack<NT>::tile_of_row(j, lane >> 4);
            int q = REVEAL ? (g * 16 + col) >> lgG : g / TQ;
            q = q < A.nq ? q : 0;
            cscale[j] = A.qscale[q] * ds;
        }
    }

    // reveal: which of this lane's result registers belong to a query that takes the batch
    unsigned qmask = ~0u;
    if constexpr (REVEAL) {
        if (A.ctl) {
            using P = Pack<NT>;
            qmask = 0u;
#pragma unroll
            for (int j = 0; j < P::NW; ++j) {
                const int x = (tile0 + P::tile_of_row(j, lane >> 4)) * 16 + col;
                const int q = x >> lgG;
                if (q < A.nq) {
                    const QueryCtl c = A.ctl[q];
                    if (c.active && c.mode == 0) qmask |= 1u << j;
                }
            }
        }
    }

    // per-document epilogue: cross-lane maxima, then the row sum (score) or the batch
    // statistics (reveal), written by the lanes that own a query
    __shared__ int relay[PACKED ? 4 * NT * 16 : 1];
    auto finalize_packed = [&](int doc) {
        using P = Pack<NT>;
        V wi[P::NW];
        P::colmax(h, wi);
        int* mine_lds = relay + wave * (NT * 16);
        const int row = lane >> 4;
#pragma unroll
        for (int j = 0; j < P::NW; ++j) mine_lds[P::tile_of_row(j, row) * 16 + col] = __builtin_bit_cast(int, wi[j]);
        __builtin_amdgcn_wave_barrier();            // a wavefront's LDS accesses are performed in order
#pragma unroll
        for (int j = 0; j < (QPW + 3) / 4; ++j) {
            const int lq = 4 * j + row;             // a row of 16 lanes per query
            const int q = pq0 + lq;
            float v[TQ];
#pragma unroll
            for (int k = 0; k < TQ; ++k) {
                const int t = 16 * k + col;
                const bool ok = lq < QPW && t < A.T;
                const int x = mine_lds[ok ? lq * A.hq * 8 + t : 0];
                float f;
                if constexpr (CODES) f = (float)x * cscale[j];
                else f = __builtin_bit_cast(float, x);
                v[k] = ok ? f : 0.f;
            }
            float s = v[0];
            if constexpr (TQ == 2) s = v[0] + v[1];
            if constexpr (TQ >= 4) s = (v[0] + v[1]) + (v[2] + v[3]);
            if constexpr (TQ == 8) s = s + ((v[4] + v[5]) + (v[6] + v[7]));
            s = rowsum16(s);
            if (lq < QPW && q < A.nq) {
                if (col == 0) A.out[(size_t)q * A.N + doc] = s;
                if (A.cells) {
#pragma unroll
                    for (int k = 0; k < TQ; ++k)
                        if (16 * k + col < A.T) A.cells[((size_t)q * A.N + doc) * A.T + 16 * k + col] = v[k];
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) h[tt] = lowest_val<V>();
    };
    auto finalize = [&](int doc) {
        using P = Pack<NT>;
        if constexpr (PACKED) {
            finalize_packed(doc);
            return;
        } else {
        if (!mine(doc)) {                       // another wavefront's document: nothing to write
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) h[tt] = lowest_val<V>();
            return;
        }
        // cross-lane column maxima, decoded to float cells
        float w[P::NW];
        if constexpr (CODES) {
            V wi[P::NW];
            P::colmax(h, wi);
#pragma unroll
            for (int j = 0; j < P::NW; ++j) w[j] = (float)wi[j] * cscale[j];
        } else {
            P::colmax(h, w);
        }
        if constexpr (REVEAL) {
            const int row = lane >> 4;
#pragma unroll
            for (int j = 0; j < P::NW; ++j) {
                const int x = (tile0 + P::tile_of_row(j, row)) * 16 + col;
                const int q = x >> lgG, sl = x & (A.G - 1);
                float sb, m2b;
                batch_stats(w[j], sl, A.nb, A.G, sb, m2b);
                if (sl == 0 && q < A.nq && P::row_is_primary(row) && ((qmask >> j) & 1u))
                    A.stat[(size_t)q * A.N + doc] = make_float2(sb, m2b);
            }
        } else {
            using SC = Score<NT, TQ>;
            float sc[SC::NS];
            SC::finish(w, A.T, col, sc);
#pragma unroll
            for (int j = 0; j < SC::NS; ++j) {
                const int lq = SC::writer(j, lane);
                const int q = tile0 / TQ + lq;
                if (lq >= 0 && q < A.nq) A.out[(size_t)q * A.N + doc] = sc[j];
            }
            if (A.cells) {
                const int row = lane >> 4;
#pragma unroll
                for (int j = 0; j < SC::NW; ++j) {
                    const int g = tile0 + Pack<NT>::tile_of_row(j, row);
                    const int q = g / TQ, t = (g % TQ) * 16 + col;
                    if (Pack<NT>::row_is_primary(row) && q < A.nq && t < A.T)
                        A.cells[((size_t)q * A.N + doc) * A.T + t] = w[j];
                }
            }
        }
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) h[tt] = lowest_val<V>();
        }
    };

    // ---- stage bookkeeping.  The reader walks the chunk stage by stage; when it enters stage st
    // the stages up to st+1 are visible to every wavefront (the first block of st+1 is read as
    // the "next block" while the last block of st is multiplied) and the following stage is in
    // flight.  All four wavefronts walk the same blocks, so they reach stage_enter at
    // the same points and its barrier matches up.
    // Slot safety: a stage is requested into the slot of a stage at least two behind the
    // reader, which no wavefront reads any more once all have passed the barrier.
    const int nst = (ntok + STAGE_ROWS - 1) / STAGE_ROWS;
    const int nfull = ntok / STAGE_ROWS;            // stages with all their rows
    // wait until this wavefront's copies have landed (keeping a second stage in flight across
    // the barrier was measured and gained nothing)
    auto wait_copies = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); /* vmcnt(0) */ };
    // Workgroup barrier without a memory fence: the copies a wavefront is responsible for have
    // been awaited explicitly just before and every ring read of the slot that is about to be
    // overwritten has been consumed by its MFMAs.  The empty asm statements keep the compiler from moving ring accesses across.
    auto ring_barrier = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    if constexpr (!F32) {
        stage_fetch(0);
        if (nst > 1) stage_fetch(1);
        wait_copies();
        ring_barrier();
        if (nst > 2) stage_fetch(2);
    }
    // the reader enters stage st >= 1: publish stage st+1, request the next one
    auto stage_enter = [&](int st) {
        if (st + 1 >= nst) return;                  // everything is visible already
        wait_copies();
        ring_barrier();
        if (st + 2 < nst) stage_fetch(st + 2);
    };

    // ---- block stream.  The chunk's tokens are one stream cut into aligned blocks of 16 rows,
    // whatever the document boundaries: no row is multiplied twice.  A block that lies inside
    // one document (most do) folds into the running maxima as it is; a block in which a
    // document ends is folded in two parts, rows before the boundary into the ending document
    // and the rows after it into fresh maxima for the next one (block_mma_split); further
    // boundaries in the same block repeat the block's MFMAs for the next part.  The rows past
    // the chunk's end in its last block repeat the last token.
    // a lane's operand pieces inside an aligned block: row `col` of the block, piece
    // (ks*4 + kg) ^ key(row); the key does not depend on the block (blocks start at multiples
    // of 16 rows)
    unsigned blk_off[F::KS];
#pragma unroll
    for (int ks = 0; ks < F::KS; ++ks)
        blk_off[ks] = (unsigned)(col * PITCH + (((ks * 4 + kg) ^ ((col >> KEY_SHIFT) & KEY_MASK)) * 16));
    // a complete block (bs + 16 <= ntok) of a visible stage
    auto load_aligned = [&](auto& a, int bs) {
        using piece_t = __remove_reference_t(decltype(a.v[0]));
        const char* rp = ring + (bs & (RING_ROWS - 1)) * PITCH;      // uniform
#pragma unroll
        for (int ks = 0; ks < F::KS; ++ks) a.v[ks] = *(const piece_t*)(rp + blk_off[ks]);
    };
    // any block of a visible stage; the chunk's last block repeats the last token
    auto load_block = [&](auto& a, int bs) {
        if (bs + 16 <= ntok) {
            load_aligned(a, bs);
            return;
        }
        using piece_t = __remove_reference_t(decltype(a.v[0]));
        int row = bs + col;
        row = row < ntok ? row : ntok - 1;
        const char* rp = ring + (row & (RING_ROWS - 1)) * PITCH;
        const int sw = (row >> KEY_SHIFT) & KEY_MASK;
#pragma unroll
        for (int ks = 0; ks < F::KS; ++ks) a.v[ks] = *(const piece_t*)(rp + (((ks * 4 + kg) ^ sw) * 16));
    };
    int doc = i0;                   // document whose maxima are being accumulated
    int dend = rel_off(i0 + 1);     // its end, relative to the chunk
    const int rowbase = 4 * kg;
    auto process = [&](const F& a, int bs, bool wild = false) {
        int b = dend - bs;
        if (b > 16 || doc >= i1) {              // the block lies inside the current document
            if (mine(doc)) block_mma<NT>(a, bq, h, wild);
            return;
        }
        int lo = 0;
        if (b == 16) {                          // it ends exactly with the block: no split needed
            block_mma<NT>(a, bq, h, wild);
            finalize(doc);
            ++doc;
            if (doc >= i1) return;
            dend = rel_off(doc + 1);
            b = dend - bs;
            if (b > 16) return;                 // the usual case: the next document has tokens
            lo = 16;
        }
        for (;;) {
            V hB[NT];
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) hB[tt] = lowest_val<V>();
            const int bb = b < lo ? lo : b;     // offsets that run backwards: an empty part
            // the usual case - one document end in the block - takes the fold specialised by the
            // row of the end (six and eight tiles only: it is 15 copies of the block's code)
            if (NT >= PACKED_NT && lo == 0 && bb >= 1 && bb <= 15) block_mma_split_rows<NT>(a, bq, h, hB, bb);
            else block_mma_split<NT>(a, bq, h, hB, lo, bb, rowbase, wild);
            finalize(doc);
            ++doc;
            if (doc >= i1) return;
            lo = bb;
            dend = rel_off(doc + 1);
            b = dend - bs;
            if (b > 16) {                       // the rest of the block starts the next document
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) h[tt] = hB[tt];
                return;
            }
        }
    };

    // ---- fp32: a stage's rows pass through registers, where they are cut into their three pieces (split_first),
    // once for all wavefronts (50 vector instructions a wavefront and stage at d = 128 with eight wavefronts, twice as many
    // with four; each for itself would take 400, as long as the matrix work of two tiles).  A thread takes
    // the 16 + 16 bytes that a lane of a wavefront holds of one k-step (Frag): one 16-byte piece in each plane.
    // A wavefront writes stage s + 1 when it has finished stage s itself, over stage s - 1, which all finished
    // before the barrier of stage s.  (Three slots, the first block of a stage read before its barrier: eight
    // wavefronts 0 to 3 % faster, four 2 to 6 % slower.)
    if constexpr (F32) {
        constexpr int PIECES = D / 8;               // of a row
        constexpr int THREADS = 64 * WAVES;
        constexpr int PER = (STAGE_ROWS * PIECES + THREADS - 1) / THREADS;
        constexpr int PLANE = RING_ROWS * PITCH, SLOT = STAGE_ROWS * PITCH;
        __shared__ int wild_stage[2];               // by slot: the stage (and one) if it holds a wild value (Frag)
        if (threadIdx.x < 2) wild_stage[threadIdx.x] = 0;
        __syncthreads();
        f32x4_t raw[PER][2] = {};
        int prow[PER];
        unsigned src_off[PER], dst_off[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int x = i * THREADS + (int)threadIdx.x;
            const int c = x % PIECES;
            prow[i] = x / PIECES;
            src_off[i] = (unsigned)((c >> 2) * 128 + (c & 3) * 16);
            dst_off[i] = (unsigned)(prow[i] * PITCH + (c ^ ((prow[i] >> KEY_SHIFT) & KEY_MASK)) * 16);
        }
        auto has = [&](int i) { return PER * THREADS == STAGE_ROWS * PIECES || prow[i] < STAGE_ROWS; };   // whole wavefronts
        // rows past the chunk's end repeat the last token
        auto fetch = [&](int s) {
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (has(i)) {
                    int row = s * STAGE_ROWS + prow[i];
                    row = row < ntok ? row : ntok - 1;
                    const char* p = src + (size_t)row * ROWB + src_off[i];
                    raw[i][0] = *(const f32x4_t*)p;
                    raw[i][1] = *(const f32x4_t*)(p + 64);
                }
        };
        auto publish = [&](int s) {
            char* at = ring + (s & 1) * SLOT;
            bf16x8_t hi[PER], mid, lo;
            split_first<PER>(raw, hi, [&]() { wild_stage[s & 1] = s + 1; });
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (has(i)) {
                    split_rest(raw[i], hi[i], mid, lo);
                    *(bf16x8_t*)(at + dst_off[i]) = hi[i];
                    *(bf16x8_t*)(at + PLANE + dst_off[i]) = mid;
                    *(bf16x8_t*)(at + 2 * PLANE + dst_off[i]) = lo;
                }
        };
        auto load_half = [&](F& a, int s, int half) {
            const char* rp = ring + (s & 1) * SLOT + half * (16 * PITCH);
#pragma unroll
            for (int p = PLANES - 1; p >= 0; --p)
#pragma unroll
                for (int ks = 0; ks < F::KS; ++ks) a.v[p][ks] = *(const bf16x8_t*)(rp + p * PLANE + blk_off[ks]);
        };
        fetch(0);
        for (int s = 0; s < nst; ++s) {
            publish(s);
            if (s + 1 < nst) fetch(s + 1);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0): this wavefront's pieces are written
            ring_barrier();
            const int bs = s * STAGE_ROWS;
            const int flag = wild_stage[s & 1];     // (read first: its wait is not one for the operands)
            F a0, a1;
            load_half(a0, s, 0);
            load_half(a1, s, 1);
            const bool wild = query_wild | (__builtin_amdgcn_readfirstlane(flag) == s + 1);
            process(a0, bs, wild);
            if (bs + 16 < ntok) process(a1, bs + 16, wild);
        }
        while (doc < i1) finalize(doc++);           // documents without tokens at the chunk's end
        return;
    } else {

    // ---- consumer: the MFMAs of block k overlap the operand reads of block k+1.  a0 always
    // holds the block at bs; the stage that begins at bs (if one does) is entered just before
    // block bs is multiplied.  Runs of blocks that lie inside one document go through a loop
    // that holds nothing but the operand reads and the MFMAs of two blocks (and, every fourth
    // block, the stage entry); it covers the rows below tight_end, where every block has a
    // complete successor and every stage entered requests a complete stage.  A block in which a
    // document ends, and the chunk's last stages, take the general path.  (The loop without it for up to
    // four tiles a wavefront, us: 64 queries x 20,000 pages, Col-Bandit, 3,015 with the general path and 2,805,
    // 64 x 50,000 495 and 482, 8 x 200,000 exhaustive 1,380 and 1,285, 3 x 200,000 in d = 32 408 and 304; where
    // wavefronts split the documents 1 x 500,000 1,993 and 1,926, 1 x 200,000 of 100 tokens 1,692 and 1,412.)
    const int tight_end = (nfull - 2) * STAGE_ROWS;
    auto stage_enter_full = [&](int bs) {        // bs < tight_end is a stage boundary
        wait_copies();
        ring_barrier();
#pragma unroll
        for (int i = 0; i < LOADS_PER_WAVE; ++i) {
            const int r0 = bs + 2 * STAGE_ROWS + i * LOAD_WAVES * ROWS_PER_LOAD;      // uniform
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void*)(src + (size_t)r0 * ROWB + fetch_off),
                (__attribute__((address_space(3))) void*)(ring + ((r0 + wave * ROWS_PER_LOAD) & (RING_ROWS - 1)) * PITCH),
                16, 0, LOAD_POLICY);
        }
    };
    auto at_boundary = [&](int bs) { return (bs & (STAGE_ROWS - 1)) == 0 && bs > 0; };
    F a0, a1;
    int bs = 0;
    load_block(a0, 0);
    while (bs < ntok) {
        if (bs < tight_end) {
            // blocks from bs on that end before the current document does
            int run = doc < i1 ? (dend - bs - 1) >> 4 : RING_ROWS;
            const int left = (tight_end - bs) >> 4;
            run = run < 0 ? 0 : (run > left ? left : run);
            if (SPLIT_DOCS != 0 && run >= 1 && !mine(doc)) {    // another wavefront's: on to the run's end
                for (; run >= 1; --run) {
                    if (at_boundary(bs)) stage_enter_full(bs);
                    bs += 16;
                }
                load_aligned(a0, bs);
            }
            if (run >= 1 && (bs & 16)) {        // to an even block: pairs never straddle a stage
                load_aligned(a1, bs + 16);
                __builtin_amdgcn_sched_barrier(0);
                block_mma<NT>(a0, bq, h, false);
                a0 = a1;
                bs += 16;
                --run;
            }
#pragma unroll 1
            for (; run >= 2; run -= 2) {
                if (at_boundary(bs)) stage_enter_full(bs);
                load_aligned(a1, bs + 16);
                block_mma<NT>(a0, bq, h, false);
                load_aligned(a0, bs + 32);
                block_mma<NT>(a1, bq, h, false);
                bs += 32;
            }
            if (run == 1) {
                if (at_boundary(bs)) stage_enter_full(bs);
                load_aligned(a1, bs + 16);
                __builtin_amdgcn_sched_barrier(0);
                block_mma<NT>(a0, bq, h, false);
                a0 = a1;
                bs += 16;
            }
        }
        if (at_boundary(bs)) stage_enter(bs / STAGE_ROWS);
        if (bs + 16 < ntok) load_block(a1, bs + 16);
        __builtin_amdgcn_sched_barrier(0);      // keep the reads of the next block up here
        process(a0, bs);
        a0 = a1;
        bs += 16;
    }
    while (doc < i1) finalize(doc++);           // documents without tokens at the chunk's end
    }
}

// ---- first document of every token chunk
__global__ void k_chunk_docs(const int64_t* off, int64_t N, int C, int n_chunks, int32_t* chunk_doc) {
    chunk_docs((int64_t)blockIdx.x * blockDim.x + threadIdx.x, off, N, C, n_chunks, chunk_doc);
}

int dense_chunks(const Problem& P, const Work& W) {
    return (int)((P.total + W.chunk_tokens - 1) / W.chunk_tokens);
}

bool dense_supported(const Problem& P, const Coarse* co) {
    // int8 codes: the instruction contracts 64 elements at a time
    return (co ? P.d == 64 || P.d == 128 : P.d == 32 || P.d == 64 || P.d == 96 || P.d == 128) &&
           P.total / 4096 < 0x7fffff00;
}

hipError_t launch_dense_prepare(const Problem& P, const Work& W, int* n_chunks, hipStream_t st) {
    const int C = W.chunk_tokens;
    const int nc = dense_chunks(P, W);
    *n_chunks = nc;
    const int64_t n = P.N + 1;
    k_chunk_docs<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(P.off, P.N, C, nc, W.chunk_doc);
    return hipGetLastError();
}

static void fill_dense(DenseArgs& A, const Problem& P, const Work& W, int n_chunks) {
    A.Q = P.Q;
    A.docs = P.docs;
    A.off = P.off;
    A.chunk_doc = W.chunk_doc;
    A.N = P.N;
    A.total = P.total;
    A.nq = P.nq;
    A.T = P.T;
    A.n_chunks = n_chunks;
    A.pi = W.pi;
    A.stat = W.stat;
}

template <typename Tag, int D, int TILES, int TQ, bool REVEAL, int SPLIT = 0, bool PACKED = false>
static hipError_t dense_go(DenseArgs& A, int groups, hipStream_t st) {
    A.n_groups = groups;
    const int chunks8 = (A.n_chunks + 7) / 8 * 8;
    const long long blocks = (long long)chunks8 * A.n_groups;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    k_dense<Tag, D, TILES, TQ, REVEAL, SPLIT, PACKED><<<(unsigned)blocks, 64 * dense_waves<Tag, D, TILES, TQ, SPLIT>(), 0, st>>>(A);
    return hipGetLastError();
}

bool in_pairs(const Problem& P, int64_t tiles, bool codes) {
    return (codes || P.dt == DT_BF16) && P.d * (codes ? 1 : 2) == 128 && tiles > 8 && tiles <= 16 && pair_pays(P.total, P.N);
}

ScoreShape score_shape(const Problem& P, bool codes) {
    const bool f32 = P.dt == DT_F32 && !codes;
    const int tq = (P.T + 15) / 16;
    ScoreShape s{};
    s.tq = tq <= 1 ? 1 : tq <= 2 ? 2 : tq <= 4 ? 4 : 8;
    s.tiles = (int64_t)P.nq * s.tq;
    // one or two queries (twice as many of at most 16 tokens): the tiles fit one or two
    // wavefronts, and four or two wavefronts split the documents
    const int few = s.tq <= 2 ? 2 : s.tq;
    if (s.tiles <= 2 * few) {
        s.nt = few;
        s.split = s.tiles <= few ? 4 : 2;
        s.groups = 1;
        return s;
    }
    if (s.tq <= 2 && s.tiles <= 8) s.nt = 2;
    // fp32 is bound by the matrix pipes: groups half as large where that leaves clearly fewer tiles empty (10
    // queries of two tiles, 24 instead of 32 multiplied: 20,000 documents of d = 128 1,303 -> 998 us).  In d = 96
    // and 128 large groups, of eight wavefronts, gain only where all of them are whole (16 queries x 20,000
    // documents: d = 128 1,288 us with half as large groups and 1,302, 32 of 16 tokens at d = 96 1,108 and
    // 1,030) and are fewer to balance (5 queries x 5,000 documents of d = 128 209 and 260)
    else if (f32 && s.tq <= 2 && (P.d >= 96 ? s.tiles % 16 != 0 : (s.tiles + 7) / 8 * 8 * 9 < (s.tiles + 15) / 16 * 16 * 8)) s.nt = 2;
    else if (f32 || (s.tq <= 4 && s.tiles <= 16)) s.nt = 4;
    else s.nt = 8;
    s.groups = (int)((s.tiles + 4 * s.nt - 1) / (4 * s.nt));
    return s;
}

template <typename Tag, int D, int TQ>
static hipError_t dense_score_nt(DenseArgs& A, const ScoreShape& s, hipStream_t st) {
    constexpr int FEW = TQ <= 2 ? 2 : TQ;           // tiles of a wavefront that splits documents
    if constexpr (!Tag::wide) {
        if (always_gathers(s, D)) return hipErrorInvalidValue;
    }
    if constexpr (Tag::wide || TQ == 1) {
        if (s.split == 4) return dense_go<Tag, D, FEW, TQ, false, 4>(A, 1, st);
    }
    if constexpr (Tag::wide || TQ == 1 || (TQ == 2 && D != 96)) {
        if (s.split == 2) return dense_go<Tag, D, FEW, TQ, false, 2>(A, 1, st);
    }
    if constexpr (TQ <= 2) {
        if (s.nt == 2) return dense_go<Tag, D, 2, TQ, false>(A, s.groups, st);
    }
    if constexpr (TQ <= 4) {
        if constexpr (can_pair<Tag, D>()) {
            if (s.nt == 4 && pair_pays(A.total, A.N)) return dense_go<Tag, D, 4, TQ, false, PAIR>(A, s.groups, st);
        }
        if (s.nt == 4) return dense_go<Tag, D, 4, TQ, false>(A, s.groups, st);
    }
    if constexpr (Tag::wide) {
        A.hq = (A.T + 7) / 8;                       // a wavefront's queries are those of eight whole tiles
        if (A.hq * (8 / TQ) <= 2 * PACKED_NT) return dense_go<Tag, D, PACKED_NT, TQ, false, 0, true>(A, s.groups, st);
    }
    if constexpr (Tag::wide) return dense_go<Tag, D, 8, TQ, false>(A, s.groups, st);
    else return hipErrorInvalidValue;
}

template <typename Tag, int D>
static hipError_t dense_score_d(DenseArgs& A, const ScoreShape& s, hipStream_t st) {
    if (s.tq == 1) return dense_score_nt<Tag, D, 1>(A, s, st);
    if (s.tq == 2) return dense_score_nt<Tag, D, 2>(A, s, st);
    if (s.tq == 4) return dense_score_nt<Tag, D, 4>(A, s, st);
    if constexpr (Tag::wide) return dense_score_nt<Tag, D, 8>(A, s, st);
    else return hipErrorInvalidValue;
}

template <typename Tag> static hipError_t dense_score_any_d(DenseArgs& A, const ScoreShape& s, int d, hipStream_t st) {
    switch (d) {
        case 128: return dense_score_d<Tag, 128>(A, s, st);
        case 96: return dense_score_d<Tag, 96>(A, s, st);
        case 64: return dense_score_d<Tag, 64>(A, s, st);
        default: return dense_score_d<Tag, 32>(A, s, st);
    }
}

// int8 codes instead of the stored embeddings
static void use_codes(DenseArgs& A, const Coarse* co) {
    A.Q = co->Q8;
    A.docs = co->docs8;
    A.qscale = co->qscale;
    A.dscale = co->dscale;
}

hipError_t launch_dense_score(const Problem& P, const Work& W, int n_chunks, float* out,
                              float* cells, const Coarse* co, hipStream_t st) {
    DenseArgs A{};
    fill_dense(A, P, W, n_chunks);
    A.out = out;
    A.cells = cells;
    const ScoreShape s = score_shape(P, co != nullptr);
    if (co) {
        use_codes(A, co);
        return P.d == 128 ? dense_score_d<i8_tag, 128>(A, s, st) : dense_score_d<i8_tag, 64>(A, s, st);
    }
    return P.dt == DT_BF16 ? dense_score_any_d<bf16_tag>(A, s, P.d, st) : dense_score_any_d<f32_tag>(A, s, P.d, st);
}

template <typename Tag, int D>
static hipError_t dense_reveal_d(DenseArgs& A, hipStream_t st) {
    const int tiles = (A.nq * A.G + 15) / 16;
    if (tiles <= 4) return dense_go<Tag, D, 1, 1, true>(A, 1, st);
    if (tiles <= 8) return dense_go<Tag, D, 2, 1, true>(A, 1, st);
    if constexpr (can_pair<Tag, D>()) {
        if (tiles <= 16 && pair_pays(A.total, A.N)) return dense_go<Tag, D, 4, 1, true, PAIR>(A, 1, st);
    }
    if (!Tag::wide || tiles <= 16) return dense_go<Tag, D, 4, 1, true>(A, (tiles + 15) / 16, st);
    if constexpr (Tag::wide) return dense_go<Tag, D, 8, 1, true>(A, (tiles + 31) / 32, st);
    else return hipErrorInvalidValue;
}
template <typename Tag> static hipError_t dense_reveal_any_d(DenseArgs& A, int d, hipStream_t st) {
    switch (d) {
        case 128: return dense_reveal_d<Tag, 128>(A, st);
        case 96: return dense_reveal_d<Tag, 96>(A, st);
        case 64: return dense_reveal_d<Tag, 64>(A, st);
        default: return dense_reveal_d<Tag, 32>(A, st);
    }
}

static hipError_t dense_reveal_any(DenseArgs& A, const Problem& P, const Coarse* co, hipStream_t st) {
    if (co) {
        use_codes(A, co);
        return P.d == 128 ? dense_reveal_d<i8_tag, 128>(A, st) : dense_reveal_d<i8_tag, 64>(A, st);
    }
    return P.dt == DT_BF16 ? dense_reveal_any_d<bf16_tag>(A, P.d, st) : dense_reveal_any_d<f32_tag>(A, P.d, st);
}

hipError_t launch_dense_reveal(const Problem& P, const Work& W, int n_chunks,
                               const RevealRound& rr, int G, const Coarse* co, hipStream_t st) {
    DenseArgs A{};
    fill_dense(A, P, W, n_chunks);
    A.lo = rr.lo;
    A.nb = rr.nb;
    A.G = G;
    return dense_reveal_any(A, P, co, st);
}

hipError_t launch_dense_reveal_later(const Problem& P, const Work& W, int n_chunks,
                                     const RevealRound& rr, int G, const Coarse* co,
                                     hipStream_t st) {
    if (rr.dense.thr == NEVER_DENSE) return hipSuccess;
    DenseArgs A{};
    fill_dense(A, P, W, n_chunks);
    A.lo = rr.lo;
    A.nb = rr.nb;
    A.G = G;
    A.stat = W.stat2;
    A.pairs_r = W.pairs + rr.r;
    A.dense = rr.dense;
    A.ctl = W.ctl;
    return dense_reveal_any(A, P, co, st);
}

}  // namespace cb
