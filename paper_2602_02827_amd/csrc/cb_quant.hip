// int8 codes for the coarse elimination pass (paper, implementation appendix, paragraph on the
// quantized layout: magnitudes are clipped at the 999th permille and the clipped range is coded
// linearly in 8 bits).
//
// Reading of the paper fixed here: the percentile is the nearest-rank one -- the element of
// rank ceil(n * permille / 1000) of the ascending order of |x| over one segment (the whole
// corpus matrix, or one query's T x d matrix) -- found exactly by a radix select on the bit
// pattern of |x| (for non-negative floats the bit pattern orders like the value).  A code is
// rint(x * (127 / clip)) saturated to [-127, 127], all in single precision, and decodes to
// code * (clip / 127).
//
// Everything stays on the device: three histogram passes (11 + 11 + 10 bits; bf16 inputs need
// only the first two) each followed by a one-wavefront kernel that picks the bin holding the
// rank, then the quantising pass.  Segments are independent (grid.y).
//
// The first of those passes is bound by its LDS atomics (one per element, most on the bins of a few
// exponents), not by memory.  Long bf16 segments therefore count only the values above a
// lower bound taken from a sample: a few per mille of them at the percentiles in use, whose bf16
// values fit the bins one by one, so that one pass at the speed of memory finds the clip.  A bound
// that turns out too high or too low is noticed from the counts, and the two passes follow: such
// inputs pay for the counting pass too (8,000,000 rows of 128: 1.07 ms with a bound that holds, 1.95 with
// one that misses, 1.6 by the two passes alone).  From 2^29 values on the clip is mostly guessed from a part
// of them and confirmed by the coding pass, which reads the segment alone.
#include "cb_launch.h"
#include "cb_sample.h"

namespace cb {

constexpr int QH_BINS = 2048;
constexpr int QH_THREADS = 256;

struct SelState {                 // per segment, in the workspace
    unsigned long long rank;      // remaining 1-based ascending rank inside the current prefix
    uint32_t prefix, mask;        // key bits fixed so far
    uint32_t bound;               // k_quant_tail: values below it are not counted
    uint32_t done;                // 1: the clip is known; 2: the codes are written as well; GUESSED: prefix is
                                  // what a part of the segment says; NO_TAIL: the bound is of no use
};
constexpr uint32_t FOUND = 3, GUESSED = 4, NO_TAIL = 8;

template <bool BF16>
__device__ __forceinline__ uint32_t abs_key(const void* x, int64_t i) {
    if (BF16) return ((uint32_t)(((const uint16_t*)x)[i] & 0x7fffu)) << 16;
    return ((const uint32_t*)x)[i] & 0x7fffffffu;
}

__global__ void k_quant_init(SelState* st, unsigned long long* hist, int64_t nseg,
                             unsigned long long rank) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nseg) {
        SelState s;
        s.rank = rank;
        s.prefix = 0;
        s.mask = 0;
        s.bound = s.done = 0;
        st[i] = s;
    }
    if (i < nseg * QH_BINS) hist[i] = 0ull;
}

// VEC elements per 16-byte load
template <bool BF16> struct QVec { static constexpr int N = BF16 ? 8 : 4; };

// the VEC keys of 16 aligned bytes
template <bool BF16>
__device__ __forceinline__ void abs_keys16(const uint4& v, uint32_t (&k)[QVec<BF16>::N]) {
    if constexpr (BF16) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            k[2 * i] = (w[i] & 0x7fffu) << 16;
            k[2 * i + 1] = w[i] & 0x7fff0000u;
        }
    } else {
        k[0] = v.x & 0x7fffffffu;
        k[1] = v.y & 0x7fffffffu;
        k[2] = v.z & 0x7fffffffu;
        k[3] = v.w & 0x7fffffffu;
    }
}

// histogram of the `shift`-ed digit over the keys that match the segment's prefix.
// vec: the segment starts 16-byte aligned and holds a multiple of VEC elements.
template <bool BF16>
__global__ __launch_bounds__(QH_THREADS) void k_quant_hist(const void* x, int64_t seg_elems,
                                                           const SelState* st,
                                                           unsigned long long* hist, int shift,
                                                           int nbins, int vec) {
    __shared__ uint32_t lh[QH_BINS];
    constexpr int VEC = QVec<BF16>::N;
    const int64_t seg = blockIdx.y;
    for (int i = threadIdx.x; i < QH_BINS; i += QH_THREADS) lh[i] = 0;
    __syncthreads();
    const SelState s = st[seg];
    if (s.done & FOUND) return;
    const uint32_t prefix = s.prefix, mask = s.mask;
    const int64_t base = seg * seg_elems;
    // a block's share stays below 2^32 elements (the launch gives every block <= 2^32)
    if (vec) {
        const uint4* xv = (const uint4*)((const char*)x + base * (BF16 ? 2 : 4));
        const int64_t nv = seg_elems / VEC;
        for (int64_t i = (int64_t)blockIdx.x * QH_THREADS + threadIdx.x; i < nv;
             i += (int64_t)gridDim.x * QH_THREADS) {
            uint32_t k[VEC];
            abs_keys16<BF16>(xv[i], k);
#pragma unroll
            for (int u = 0; u < VEC; ++u)
                if ((k[u] & mask) == prefix) atomicAdd(&lh[(k[u] >> shift) & (nbins - 1)], 1u);
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * QH_THREADS + threadIdx.x; i < seg_elems;
             i += (int64_t)gridDim.x * QH_THREADS) {
            const uint32_t k = abs_key<BF16>(x, base + i);
            if ((k & mask) == prefix) atomicAdd(&lh[(k >> shift) & (nbins - 1)], 1u);
        }
    }
    __syncthreads();
    unsigned long long* gh = hist + seg * QH_BINS;
    for (int i = threadIdx.x; i < nbins; i += QH_THREADS)
        if (lh[i]) atomicAdd(&gh[i], (unsigned long long)lh[i]);
}

// One wavefront: ascending walk to the bin that holds the segment's rank; every lane gets the
// state with that digit fixed.
__device__ __forceinline__ SelState pick_bin(SelState s, const unsigned long long* gh, int shift, int nbins) {
    const int lane = threadIdx.x & 63;
    const int per = nbins / 64;
    unsigned long long local = 0;
    for (int j = 0; j < per; ++j) local += gh[lane * per + j];
    unsigned long long incl = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    unsigned long long run = incl - local;
    const bool mine = run < s.rank && s.rank <= incl;
    int bin = 0;
    if (mine) {
        for (int j = 0; j < per; ++j) {
            const unsigned long long c = gh[lane * per + j];
            if (run + c >= s.rank) {
                bin = lane * per + j;
                break;
            }
            run += c;
        }
    }
    const unsigned long long m = __ballot(mine);
    if (m == 0ull) return s;
    const int src = __ffsll((long long)m) - 1;
    s.prefix |= (uint32_t)__shfl(bin, src) << shift;
    s.mask |= (uint32_t)(nbins - 1) << shift;
    s.rank -= __shfl(run, src);
    return s;
}

// the same for the next pass; clears the bins
__global__ __launch_bounds__(64) void k_quant_pick(SelState* st, unsigned long long* hist,
                                                   int shift, int nbins) {
    const int64_t seg = blockIdx.x;
    unsigned long long* gh = hist + seg * QH_BINS;
    const SelState s = st[seg];
    if (s.done & FOUND) return;
    const SelState next = pick_bin(s, gh, shift, nbins);
    if (threadIdx.x == 0) st[seg] = next;
    __syncthreads();
    for (int i = threadIdx.x; i < QH_BINS; i += 64) gh[i] = 0ull;
}

// ---- long bf16 segments
constexpr int QT_SAMPLE_VECS = 16384;         // sampled 16-byte pieces: 131,072 values
constexpr int QT_BINS = 16384;                // their histogram: exponent and six mantissa bits
constexpr int64_t QT_MIN_ELEMS = 1ll << 26;   // below, the sample and three launches (60 us) cost as much as
                                              // the atomics they save (1 us per million values)

// From 2^29 values on a sixteenth of the segment is counted first.  bf16 values are so few that it names the clip
// itself, but where the rank lies close to an edge of the values that round to it (at 6.8 G independent
// values 0.46 % of the tail to either side, of 6 to 8; k_quant_guess).  Then one pass codes and counts, and
// the count confirms the guess: 6.8 G values 6.55 -> 3.95 ms (20.4 GB; the pass 3.6 ms).  No guess costs the
// sixteenth (6.75 ms), one that is wrong after all a coding pass (8.09), and one made where the bound was
// wrong too 13.9 ms in the place of 12.5.  (Below, the sixteenth's tail is too short to tell.)
constexpr int64_t QT_GUESS_ELEMS = 1ll << 29;

// Lower bound for k_quant_tail from pieces all over the segment (sample_piece): the largest histogram edge
// with a sixth (and 40) more sampled values above it than the wanted rank calls for.
// `above`: values of rank `rank` and higher.
__global__ __launch_bounds__(1024) void k_quant_sample(const void* x, int64_t seg_elems, SelState* st,
                                                       unsigned long long above) {
    __shared__ uint32_t lh[QT_BINS];
    __shared__ int part[1024];
    const int64_t seg = blockIdx.x;
    const int tid = threadIdx.x;
    const uint4* xv = (const uint4*)((const char*)x + seg * seg_elems * 2);
    const int64_t nv = seg_elems / 8;
    const int64_t step = nv / QT_SAMPLE_VECS;
    for (int i = tid; i < QT_BINS; i += 1024) lh[i] = 0;
    __syncthreads();
#pragma unroll 4
    for (int i = tid; i < QT_SAMPLE_VECS; i += 1024) {
        uint32_t k[8];
        abs_keys16<true>(xv[sample_piece((uint32_t)i, step)], k);
#pragma unroll
        for (int u = 0; u < 8; ++u) atomicAdd(&lh[k[u] >> 17], 1u);
    }
    __syncthreads();
    // bins from the highest down, 16 per thread
    constexpr int PER = QT_BINS / 1024;
    const int hi = QT_BINS - 1 - tid * PER;
    int local = 0;
    for (int j = 0; j < PER; ++j) local += (int)lh[hi - j];
    part[tid] = local;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int v = tid >= o ? part[tid - o] : 0;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
    const double share = (double)above / (double)seg_elems;
    const int want = (int)(share * (QT_SAMPLE_VECS * 8.0) * (7.0 / 6.0)) + 40;
    const int excl = part[tid] - local;
    if (excl < want && want <= part[tid]) {      // one thread, if the sample has that many values
        int run = excl, j = 0;
        for (; j < PER - 1; ++j) {
            run += (int)lh[hi - j];
            if (run >= want) break;
        }
        st[seg].bound = (uint32_t)(hi - j) << 17;
    }
}

// Counts those of 16 bytes' values that are at or above the bound in their bins: bf16 value relative to the
// bound, bin LAST takes the rest.  A few per mille of the values are.
template <int LAST>
__device__ __forceinline__ void count_tail(const u32x4_t& w, uint32_t lo, uint32_t* lh) {
    unsigned hit = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        hit |= (w[u] & 0x7fffu) >= lo ? 1u << (2 * u) : 0u;
        hit |= ((w[u] >> 16) & 0x7fffu) >= lo ? 2u << (2 * u) : 0u;
    }
    while (hit) {
        const int b = __ffs((int)hit) - 1;
        hit &= hit - 1;
        const uint32_t p = b < 4 ? (b < 2 ? w[0] : w[1]) : (b < 6 ? w[2] : w[3]);
        const uint32_t k = ((b & 1) ? p >> 16 : p) & 0x7fffu;
        const uint32_t bin = k - lo < LAST ? k - lo : LAST;
        atomicAdd(&lh[bin], 1u);
    }
}
__device__ __forceinline__ void flush_tail(const uint32_t* lh, unsigned long long* gh) {
    __syncthreads();
    for (int j = threadIdx.x; j < QH_BINS; j += QH_THREADS)
        if (lh[j]) atomicAdd(&gh[j], (unsigned long long)lh[j]);
}

// Counts the values at or above the bound.  Bound by memory: 6.8 G values (13.6 GB) in 2.42 ms = 5.6 TB/s;
// the two histogram passes that it replaces took 3.49 and 2.38 ms.  groups > 0: of every 16 runs of 4 KB only
// one, at a mixed place (sample_piece), `groups` of them, as many in each workgroup; the two bins behind
// PART_LAST take the sum of the workgroups' counts and of their squares.
constexpr int QT_RUN = 256, QT_PART = 16;
constexpr int PART_LAST = QH_BINS - 3;
__global__ __launch_bounds__(QH_THREADS) void k_quant_tail(const void* x, int64_t seg_elems,
                                                           const SelState* st, unsigned long long* hist, int64_t groups) {
    __shared__ uint32_t lh[QH_BINS];
    __shared__ uint32_t counted;
    static_assert(QT_RUN == QH_THREADS, "a workgroup takes a run at a time");
    const int64_t seg = blockIdx.y;
    if (st[seg].done) return;
    const uint32_t lo = st[seg].bound >> 16;
    for (int i = threadIdx.x; i < QH_BINS; i += QH_THREADS) lh[i] = 0;
    if (threadIdx.x == 0) counted = 0;
    __syncthreads();
    const u32x4_t* xv = (const u32x4_t*)((const char*)x + seg * seg_elems * 2);
    const int64_t nv = seg_elems / 8;
    unsigned long long* gh = hist + seg * QH_BINS;
    if (groups > 0) {
        for (int64_t g = blockIdx.x; g < groups; g += gridDim.x)
            count_tail<PART_LAST>(xv[sample_piece((uint32_t)g, QT_PART) * QT_RUN + threadIdx.x], lo, lh);
        __syncthreads();
        uint32_t mine = 0;
        for (int j = threadIdx.x; j < QH_BINS; j += QH_THREADS) mine += lh[j];
        if (mine) atomicAdd(&counted, mine);
        __syncthreads();
        if (threadIdx.x == 0 && counted) {
            atomicAdd(&gh[PART_LAST + 1], (unsigned long long)counted);
            atomicAdd(&gh[PART_LAST + 2], (unsigned long long)counted * counted);
        }
    } else {
        const int64_t stride = (int64_t)gridDim.x * QH_THREADS;
        int64_t i = (int64_t)blockIdx.x * QH_THREADS + threadIdx.x;
        for (; i + 3 * stride < nv; i += 4 * stride) {
            const u32x4_t a = xv[i], b = xv[i + stride], c = xv[i + 2 * stride], d = xv[i + 3 * stride];
            count_tail<QH_BINS - 1>(a, lo, lh);
            count_tail<QH_BINS - 1>(b, lo, lh);
            count_tail<QH_BINS - 1>(c, lo, lh);
            count_tail<QH_BINS - 1>(d, lo, lh);
        }
        for (; i < nv; i += stride) count_tail<QH_BINS - 1>(xv[i], lo, lh);
    }
    flush_tail(lh, gh);
}

// What the counts of a wavefront's segment say of the value with `above` counted values at or above it: its
// bin and the values counted above that bin and from it on.  False where too few were counted or it lies
// among the values that share the last bin.
__device__ __forceinline__ bool tail_bin(const unsigned long long* gh, unsigned long long above, int& bin,
                                         unsigned long long& higher, unsigned long long& from) {
    const int lane = threadIdx.x & 63;
    constexpr int PER = QH_BINS / 64;
    const int hi = QH_BINS - 1 - lane * PER;
    unsigned long long local = 0;
    for (int j = 0; j < PER; ++j) local += gh[hi - j];
    unsigned long long incl = local;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    unsigned long long run = incl - local, next = run;
    const bool mine = run < above && above <= incl;
    int j = 0;
    if (mine)
        for (;; ++j) {
            next = run + gh[hi - j];
            if (next >= above || j == PER - 1) break;
            run = next;
        }
    const unsigned long long m = __ballot(mine);
    if (m == 0ull) return false;
    const int src = __ffsll((long long)m) - 1;
    bin = __shfl(hi - j, src);
    higher = __shfl(run, src);
    from = __shfl(next, src);
    return bin < QH_BINS - 1;
}
__device__ __forceinline__ void clear_bins(unsigned long long* gh) {
    __syncthreads();
    for (int i = threadIdx.x; i < QH_BINS; i += 64) gh[i] = 0ull;
}

// After the count of a part: its value of that rank, if the counts put the rank three deviations or more of independent
// values (the square root of the count) inside the values that round to it, and two of these.  These: how much
// more the workgroups' counts vary.  Neighbouring rows of a corpus are alike; tokens of documents with a
// topic vary 1.8 times as much in d = 128, 3 times in d = 64.  (A guess that is right 39 times of 40 saves 2.8 ms of 6.7
// and costs 4.1 when it is wrong.)
__global__ __launch_bounds__(64) void k_quant_guess(SelState* st, unsigned long long* hist, unsigned long long above,
                                                    int workgroups) {
    const int64_t seg = blockIdx.x;
    unsigned long long* gh = hist + seg * QH_BINS;
    const double sum = (double)gh[PART_LAST + 1], squares = (double)gh[PART_LAST + 2];
    __syncthreads();
    if (threadIdx.x < 2) gh[PART_LAST + 1 + threadIdx.x] = 0ull;
    __syncthreads();
    int bin;
    unsigned long long higher, from;
    const bool found = tail_bin(gh, above, bin, higher, from) && bin < PART_LAST;
    const double mean = sum / workgroups, variance = (squares - sum * mean) / (workgroups - 1);
    const double margin = fmax(3.0 * sqrt((double)above), 2.0 * sqrt((double)above * variance / fmax(mean, 1.0)));
    if (threadIdx.x == 0 && found && (double)(above - higher) >= margin && (double)(from - above) >= margin) {
        st[seg].prefix = ((st[seg].bound >> 16) + (uint32_t)bin) << 16;
        st[seg].done = GUESSED;
    }
    clear_bins(gh);
}

// After the count of the whole segment: its value of that rank.  A guess that it confirms has its codes; where
// the count finds none (too few values from the bound on), another would not either.
__global__ __launch_bounds__(64) void k_quant_tail_pick(SelState* st, unsigned long long* hist,
                                                        unsigned long long above, uint32_t when) {
    const int64_t seg = blockIdx.x;
    unsigned long long* gh = hist + seg * QH_BINS;
    const SelState s = st[seg];
    if (s.done != when) return;
    int bin;
    unsigned long long higher, from;
    const bool found = tail_bin(gh, above, bin, higher, from);
    if (threadIdx.x == 0) {
        const uint32_t clip = found ? ((s.bound >> 16) + (uint32_t)bin) << 16 : 0u;
        st[seg].prefix = clip;
        st[seg].done = !found ? NO_TAIL : s.done == GUESSED && clip == s.prefix ? 2u : 1u;
    }
    clear_bins(gh);
}

__device__ __forceinline__ int code_of(float v, float inv) {
    float r = rintf(v * inv);
    r = r > 127.f ? 127.f : (r < -127.f ? -127.f : r);
    return (int)r;
}

// nbins > 0: the last digit's histogram has not been looked at yet, and every workgroup picks the bin
// for itself: a launch less where the workgroups are few.
// STREAM: a segment larger than the caches, whose values are not read again nor the codes by this
// call: neither should stay in L2 (6.8 G values: 3.80 -> 3.60 ms).
// COUNT: with the guessed clip, and counts the tail on the way.
template <bool BF16, bool STREAM, bool COUNT = false>
__global__ __launch_bounds__(QH_THREADS) void k_quant_codes(const void* x, int64_t seg_elems,
                                                            const SelState* st, unsigned long long* hist,
                                                            int nbins, int8_t* out, float* scales, int vec) {
    constexpr int VEC = QVec<BF16>::N;
    __shared__ uint32_t key;
    __shared__ uint32_t lh[COUNT ? QH_BINS : 1];
    const int64_t seg = blockIdx.y;
    const uint32_t done = st[seg].done;
    if (COUNT ? done != GUESSED : done == 2u) return;
    const uint32_t lo = COUNT ? st[seg].bound >> 16 : 0u;
    if constexpr (COUNT)
        for (int i = threadIdx.x; i < QH_BINS; i += QH_THREADS) lh[i] = 0;
    if (threadIdx.x < 64) {
        SelState s = st[seg];
        if (nbins > 0 && !(s.done & FOUND)) s = pick_bin(s, hist + seg * QH_BINS, BF16 ? 10 : 0, nbins);
        if (threadIdx.x == 0) key = s.prefix;
    }
    __syncthreads();
    const float clip = __uint_as_float(key);
    const float inv = clip > 0.f ? 127.0f / clip : 0.f;
    if (blockIdx.x == 0 && threadIdx.x == 0) scales[seg] = clip / 127.0f;
    const int64_t base = seg * seg_elems;
    if (vec) {
        const uint4* xv = (const uint4*)((const char*)x + base * (BF16 ? 2 : 4));
        const int64_t nv = seg_elems / VEC;
        for (int64_t i = (int64_t)blockIdx.x * QH_THREADS + threadIdx.x; i < nv;
             i += (int64_t)gridDim.x * QH_THREADS) {
            u32x4_t w;
            if constexpr (STREAM) w = __builtin_nontemporal_load((const u32x4_t*)xv + i);
            else w = ((const u32x4_t*)xv)[i];
            if constexpr (COUNT) count_tail<QH_BINS - 1>(w, lo, lh);
            uint32_t packed[VEC / 4];
#pragma unroll
            for (int j = 0; j < VEC / 4; ++j) packed[j] = 0;
#pragma unroll
            for (int u = 0; u < VEC; ++u) {
                float f;
                if constexpr (BF16) f = __uint_as_float((u & 1) ? (w[u >> 1] & 0xffff0000u) : (w[u >> 1] << 16));
                else f = __uint_as_float(w[u]);
                packed[u >> 2] |= ((uint32_t)code_of(f, inv) & 0xffu) << (8 * (u & 3));
            }
            if constexpr (BF16) {
                const unsigned long long two = (unsigned long long)packed[0] | (unsigned long long)packed[1] << 32;
                if constexpr (STREAM) __builtin_nontemporal_store(two, (unsigned long long*)(out + base) + i);
                else ((unsigned long long*)(out + base))[i] = two;
            } else {
                if constexpr (STREAM) __builtin_nontemporal_store(packed[0], (uint32_t*)(out + base) + i);
                else ((uint32_t*)(out + base))[i] = packed[0];
            }
        }
        if constexpr (COUNT) flush_tail(lh, hist + seg * QH_BINS);
        return;
    }
    for (int64_t i = (int64_t)blockIdx.x * QH_THREADS + threadIdx.x; i < seg_elems;
         i += (int64_t)gridDim.x * QH_THREADS) {
        float v;
        if (BF16) v = __uint_as_float((uint32_t)((const uint16_t*)x)[base + i] << 16);
        else v = ((const float*)x)[base + i];
        out[base + i] = (int8_t)code_of(v, inv);
    }
}

// Small segments (a query's T x d matrix): the whole job in one launch, one workgroup per
// segment.  Same selection (ascending rank over the radix digits of |x|) with the histogram in
// LDS; the segment is re-read from cache in every pass.
constexpr int QS_MAX_ELEMS = 65536;
template <bool BF16>
__global__ __launch_bounds__(QH_THREADS) void k_quant_small(const void* x, int seg_elems,
                                                            unsigned long long rank0, int8_t* out,
                                                            float* scales) {
    __shared__ uint32_t lh[QH_BINS];
    __shared__ uint32_t sel[2];           // chosen bin, remaining rank
    const int64_t base = (int64_t)blockIdx.x * seg_elems;
    uint32_t prefix = 0, mask = 0;
    uint32_t rank = (uint32_t)rank0;
    const int npass = BF16 ? 2 : 3;
#pragma unroll 1
    for (int p = 0; p < npass; ++p) {
        const int shift = p == 0 ? 21 : (p == 1 ? 10 : 0);
        const int nbins = p == 2 ? 1024 : 2048;
        for (int i = threadIdx.x; i < QH_BINS; i += QH_THREADS) lh[i] = 0;
        if (threadIdx.x == 0) {
            sel[0] = 0;
            sel[1] = 1;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < seg_elems; i += QH_THREADS) {
            const uint32_t k = abs_key<BF16>(x, base + i);
            if ((k & mask) == prefix) atomicAdd(&lh[(k >> shift) & (nbins - 1)], 1u);
        }
        __syncthreads();
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            const int per = nbins / 64;
            uint32_t local = 0;
            for (int j = 0; j < per; ++j) local += lh[lane * per + j];
            uint32_t incl = local;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_up(incl, o);
                if (lane >= o) incl += t;
            }
            const uint32_t excl = incl - local;
            if (excl < rank && rank <= incl) {
                uint32_t run = excl;
                for (int j = 0; j < per; ++j) {
                    const uint32_t c = lh[lane * per + j];
                    if (run + c >= rank) {
                        sel[0] = (uint32_t)(lane * per + j);
                        sel[1] = rank - run;
                        break;
                    }
                    run += c;
                }
            }
        }
        __syncthreads();
        prefix |= sel[0] << shift;
        mask |= (uint32_t)(nbins - 1) << shift;
        rank = sel[1];
        __syncthreads();
    }
    const float clip = __uint_as_float(prefix);
    const float inv = clip > 0.f ? 127.0f / clip : 0.f;
    if (threadIdx.x == 0) scales[blockIdx.x] = clip / 127.0f;
    for (int i = threadIdx.x; i < seg_elems; i += QH_THREADS) {
        float v;
        if (BF16) v = __uint_as_float((uint32_t)((const uint16_t*)x)[base + i] << 16);
        else v = ((const float*)x)[base + i];
        out[base + i] = (int8_t)code_of(v, inv);
    }
}

size_t quantize_scratch_bytes(int64_t n_segments) {
    return (size_t)n_segments * (sizeof(SelState) + sizeof(unsigned long long) * QH_BINS);
}

// x: [n_segments][seg_elems] of dt; codes: same shape; scales: [n_segments].
hipError_t launch_quantize_i8(const void* x, int dt, int64_t n_segments, int64_t seg_elems,
                              int permille, int8_t* codes, float* scales, void* scratch,
                              hipStream_t st) {
    const unsigned long long rank_all =
        ((unsigned long long)seg_elems * (unsigned long long)permille + 999ull) / 1000ull;
    if (seg_elems <= QS_MAX_ELEMS) {
        const unsigned long long r1 = rank_all < 1 ? 1 : rank_all;
        if (dt == DT_BF16)
            k_quant_small<true><<<(unsigned)n_segments, QH_THREADS, 0, st>>>(x, (int)seg_elems, r1, codes, scales);
        else
            k_quant_small<false><<<(unsigned)n_segments, QH_THREADS, 0, st>>>(x, (int)seg_elems, r1, codes, scales);
        return hipGetLastError();
    }
    SelState* state = (SelState*)scratch;
    unsigned long long* hist = (unsigned long long*)(state + n_segments);
    // ceil(seg_elems * permille / 1000), exact in 64-bit integers
    const unsigned long long rank =
        ((unsigned long long)seg_elems * (unsigned long long)permille + 999ull) / 1000ull;
    const int64_t init_n = n_segments * QH_BINS;
    k_quant_init<<<(unsigned)((init_n + 255) / 256), 256, 0, st>>>(state, hist, n_segments,
                                                                  rank < 1 ? 1 : rank);
    int64_t bx = (seg_elems + (int64_t)QH_THREADS * 64 - 1) / ((int64_t)QH_THREADS * 64);
    if (bx > 8192) bx = 8192;
    if (bx < 1) bx = 1;
    while (seg_elems / bx > (1ll << 24) * QH_THREADS) bx *= 2;   // per-block counts fit 32 bits
    const dim3 grid((unsigned)bx, (unsigned)n_segments);
    const bool bf = dt == DT_BF16;
    // 16-byte accesses need every segment (and the codes, 8 or 4 per store) aligned
    const int vec_n = bf ? 8 : 4;
    const int vec = (seg_elems % vec_n == 0 && ((uintptr_t)x & 15) == 0 && ((uintptr_t)codes & 7) == 0) ? 1 : 0;
    const int npass = bf ? 2 : 3;
    const unsigned long long above = (unsigned long long)seg_elems - (rank < 1 ? 1 : rank) + 1ull;
    if (bf && vec && seg_elems >= QT_MIN_ELEMS && above <= (unsigned long long)seg_elems / 64) {
        const unsigned nseg = (unsigned)n_segments;
        k_quant_sample<<<nseg, 1024, 0, st>>>(x, seg_elems, state, above);
        const dim3 tail((unsigned)(bx < 2048 ? bx : 2048), nseg);   // eight per CU
        const int64_t groups = seg_elems / 8 / (QT_RUN * QT_PART) / tail.x * tail.x;
        const int64_t counted = groups * QT_RUN * 8;
        const unsigned long long of_part = (unsigned long long)((double)above * ((double)counted / (double)seg_elems) + 0.5);
        // (fewer than nine: k_quant_guess's margin is more than there are)
        if (seg_elems >= QT_GUESS_ELEMS && of_part >= 9) {
            k_quant_tail<<<tail, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, groups);
            k_quant_guess<<<nseg, 64, 0, st>>>(state, hist, of_part, (int)tail.x);
            // 48 loads of 16 bytes a thread, or more for up to 32,768 workgroups (us: 6.8 G values 4,300 with 8,192,
            // 4,040 with 16,384, 3,940 with 32,768, 4,005 with 65,536; 1.3 G 980, 920, 965, 1,590)
            const int64_t blocks = seg_elems / (8 * QH_THREADS * 48);
            const dim3 both((unsigned)(blocks < 32768 ? blocks : 32768), nseg);
            k_quant_codes<true, true, true><<<both, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, 0, codes, scales, vec);
            k_quant_tail_pick<<<nseg, 64, 0, st>>>(state, hist, above, GUESSED);
        }
        k_quant_tail<<<tail, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, 0);
        k_quant_tail_pick<<<nseg, 64, 0, st>>>(state, hist, above, 0u);
    }
    // 16 KB of bins read by each workgroup of the coding pass against a launch: 4 M values 39.7 -> 38.3 us
    const bool pick_last = bx * n_segments <= 1024;
    for (int p = 0; p < npass; ++p) {
        const int shift = p == 0 ? 21 : (p == 1 ? 10 : 0);
        const int nbins = p == 2 ? 1024 : 2048;
        if (bf) k_quant_hist<true><<<grid, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, shift, nbins, vec);
        else k_quant_hist<false><<<grid, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, shift, nbins, vec);
        if (p < npass - 1 || !pick_last) k_quant_pick<<<(unsigned)n_segments, 64, 0, st>>>(state, hist, shift, nbins);
    }
    const int last_bins = pick_last ? (bf ? 2048 : 1024) : 0;
    const bool stream = seg_elems >= QT_MIN_ELEMS;
    if (bf && stream) k_quant_codes<true, true><<<grid, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, last_bins, codes, scales, vec);
    else if (bf) k_quant_codes<true, false><<<grid, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, last_bins, codes, scales, vec);
    else if (stream) k_quant_codes<false, true><<<grid, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, last_bins, codes, scales, vec);
    else k_quant_codes<false, false><<<grid, QH_THREADS, 0, st>>>(x, seg_elems, state, hist, last_bins, codes, scales, vec);
    return hipGetLastError();
}

}  // namespace cb
