// Final SDs inside potential SD regions (Section 3.3): exact seeds of k
// bases (k = 11) anchor both sides, anchors are chained in two tiers, the
// chains are aligned globally, and the alignments meeting the SD conditions
// are reported with CIGAR operations and Kimura two-parameter / Jukes-Cantor
// distances.  The readings of the steps the paper leaves open are those of
// the header of sdf_align_regions (include/sdf.h).
//
// Device pipeline, all regions of a call at once:
//   1. one workgroup per 16,384 to 65,536 query positions of a region puts the k-mers of
//      the target side T' (the target read reverse-complemented on strand 1)
//      in buckets in LDS, and every query k-mer finds its target occurrences
//      there; seeds occurring more than 32 times are skipped;
//   2. matches as keys (region, diagonal, query position), radix sorted;
//      maximal runs of consecutive positions on a diagonal are the anchors;
//   3. tier 1: one workgroup per region scores its anchors 64 at a time in
//      (x, y) order, testing the predecessors that end within the gap limit
//      or inside the anchor itself (a link then cuts the overlap from the
//      later anchor's start), a window of a second order, by end, and then
//      the links inside the batch; the anchors are then ordered by (region,
//      score descending, x, y), and every anchor finds the chain it is taken
//      out with; the chains become nodes, ordered by (region, x, y) and by
//      (region, end);
//   4. tier 2: the same scoring over the nodes (affine cost, gaps up to
//      10 kbp, blocks of candidates that cannot give a positive link
//      skipped), the same ordering and extraction of the final chains;
//   5. the stretches between consecutive anchors of every final chain are
//      aligned by one thread each (three-state affine recurrence over two
//      rolling rows, one byte of traceback per cell), the large ones by one
//      wave each;
//   6. the shares of the final chains (a stretch and the anchor after it) are
//      counted one per lane (matches, transitions, gaps, runs of equal
//      operations), summed up by chain, which applies the report rule, and
//      written to the CIGARs at the places a prefix sum gives them.
#include <vector>

#include "sdf_impl.h"
#include "search.h"

namespace sdf {

namespace {

constexpr uint32_t MAXOCC = 32;
constexpr uint32_t TIER2_GAP = 10000;
constexpr uint32_t T2_BLOCKS = 4096;  // tier-2 end-order blocks per region with LDS bounds
constexpr uint32_t T2_WAVES = 16;     // waves of a tier-2 workgroup
constexpr int32_t T2_NEVER = 1 << 29;  // the cost of no link: above any score
constexpr uint32_t T1_WAVES = 8;      // waves of a tier-1 workgroup
constexpr uint64_t DP_CELLS = 1ull << 20;
enum : uint32_t { OP_EQ = 7, OP_X = 8, OP_I = 1, OP_D = 2 };

struct ARegion {
    uint64_t q0, q1, t0, t1;  // global sides
    uint32_t o, qseq, tseq, _pad;
};

// Base p of the index as 0..3, or 4 for a gap base.
__device__ __forceinline__ uint32_t base_at(const IndexView &ix, uint64_t p) {
    if ((ix.gaps[p >> 5] >> (p & 31)) & 1u) return 4u;
    return (ix.packed[p >> 4] >> (2 * (p & 15))) & 3u;
}

// Base y of the target side T' of region R.
__device__ __forceinline__ uint32_t t_base(const IndexView &ix, const ARegion &R, uint64_t y) {
    if (R.o == 0) return base_at(ix, R.t0 + y);
    const uint32_t c = base_at(ix, R.t1 - 1 - y);
    return c < 4 ? 3u - c : 4u;
}

__device__ __forceinline__ uint32_t region_of(const uint64_t *off, uint32_t nr, uint64_t f) {
    uint32_t lo = 0, hi = nr;  // last region whose offset is <= f
    while (hi - lo > 1) {
        const uint32_t m = (lo + hi) >> 1;
        if (off[m] <= f) lo = m; else hi = m;
    }
    return lo;
}

__device__ __forceinline__ uint64_t first_at_least(const uint64_t *key, uint64_t n, uint64_t x) {
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t m = (lo + hi) >> 1;
        if (key[m] < x) lo = m + 1; else hi = m;
    }
    return lo;
}

// Seeds: a workgroup joins a part of a region's query positions with its target
// side, SEED_Y start positions at a time, held in LDS by the buckets of a
// one-to-one hash of their k-mers (76 KB: two workgroups per CU).
constexpr uint32_t SEED_THREADS = 1024;
constexpr uint32_t SEED_XLO = 16384, SEED_XHI = 65536;  // query positions per workgroup
constexpr uint32_t SEED_Y = 15 * SEED_THREADS;
constexpr uint32_t SEED_BITS = 13, SEED_TAG = 22 - SEED_BITS, SEED_POS = 14;
constexpr uint32_t SEED_BUCKETS = 1u << SEED_BITS;
static_assert(SEED_Y <= 1u << SEED_POS, "an entry holds its position");
constexpr uint32_t SEED_NOT = 63u << 22;  // no k-mer: as if it occurred too often
static_assert(MAXOCC + 1 < 63, "counts up to MAXOCC + 1 and SEED_NOT's fit above 22 bits");
struct SeedWork {
    uint32_t region, x0, x1;  // query positions [x0, x1) of the region
};

// The k-mer (k <= 11) at global position p, its first base lowest; false when
// it holds a gap base.
__device__ __forceinline__ bool kmer_at(const IndexView &ix, uint64_t p, uint32_t k,
                                        uint32_t &code) {
    const uint64_t e = p + k - 1;
    const uint64_t g = ((uint64_t)ix.gaps[e >> 5] << 32) | ix.gaps[p >> 5];
    const uint64_t b = ((uint64_t)ix.packed[e >> 4] << 32) | ix.packed[p >> 4];
    code = (uint32_t)(b >> (2 * (p & 15))) & ((1u << (2 * k)) - 1);
    return ((uint32_t)(g >> (p & 31)) & ((1u << k) - 1)) == 0;
}
__device__ __forceinline__ uint32_t revcomp_kmer(uint32_t c, uint32_t k) {
    const uint32_t r = __builtin_bitreverse32(~c);  // base order and each base's bits turned
    return (((r >> 1) & 0x55555555u) | ((r & 0x55555555u) << 1)) >> (32 - 2 * k);
}
// One to one on 22 bits: the upper SEED_BITS are the bucket, the rest the tag.
__device__ __forceinline__ uint32_t kmer_mix(uint32_t code) {
    return (code * 0x9E3779B1u) & ((1u << 22) - 1);
}

// 1. seed matches per query position (EMIT false: cnt[f], 0 for seeds that
// occur more than MAXOCC times in T'), then the matches themselves (EMIT true:
// keys region << 41 | (y - x + 2^20) << 20 | x at moff[f] on; cnt[f] counts
// down).  A target position is kept by its start on the forward strand; on
// strand 1 the query's k-mer is reverse-complemented instead.  A position
// belongs to the same thread in every round over the target, so cnt needs no
// atomics (between rounds it holds count << 22 | hash); buckets are in no fixed order, which nothing depends on: the
// matches of a query position differ in their diagonals.
// Bound by the instructions of a query position in every round, so an entry is
// compared without another read (tag and position in one word), four at a
// time, and the hash is taken once.  Sorting all targets' k-mers and searching
// them for every query position took 41 ms of 50 Mbp's regions (264 Mbp on
// either side); this takes 8.9 for the counts and 7.5 for the matches.
template <bool EMIT>
__global__ __launch_bounds__(SEED_THREADS, 8) void k_seeds(const IndexView ix, const ARegion *reg,
                                                        const SeedWork *work, const uint64_t *qoff,
                                                        uint32_t k, uint32_t *cnt,
                                                        const uint64_t *moff, uint64_t *mkey) {
    __shared__ uint32_t start[SEED_BUCKETS / 2 + 1];  // 16 bits per bucket: counts, ends, starts
    __shared__ uint32_t entry[SEED_Y + 4];            // tag << SEED_POS | position
    __shared__ uint32_t wsum[SEED_THREADS / 64];
    const uint32_t tid = threadIdx.x;
    const SeedWork w = work[blockIdx.x];
    const ARegion R = reg[w.region];
    const uint32_t nq = (uint32_t)(R.q1 - R.q0), nt = (uint32_t)(R.t1 - R.t0);
    const uint64_t f0 = qoff[w.region];
    const uint32_t starts = nt < k ? 0u : nt - k + 1;  // of target k-mers
    if (starts == 0) {
        if constexpr (!EMIT)
            for (uint32_t x = w.x0 + tid; x < w.x1; x += SEED_THREADS) cnt[f0 + x] = 0;
        return;
    }
    for (uint32_t g0 = 0; g0 < starts; g0 += SEED_Y) {
        const uint32_t n = min(SEED_Y, starts - g0);
        __syncthreads();  // the round before is done with the entries
        for (uint32_t i = tid; i <= SEED_BUCKETS / 2; i += SEED_THREADS) start[i] = 0;
        __syncthreads();
        const auto target_mix = [&](uint32_t y, uint32_t &m) {
            uint32_t code;
            if (!kmer_at(ix, R.t0 + g0 + y, k, code)) return false;
            m = kmer_mix(code);
            return true;
        };
        uint32_t m;
#pragma unroll 2
        for (uint32_t y = tid; y < n; y += SEED_THREADS)
            if (target_mix(y, m)) {
                const uint32_t b = m >> SEED_TAG;
                atomicAdd(&start[b >> 1], 1u << (16 * (b & 1)));
            }
        __syncthreads();
        // counts to ends: eight buckets per thread
        constexpr uint32_t PER = SEED_BUCKETS / 2 / SEED_THREADS;  // words per thread
        uint32_t c[PER], sum = 0;
#pragma unroll
        for (uint32_t u = 0; u < PER; u++) {
            c[u] = start[tid * PER + u];
            sum += (c[u] & 0xFFFFu) + (c[u] >> 16);
        }
        uint32_t at = sum;
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t v = __shfl_up(at, d);
            if ((tid & 63) >= d) at += v;
        }
        if ((tid & 63) == 63) wsum[tid >> 6] = at;
        __syncthreads();
        at -= sum;
        for (uint32_t v = 0; v < tid >> 6; v++) at += wsum[v];
#pragma unroll
        for (uint32_t u = 0; u < PER; u++) {
            const uint32_t mid = at + (c[u] & 0xFFFFu);
            at = mid + (c[u] >> 16);
            start[tid * PER + u] = mid | (at << 16);
        }
        if (tid == SEED_THREADS - 1) start[SEED_BUCKETS / 2] = at;
        __syncthreads();
        // entries, from the end of each bucket: its end becomes its start
#pragma unroll 2
        for (uint32_t y = tid; y < n; y += SEED_THREADS)
            if (target_mix(y, m)) {
                const uint32_t b = m >> SEED_TAG, sh = 16 * (b & 1);
                const uint32_t e = ((atomicSub(&start[b >> 1], 1u << sh) >> sh) & 0xFFFFu) - 1;
                entry[e] = ((m & ((1u << SEED_TAG) - 1)) << SEED_POS) | y;
            }
        __syncthreads();
        const bool last = g0 + SEED_Y >= starts;
#pragma unroll 2
        for (uint32_t x = w.x0 + tid; x < w.x1; x += SEED_THREADS) {
            // matches so far (EMIT: to come), and the k-mer's hash
            uint32_t left = EMIT || g0 ? cnt[f0 + x] : 0u;
            if (g0 == 0) {
                uint32_t code;
                if (EMIT && left == 0) continue;
                if (x + k > nq || !kmer_at(ix, R.q0 + x, k, code)) {
                    if constexpr (!EMIT) cnt[f0 + x] = last ? 0u : SEED_NOT;
                    continue;
                }
                m = kmer_mix(R.o ? revcomp_kmer(code, k) : code);
            } else {
                m = left & ((1u << 22) - 1);
                left >>= 22;
                if (EMIT ? left == 0 : left > MAXOCC) {
                    if (!EMIT && last) cnt[f0 + x] = 0;
                    continue;
                }
            }
            const uint32_t b = m >> SEED_TAG, tag = m & ((1u << SEED_TAG) - 1);
            const uint32_t s0 = start[b >> 1], s1 = start[(b >> 1) + 1];
            const uint32_t e1 = b & 1 ? s1 & 0xFFFFu : s0 >> 16;
            bool more = true;
            for (uint32_t e = b & 1 ? s0 >> 16 : s0 & 0xFFFFu; e < e1 && more; e += 4) {
                uint32_t v[4];
#pragma unroll
                for (uint32_t q = 0; q < 4; q++) v[q] = entry[e + q];
#pragma unroll
                for (uint32_t q = 0; q < 4; q++) {
                    if (e + q >= e1 || (v[q] >> SEED_POS) != tag || !more) continue;
                    if constexpr (EMIT) {
                        const uint32_t y = g0 + (v[q] & ((1u << SEED_POS) - 1));
                        const uint64_t ty = R.o ? starts - 1 - y : y;
                        left--;
                        mkey[moff[f0 + x] + left] =
                            ((uint64_t)w.region << 41) | ((ty + (1ull << 20) - x) << 20) | x;
                        more = left != 0;
                    } else {
                        more = ++left <= MAXOCC;
                    }
                }
            }
            if (!last)
                cnt[f0 + x] = (left << 22) | m;
            else if (!EMIT)
                cnt[f0 + x] = left <= MAXOCC ? left : 0u;
        }
    }
}

__global__ void k_run_starts(const uint64_t *mkey, uint64_t m, uint32_t *flag) {
    const uint64_t f = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= m) return;
    flag[f] = (f == 0 || mkey[f - 1] + 1 != mkey[f]) ? 1u : 0u;
}

struct Anchors {
    uint32_t *reg, *x, *y, *len;
};

// 2b. the first match of each run, then an anchor per run (a run ends where
// the next one starts)
__global__ void k_run_first(const uint32_t *flag, const uint32_t *pre, uint64_t m,
                            uint64_t *first) {
    const uint64_t f = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f < m && flag[f]) first[pre[f]] = f;
}

__global__ void k_anchor_emit(const uint64_t *mkey, uint64_t m, const uint64_t *first, uint64_t na,
                              uint32_t k, Anchors an) {
    const uint64_t a = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= na) return;
    const uint64_t f = first[a], e = a + 1 < na ? first[a + 1] : m;
    const uint64_t key = mkey[f];
    const uint32_t x = (uint32_t)(key & 0xFFFFF);
    const uint64_t d = (key >> 20) & 0x1FFFFF;
    an.reg[a] = (uint32_t)(key >> 41);
    an.x[a] = x;
    an.y[a] = (uint32_t)(d + x - (1ull << 20));
    an.len[a] = (uint32_t)(e - f) + k - 1;
}

__global__ void k_order_keys(Anchors an, uint64_t na, int by_end, uint64_t *key, uint32_t *val) {
    const uint64_t a = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= na) return;
    const uint64_t x = an.x[a] + (by_end ? an.len[a] : 0), y = an.y[a] + (by_end ? an.len[a] : 0);
    key[a] = ((uint64_t)an.reg[a] << 42) | (x << 21) | y;
    val[a] = (uint32_t)a;
}

// First entry of each region in an order whose keys carry the region in
// their top bits: bounds[r] for r in [0, nr], by binary search.
__global__ void k_region_bounds(const uint64_t *key, uint64_t n, int shift, uint32_t nr,
                                uint32_t *bounds) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r > nr) return;
    bounds[r] = (uint32_t)first_at_least(key, n, (uint64_t)r << shift);
}

struct Tier1 {
    int64_t *score;
    uint32_t *pred;
};

// A link from an anchor or chain ending at (bex, bey) to one starting at
// (ax, ay) whose first anchor has alen bases.  The successor's start is cut
// by o = max(0, bex - ax, bey - ay) so that it begins after the predecessor
// ends on both sides (anchors flanking an indel overlap whenever a base next
// to it matches by chance); false when the cut would take the whole first
// anchor.  dx, dy: the gaps left after the cut (both >= 0).
__device__ __forceinline__ bool link_trim(uint32_t bex, uint32_t bey, uint32_t ax, uint32_t ay,
                                          uint32_t alen, uint32_t &o, uint32_t &dx,
                                          uint32_t &dy) {
    uint32_t t = bex > ax ? bex - ax : 0u;
    if (bey > ay && bey - ay > t) t = bey - ay;
    if (t >= alen) return false;
    o = t;
    dx = ax + t - bex;
    dy = ay + t - bey;
    return true;
}

__device__ __forceinline__ uint32_t absdiff(uint32_t a, uint32_t b) { return a > b ? a - b : b - a; }

// What link_trim and a gap limit G ask of the y coordinates alone: the cut
// leaves a base of the first anchor (bey - ay < alen) and ay - bey <= G.  Most
// anchors of a large region are chance matches far off in y, so this settles
// nearly all pairs.
__device__ __forceinline__ bool y_in_reach(uint32_t bey, uint32_t ay, uint32_t alen, uint32_t G) {
    return ay - bey + (alen - 1) < G + alen;
}

// The best predecessor seen by a lane: largest value, then the larger start (x,
// then y) as one key, value << 42 | x << 21 | y (0 for values not above 0), so
// that taking a better one is a plain selection.  (Written as nested conditions
// on the three, with the members assigned under them, the compiler lost the
// predecessor's number where values were equal.)  Starts are unique within a
// region, so the choice does not depend on the order candidates are met.
// Values lie in (-2^21, 2^21).
struct Best1 {
    uint64_t key;
    uint32_t b;
    __device__ __forceinline__ int32_t value() const { return (int32_t)(key >> 42); }
    __device__ __forceinline__ void take(uint64_t k, uint32_t id) {
        const bool better = k > key;
        key = better ? k : key;
        b = better ? id : b;
    }
};
__device__ __forceinline__ uint64_t best_key(int32_t v, uint32_t x, uint32_t y) {
    return v > 0 ? ((uint64_t)v << 42) | ((uint64_t)x << 21) | y : 0;
}

// A 32-bit value of lane i (i the same in every lane).
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, uint32_t i) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)i);
}

// A 64-bit value that is the same in every lane, as a scalar.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
    return ((uint64_t)lane_u32((uint32_t)(v >> 32), 0) << 32) | lane_u32((uint32_t)v, 0);
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    for (int m = 32; m >= 1; m >>= 1) {
        const uint32_t o = __shfl_xor(v, m);
        v = o > v ? o : v;
    }
    return v;
}

// Scores are written by the lane that owns a node and read by every lane of
// the workgroup in later batches: workgroup-scope atomics, with a fence or a
// barrier after each batch.
__device__ __forceinline__ int64_t ld_score(const int64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void st_score(int64_t *p, int64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int32_t ld_score(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void st_score(int32_t *p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// 3a. tier-1 scores (the longest chains: a link costs the indel |dx - dy|
// it implies plus its cut, gaps at most G1), one workgroup of T1_WAVES waves
// per region.  Anchors are scored 64 at a time in (x, y) order, anchor k of
// a batch in lane k of every wave:
//  1. predecessors scored before the batch: the anchors ending in [x0 - G1,
//     the last window end of the batch) (x0 its first start), read in
//     blocks of 64 entries of the end order, dealt round robin to the waves
//     and read four at a time, one entry per lane; every lane tests every
//     entry against its own anchor, and the waves' best predecessors meet in
//     LDS.
//     LDS holds the last end x of each of the region's first nblk blocks, so
//     the window's first block is found without memory reads;
//  2. predecessors inside the batch (wave 0): anchor k's score is final once
//     anchors 0..k-1 are done, so k runs from first to last over the anchors
//     that have a later one in reach, and every later lane tests anchor k as
//     its predecessor.
// Only positive link values are kept and the choice among equal ones does
// not depend on the order candidates are met, so this equals scoring the
// anchors one at a time against every earlier anchor.  Candidates' lengths,
// scores and anchor ids come from arrays kept in end order.  Bound by the
// compares of the largest region's chance anchors: an entry no window of the
// batch holds is left out by its own lane, a pair too far apart in y after
// three instructions, and inside the batch only anchors that some later one is
// in reach of are taken one by one, which all waves find out (50 Mbp, all
// regions: 25.6 -> 5.9 ms, 6.3 with 4 waves).
__global__ __launch_bounds__(64 * T1_WAVES) void k_tier1(const uint64_t *xykey, const uint32_t *byxy,
                                              const uint32_t *alen, const uint64_t *endkey,
                                              const uint32_t *byend, const uint32_t *elen,
                                              const uint32_t *pos_e, const uint32_t *bnd,
                                              uint32_t nr, uint32_t G1, Tier1 t1,
                                              int64_t *score_e, uint32_t nblk,
                                              const uint32_t *large_first) {
    extern __shared__ uint32_t t1_lds[];
    uint32_t *const exhi = t1_lds;  // [nblk]
    __shared__ Best1 part[T1_WAVES][64];  // per wave and anchor
    __shared__ uint64_t rows[T1_WAVES];   // per wave: anchors with a link inside the batch
    if (blockIdx.x >= nr) return;
    const uint32_t r = large_first[blockIdx.x];
    const uint32_t lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const uint32_t lo = bnd[r], hi = bnd[r + 1];
    const uint32_t nbr = (hi - lo + 63) / 64;  // blocks of the region's end order
    const uint32_t nbl = min(nbr, nblk);        // blocks with their last end in LDS
    const auto block_end = [&](uint32_t j) -> uint32_t {
        if (j < nbl) return exhi[j];
        return (uint32_t)(endkey[min(lo + 64 * j + 63, hi - 1)] >> 21) & 0x1FFFFFu;
    };
    for (uint32_t j = threadIdx.x; j < nbl; j += 64 * T1_WAVES)
        exhi[j] = (uint32_t)(endkey[min(lo + 64 * j + 63, hi - 1)] >> 21) & 0x1FFFFFu;
    __syncthreads();
    const uint64_t rk = (uint64_t)r << 42;
    uint32_t jlo = 0;  // first block that ends at or after the batch's window start
    for (uint32_t u0 = lo; u0 < hi; u0 += 64) {
        const uint32_t cnt = min(64u, hi - u0);
        const bool mine = lane < cnt;
        uint32_t a = NONE32, x = 0, y = 0, len = 0, apos = 0;
        if (mine) {
            const uint64_t key = xykey[u0 + lane];
            a = byxy[u0 + lane];
            x = (uint32_t)(key >> 21) & 0x1FFFFFu;
            y = (uint32_t)key & 0x1FFFFFu;
            len = alen[a];
            apos = pos_e[a];
        }
        const uint32_t xend = x + len;  // this anchor's window: ends in [x - G1, xend)
        const uint32_t x0 = lane_u32(x, 0), y0 = lane_u32(y, 0);  // the batch's first start
        const uint32_t xend_max = wave_max_u32(mine ? xend : 0u);
        const uint64_t khi_max = rk | ((uint64_t)xend_max << 21);
        Best1 B{0, NONE32};
        // 1. predecessors scored before the batch
        const uint32_t xlo = x0 >= G1 ? x0 - G1 : 0;
        for (;;) {  // blocks ending before every window: a prefix, and x0 only grows
            const uint32_t j = jlo + lane;
            const uint32_t cb = (uint32_t)__popcll(__ballot(j < nbr && block_end(j) < xlo));
            jlo += cb;
            if (cb < 64) break;
        }
        const auto scan = [&](uint64_t ek, uint32_t el, int32_t es, uint32_t esl) {
            // entries some window of the batch holds and that are scored already,
            // told by their own lanes; then one at a time against every lane's anchor
            const uint32_t lex = (uint32_t)(ek >> 21) & 0x1FFFFFu, lbx = lex - el;
            const uint32_t lby = ((uint32_t)ek & 0x1FFFFFu) - el;
            uint64_t todo = __ballot(ek < khi_max && lex + G1 >= x0 && (lbx < x0 || (lbx == x0 && lby < y0)));
            for (; todo; todo &= todo - 1) {
                const uint32_t i = (uint32_t)__builtin_ctzll(todo);
                const uint32_t elo = lane_u32((uint32_t)ek, i), ehi = lane_u32((uint32_t)(ek >> 32), i);
                const uint32_t bex = (uint32_t)((((uint64_t)ehi << 32) | elo) >> 21) & 0x1FFFFFu;
                const uint32_t bey = elo & 0x1FFFFFu;
                const bool pass = mine & (bex < xend) & (bex + G1 >= x) & y_in_reach(bey, y, len, G1);
                if (!__ballot(pass)) continue;
                const uint32_t bl = lane_u32(el, i), bx = bex - bl, by = bey - bl;
                const int32_t sb = (int32_t)lane_u32((uint32_t)es, i);
                const uint32_t b = lane_u32(esl, i);
                uint32_t o, dx, dy;
                if (pass && link_trim(bex, bey, x, y, len, o, dx, dy) && (dx > dy ? dx : dy) <= G1)
                    B.take(best_key(sb - (int32_t)(absdiff(dx, dy) + o), bx, by), b);
            }
        };
        uint32_t dealt = 0;  // blocks met so far (dealt round robin to the waves)
        for (uint32_t j0 = jlo; j0 < nbr; j0 += 64) {
            const uint32_t j = j0 + lane;
            // block j starts no earlier than block j - 1 ends
            const bool beyond = j >= nbr || (j > jlo && block_end(j - 1) >= xend_max);
            const uint64_t mbey = __ballot(beyond);
            const uint64_t mall = mbey ? (mbey & (0ull - mbey)) - 1 : ~0ull;
            uint64_t mneed = 0;  // this wave's share
            for (uint64_t m = mall; m; m &= m - 1, dealt++)
                if (dealt % T1_WAVES == wave) mneed |= m & (0ull - m);
            while (mneed) {
                uint32_t jb[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    jb[q] = mneed ? j0 + (uint32_t)__builtin_ctzll(mneed) : nbr;
                    mneed &= mneed - 1;
                }
                uint64_t ek[4];
                uint32_t el[4], esl[4];
                int32_t es[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const uint32_t v = lo + 64 * jb[q] + lane;
                    const bool ok = jb[q] < nbr && v < hi;
                    ek[q] = ok ? endkey[v] : ~0ull;
                    el[q] = ok ? elen[v] : 0u;
                    es[q] = ok ? (int32_t)ld_score(score_e + v) : INT32_MIN;
                    esl[q] = ok ? byend[v] : NONE32;
                }
#pragma unroll
                for (int q = 0; q < 4; q++)
                    if (jb[q] < nbr) scan(ek[q], el[q], es[q], esl[q]);
            }
            if (mbey) break;
        }
        // anchors of the batch that some later one of it may follow, whatever
        // their scores: each wave tests a share of them
        const auto follows = [&](uint32_t k) {
            const uint32_t lk = lane_u32(len, k);
            const uint32_t exk = lane_u32(x, k) + lk, eyk = lane_u32(y, k) + lk;
            return (lane > k) & mine & (exk < xend) & (exk + G1 >= x) & y_in_reach(eyk, y, len, G1);
        };
        uint64_t own = 0;
        for (uint32_t k = wave; k + 1 < cnt; k += T1_WAVES)
            if (__ballot(follows(k))) own |= 1ull << k;
        if (lane == 0) rows[wave] = own;
        part[wave][lane] = B;
        __syncthreads();
        if (wave == 0) {
            for (uint32_t q = 1; q < T1_WAVES; q++) {
                const Best1 o = part[q][lane];
                B.take(o.key, o.b);
                own |= rows[q];
            }
            // 2. predecessors inside the batch
            for (own = uniform_u64(own); own; own &= own - 1) {
                const uint32_t k = (uint32_t)__builtin_ctzll(own);
                const int32_t sk = (int32_t)lane_u32((uint32_t)((int32_t)len + B.value()), k);
                const uint32_t xk = lane_u32(x, k), yk = lane_u32(y, k), lk = lane_u32(len, k);
                const uint32_t exk = xk + lk, eyk = yk + lk, ak = lane_u32(a, k);
                if (follows(k)) {
                    uint32_t o, dx, dy;
                    if (link_trim(exk, eyk, x, y, len, o, dx, dy) && (dx > dy ? dx : dy) <= G1)
                        B.take(best_key(sk - (int32_t)(absdiff(dx, dy) + o), xk, yk), ak);
                }
            }
            if (mine) {
                const int64_t sa = (int64_t)len + B.value();  // scores < 2^21
                st_score(t1.score + a, sa);
                st_score(score_e + apos, sa);
                t1.pred[a] = B.b;
            }
        }
        __syncthreads();  // scores seen by every wave
    }
}

// Lengths and end-order positions of the anchors: elen[v] = len(byend[v]),
// pos_e[byend[v]] = v.
__global__ void k_end_order(const Anchors an, const uint32_t *byend, uint64_t na, uint32_t *elen,
                            uint32_t *pos_e) {
    const uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= na) return;
    const uint32_t a = byend[v];
    elen[v] = an.len[a];
    pos_e[a] = (uint32_t)v;
}

// The score order of tier-1 extraction: (region, score descending, x), then
// y by an earlier stable pass.
__global__ void k_score_keys(Anchors an, uint64_t na, const Tier1 t1, int pass, uint64_t *key,
                             uint32_t *val, const uint32_t *perm) {
    const uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= na) return;
    const uint32_t a = perm ? perm[u] : (uint32_t)u;
    if (pass == 0) {
        key[u] = an.y[a];
    } else {
        const uint64_t inv = (1ull << 21) - 1 - (uint64_t)t1.score[a];  // scores < 2^21
        key[u] = ((uint64_t)an.reg[a] << 41) | (inv << 20) | an.x[a];
    }
    val[u] = a;
}

struct Chains1 {
    uint32_t *member;        // anchors of the chains, chain by chain, each in x order
    uint32_t *start, *end;   // member range of each node (slot)
    uint32_t *count;         // chains per region
    uint32_t *cx, *cy, *cex, *cey;  // node extents
    int64_t *w;                     // node weights
    uint32_t *flen;                 // length of each node's first anchor
};

// 3b, 4b. Chains by score: entries (anchors, then nodes) are taken in extraction
// order; one not yet used starts a chain that follows kept predecessors until
// a used one (or none); the chain's entries in start order are its members.  So
// an entry belongs to the chain of the first entry, in extraction order, among
// itself and all that reach it over kept predecessors: what is used earlier on
// the way there is used by one of these too.  That minimum is taken over paths
// of 1, 2, 4, ... predecessors, for all regions at once; sorted by it, stably
// from start order, the entries are the members of the chains in the order in
// which these are taken out.
// (Before, one wave per region followed the chains one after another: 18.5 ms
// for both tiers of 50 Mbp's regions, where this takes 4.5.)

// own[id] = the entry's place in extraction order, jump[id] = its predecessor.
__global__ void k_own_init(const uint32_t *order, uint64_t na, const uint32_t *nlive,
                           const uint32_t *pred, uint32_t *own, uint32_t *jump) {
    const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= na || (nlive && e >= *nlive)) return;
    const uint32_t id = order[e];
    own[id] = (uint32_t)e;
    jump[id] = pred[id];
}

// One doubling: jin leads 2^i predecessors on, jout twice as far.  own only
// falls, to places of entries that reach the entry, so a value that has
// fallen in the same launch already does no harm.
__global__ void k_own_double(const uint32_t *list, uint64_t na, const uint32_t *nlive,
                             uint32_t *own, const uint32_t *jin, uint32_t *jout) {
    const uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= na || (nlive && u >= *nlive)) return;
    const uint32_t id = list[u], p = jin[id];
    uint32_t next = NONE32;
    if (p != NONE32) {
        atomicMin(own + p, own[id]);
        next = jin[p];
    }
    jout[id] = next;
}

__global__ void k_own_keys(const uint32_t *list, uint64_t na, const uint32_t *nlive,
                           const uint32_t *own, uint32_t *key, uint32_t *val) {
    const uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= na) return;
    const bool live = !nlive || u < *nlive;
    key[u] = live ? own[list[u]] : ~0u;  // its low bits sort after every place
    val[u] = live ? list[u] : NONE32;
}

// The three for few entries, by one workgroup in LDS: a small call is bound by its
// launches (one region of 1.5 kbp: 1,031 us a call; 1,066 with a launch per doubling).
constexpr uint32_t OWN_SMALL = 4096;
__global__ __launch_bounds__(1024) void k_own_small(const uint32_t *order, const uint32_t *list,
                                                    uint32_t na, const uint32_t *nlive,
                                                    const uint32_t *pred, uint32_t most,
                                                    uint32_t *key, uint32_t *val) {
    __shared__ uint32_t own[OWN_SMALL], jump[2][OWN_SMALL];
    const uint32_t live = nlive ? min(na, *nlive) : na;
    for (uint32_t e = threadIdx.x; e < live; e += 1024) {
        const uint32_t id = order[e];
        own[id] = e;
        jump[0][id] = pred[id];
    }
    __syncthreads();
    uint32_t from = 0;
    for (uint32_t reach = 1; reach < most; reach *= 2, from ^= 1) {
        for (uint32_t u = threadIdx.x; u < live; u += 1024) {
            const uint32_t id = list[u], p = jump[from][id];
            uint32_t next = NONE32;
            if (p != NONE32) {
                atomicMin(&own[p], own[id]);
                next = jump[from][p];
            }
            jump[from ^ 1][id] = next;
        }
        __syncthreads();
    }
    for (uint32_t u = threadIdx.x; u < na; u += 1024) {
        key[u] = u < live ? own[list[u]] : ~0u;
        val[u] = u < live ? list[u] : NONE32;
    }
}

__global__ void k_own_heads(const uint32_t *key, uint64_t na, const uint32_t *nlive,
                            uint32_t *flag) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= na) return;
    flag[j] = (!nlive || j < *nlive) && (j == 0 || key[j - 1] != key[j]) ? 1u : 0u;
}

// Chains per region, from the chains before each member position.
__global__ void k_chain_count(const uint32_t *bnd, uint32_t nr, const uint32_t *pre,
                              uint32_t *count) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < nr) count[r] = pre[bnd[r + 1]] - pre[bnd[r]];
}

// 3c. the tier-1 chains as nodes: a region's in the slots from bnd[r] on.  A
// chain's weight is what its scores grew by, its links' costs included.
__global__ void k_nodes1(const Anchors an, const uint32_t *bnd, uint64_t na, const uint32_t *flag,
                         const uint32_t *pre, const uint64_t *first, const int64_t *score,
                         Chains1 c) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= na || !flag[j]) return;
    const uint32_t i = pre[j];
    const uint64_t end = i + 1 < pre[na] ? first[i + 1] : na;
    const uint32_t f = c.member[j], l = c.member[end - 1];
    const uint32_t lo = bnd[an.reg[f]], node = lo + (i - pre[lo]);
    c.start[node] = (uint32_t)j;
    c.end[node] = (uint32_t)end;
    c.cx[node] = an.x[f];
    c.cy[node] = an.y[f];
    c.cex[node] = an.x[l] + an.len[l];
    c.cey[node] = an.y[l] + an.len[l];
    c.w[node] = score[l] - score[f] + an.len[f];
    c.flen[node] = an.len[f];
}

__global__ void k_slot_regions(const Anchors an, const uint32_t *byxy, uint64_t na,
                               uint32_t *reg_of_slot) {
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s < na) reg_of_slot[s] = an.reg[byxy[s]];
}

// node keys (region, x, y) of the tier-1 chains; unused slots sort last
__global__ void k_node_keys(const uint32_t *bnd, const uint32_t *reg_of_slot, uint64_t na,
                            const Chains1 c, uint64_t *key, uint32_t *val) {
    const uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= na) return;
    const uint32_t r = reg_of_slot[s];
    const bool live = s - bnd[r] < c.count[r];
    key[s] = live ? (((uint64_t)r << 42) | ((uint64_t)c.cx[s] << 21) | c.cy[s]) : ~0ull;
    val[s] = (uint32_t)s;
}

struct Final {
    uint32_t *member;        // tier-1 node slots of the final chains, chain by chain
    uint32_t *start, *end;   // member range of each final chain
    uint32_t *count;         // final chains per region
};

// Lower bound of the tier-2 cost of a link whose predecessor ends at x - d
// or earlier (d >= 0): with equal gaps the cost is min(dx, dy) = dx >= d;
// with unequal ones it is at least 10 + ceil(dx / 10) (the smaller gap plus
// a tenth of the difference is at least a tenth of dx); both grow with dx,
// and the trim only adds.
__device__ __forceinline__ int32_t tier2_min_cost(uint32_t d) {
    const uint32_t u = 10 + (d + 9) / 10;
    return (int32_t)(d < u ? d : u);
}

// The cost of a link with gaps dx, dy <= TIER2_GAP and cut o < 2^20.
__device__ __forceinline__ int32_t tier2_cost(uint32_t dx, uint32_t dy, uint32_t o) {
    const uint32_t g = absdiff(dx, dy);
    return (int32_t)((dx < dy ? dx : dy) + (g > 0 ? 10 + (g + 9) / 10 : 0) + o);
}

// A node (tier-1 chain) as tier 2 reads it, in start order.
struct Node2 {
    uint32_t x, y, ex, ey;  // its first base and past its last
    uint32_t flen;          // length of its first anchor
    int32_t w;
    uint32_t epos;  // its entry in end order
    uint32_t slot;
};
// A node's best predecessor: value << 32 | start-order entry (among equal
// values the later start wins, as starts are unique within a region); 0 none.
__device__ __forceinline__ int32_t best_val(uint64_t b) { return (int32_t)(b >> 32); }

// 4a. tier-2 scores, one workgroup of T2_WAVES waves per region: the
// region's nodes (tier-1 chains) are the entries [nbnd[r], nbnd[r+1]) of
// `node` (by start) and of ekey (by end, region | ex | ey) with ue (start-order
// entries); the predecessors of a node are the earlier ones ending in
// [x - 10000, x + first anchor length), with the affine cost plus the cut.
// Scores are kept in start order (score_s) and by end order (score_e).  Nodes
// are scored 64 at a time in start order, node k of a batch in lane k of every
// wave:
//  1. predecessors scored before the batch: the end order is cut into
//     blocks of 64 entries, and LDS holds, for the first nblk blocks of the
//     region, the last end x of each block (static) and the best score of
//     its nodes scored so far.  A block that cannot give any node of the
//     batch a positive link value (its best score does not exceed the least
//     cost of a link from its last end to the batch's first start) is not
//     read; the others are dealt round robin to the waves, the last (and
//     highest scored) first, which read them four at a time, one entry per
//     lane.  Every entry that is still a candidate is tested against every
//     lane's node for reach and the least cost; the pairs left are queued and
//     scored 64 at a time;
//  2. predecessors inside the batch: the links' costs, which need no scores,
//     by all waves; then wave 0: node k's score is final once nodes 0..k-1 are
//     done, so k runs from first to last and every later lane tests node k as
//     its predecessor.
// Only positive link values are kept and the choice among equal ones does
// not depend on the order candidates are met, so this equals scoring the
// nodes one at a time against every earlier node.  Bound by the instructions
// of the largest region's workgroup: an entry whose score the batch's first
// start is too far for is left out by its own lane; an entry is in reach of
// one or two nodes of a batch, so their full scoring is gathered; and a node's
// inputs come in one load, a batch ahead (50 Mbp, all regions: 25.8 -> 13.5 ms,
// 16.3 with 8 waves).
__global__ __launch_bounds__(64 * T2_WAVES) void k_tier2(
    const uint32_t *nbnd, uint32_t nr, const Node2 *node, const uint64_t *ekey, const uint32_t *ue,
    int32_t *score_s, int32_t *score_e, uint32_t *pred_s, uint32_t nblk,
    const uint32_t *large_first) {
    extern __shared__ uint32_t t2_lds[];
    uint32_t *const exhi = t2_lds;                                      // [nblk]
    int32_t *const bmax = reinterpret_cast<int32_t *>(t2_lds + nblk);  // [nblk]
    __shared__ unsigned long long best[2][64];  // per node of the batch, and for the next
    __shared__ int32_t inner[64][64];  // the cost of node l following node k of the batch
    __shared__ uint16_t queue[T2_WAVES][128];  // pairs to score: entry << 6 | node
    if (blockIdx.x >= nr) return;
    const uint32_t r = large_first[blockIdx.x];
    const uint32_t lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const uint32_t lo = nbnd[r], hi = nbnd[r + 1];
    const uint32_t nbr = (hi - lo + 63) / 64;  // blocks of the region
    const uint32_t nbl = min(nbr, nblk);        // blocks with bounds in LDS
    const auto block_end = [&](uint32_t j) -> uint32_t {  // end x of block j's last entry
        if (j < nbl) return exhi[j];
        return (uint32_t)(ekey[min(lo + 64 * j + 63, hi - 1)] >> 21) & 0x1FFFFFu;
    };
    for (uint32_t j = threadIdx.x; j < nbl; j += 64 * T2_WAVES) {
        exhi[j] = (uint32_t)(ekey[min(lo + 64 * j + 63, hi - 1)] >> 21) & 0x1FFFFFu;
        bmax[j] = INT32_MIN;
    }
    if (wave == 0) best[0][lane] = 0;
    uint32_t odd = 0;  // the batch's half of best
    __syncthreads();
    const uint64_t rk = (uint64_t)r << 42;
    uint16_t *const wq = queue[wave];
    uint32_t jlo = 0;  // first block that ends at or after the batch's window start
    Node2 ahead{};     // the next batch's node
    if (lo + lane < hi) ahead = node[lo + lane];
    for (uint32_t u0 = lo; u0 < hi; u0 += 64) {
        const uint32_t cnt = min(64u, hi - u0);
        const bool mine = lane < cnt;
        const Node2 N = ahead;
        ahead = Node2{};
        if (u0 + 64 + lane < hi) ahead = node[u0 + 64 + lane];
        const uint32_t x = N.x, y = N.y, flen = N.flen;
        const uint32_t xend = x + flen;  // this node's window: ends in [x - 10000, xend)
        const uint32_t x0 = lane_u32(x, 0);  // the batch's first start
        const uint32_t xend_max = wave_max_u32(mine ? xend : 0u);
        const uint64_t khi_max = rk | ((uint64_t)xend_max << 21);
        // 1. predecessors scored before the batch
        const uint32_t xlo = x0 >= TIER2_GAP ? x0 - TIER2_GAP : 0;
        for (;;) {  // blocks ending before every window: a prefix, and x0 only grows
            const uint32_t j = jlo + lane;
            const uint32_t cb = (uint32_t)__popcll(__ballot(j < nbr && block_end(j) < xlo));
            jlo += cb;
            if (cb < 64) break;
        }
        const auto scan = [&](uint64_t ek, uint32_t eu, int32_t es) {
            // entries before the windows' end, scored already, whose score exceeds
            // the least cost of a link to the batch's first start (the others are no
            // nearer), told by their own lanes
            const uint32_t lex = (uint32_t)(ek >> 21) & 0x1FFFFFu, ley = (uint32_t)ek & 0x1FFFFFu;
            uint64_t todo =
                __ballot(ek < khi_max && eu < u0 && es > tier2_min_cost(x0 > lex ? x0 - lex : 0));
            const int32_t least = max(best_val(best[odd][lane]), 1);
            uint32_t nq = 0;  // pairs queued
            while (todo || nq) {
                while (todo && nq <= 64) {
                    const uint32_t i = (uint32_t)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    const uint32_t bex = lane_u32(lex, i), bey = lane_u32(ley, i);
                    const int32_t sb = (int32_t)lane_u32((uint32_t)es, i);
                    const bool pass = mine & (bex < xend) & y_in_reach(bey, y, flen, TIER2_GAP) &
                                      (sb - tier2_min_cost(x > bex ? x - bex : 0) >= least);
                    const uint64_t p = __ballot(pass);
                    if (!p) continue;
                    if (pass)
                        wq[nq + __builtin_amdgcn_mbcnt_hi((uint32_t)(p >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)p, 0))] =
                            (uint16_t)(i << 6 | lane);
                    nq += (uint32_t)__popcll(p);
                }
                if (!nq) break;
                // the last 64 pairs at most, one per lane
                const uint32_t m = min(nq, 64u);
                nq -= m;
                __builtin_amdgcn_wave_barrier();
                const uint32_t pr = lane < m ? wq[nq + lane] : 0u;
                __builtin_amdgcn_wave_barrier();
                const uint32_t i = pr >> 6, l = pr & 63;
                const uint32_t bex = __shfl(lex, i), bey = __shfl(ley, i), bu = __shfl(eu, i);
                const int32_t sb = __shfl(es, i);
                const uint32_t px = __shfl(x, l), py = __shfl(y, l), pf = __shfl(flen, l);
                uint32_t o, dx, dy;
                if (lane < m && link_trim(bex, bey, px, py, pf, o, dx, dy) &&
                    (dx > dy ? dx : dy) <= TIER2_GAP) {
                    const int32_t val = sb - tier2_cost(dx, dy, o);
                    if (val > 0)
                        atomicMax(&best[odd][l], ((unsigned long long)(uint32_t)val << 32) | bu);
                }
            }
        };
        // the first block past every window: block j starts no earlier than block
        // j - 1 ends
        uint32_t jhi = jlo;
        for (;;) {
            const uint32_t j = jhi + lane;
            const uint64_t mbey =
                __ballot(j >= nbr || (j > jlo && block_end(j - 1) >= xend_max));
            jhi += mbey ? (uint32_t)__builtin_ctzll(mbey) : 64u;
            if (mbey) break;
        }
        // blocks from the last on: their scores are the highest, and drop entries of
        // the others
        uint32_t dealt = 0;  // needed blocks met so far
        for (uint32_t jt = jhi; jt > jlo; jt -= min(64u, jt - jlo)) {
            const uint32_t j = jt - 1 - lane;  // lane 0: the last block of the group
            bool need = lane < jt - jlo;
            if (need && j < nbl) {
                const uint32_t eh = exhi[j];
                need = bmax[j] > tier2_min_cost(x0 > eh ? x0 - eh : 0);
            }
            // this wave's share: every T2_WAVES-th needed block
            uint64_t mine_b = 0;
            for (uint64_t m = __ballot(need); m; m &= m - 1, dealt++)
                if (dealt % T2_WAVES == wave) mine_b |= m & (0ull - m);
            while (mine_b) {
                uint32_t jb[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    jb[q] = mine_b ? jt - 1 - (uint32_t)__builtin_ctzll(mine_b) : nbr;
                    mine_b &= mine_b - 1;
                }
                uint64_t ek[4];
                uint32_t eu[4];
                int32_t es[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const uint32_t v = lo + 64 * jb[q] + lane;
                    const bool ok = jb[q] < nbr && v < hi;
                    ek[q] = ok ? ekey[v] : ~0ull;
                    eu[q] = ok ? ue[v] : NONE32;
                    es[q] = ok ? ld_score(score_e + v) : INT32_MIN;
                }
#pragma unroll
                for (int q = 0; q < 4; q++)
                    if (jb[q] < nbr) scan(ek[q], eu[q], es[q]);
            }
        }
        // the costs of the links inside the batch, a share of the rows per wave
        for (uint32_t k = wave; k + 1 < cnt; k += T2_WAVES) {
            const uint32_t exk = lane_u32(N.ex, k), eyk = lane_u32(N.ey, k);
            int32_t cost = T2_NEVER;
            if ((lane > k) & mine & (exk < xend) & y_in_reach(eyk, y, flen, TIER2_GAP)) {
                uint32_t o, dx, dy;
                if (link_trim(exk, eyk, x, y, flen, o, dx, dy) &&
                    (dx > dy ? dx : dy) <= TIER2_GAP)
                    cost = tier2_cost(dx, dy, o);
            }
            inner[k][lane] = cost;
        }
        __syncthreads();
        if (wave == 0) {
            const uint64_t b = best[odd][lane];
            best[odd ^ 1][lane] = 0;
            int32_t bv = best_val(b);
            uint32_t bu = bv > 0 ? (uint32_t)b : NONE32;
            // 2. predecessors inside the batch.  They start after every other one and
            // in the order of their lanes, so a later one wins among equal values.
#pragma unroll 8
            for (uint32_t k = 0; k + 1 < cnt; k++) {
                const int32_t val = (int32_t)lane_u32((uint32_t)(N.w + bv), k) - inner[k][lane];
                const bool take = val >= max(bv, 1);
                bv = take ? val : bv;
                bu = take ? u0 + k : bu;
            }
            if (mine) {
                const int32_t sa = N.w + bv;
                st_score(score_e + N.epos, sa);
                score_s[u0 + lane] = sa;
                pred_s[u0 + lane] = bu;
                const uint32_t jp = (N.epos - lo) / 64;  // the node's block in end order
                if (jp < nbl) atomicMax(bmax + jp, sa);
            }
        }
        odd ^= 1;
        __syncthreads();  // scores and block bounds seen by every wave
    }
}

// Tier 2's inputs by start order, and the start-order entries by end order.
__global__ void k_node_starts(const uint32_t *nodes, uint64_t na, const uint32_t *nlive,
                              const uint32_t *pos_e, const Chains1 c, Node2 *node, uint32_t *ue) {
    const uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= na || u >= *nlive) return;
    const uint32_t s = nodes[u];
    Node2 n;
    n.x = c.cx[s];
    n.y = c.cy[s];
    n.ex = c.cex[s];
    n.ey = c.cey[s];
    n.flen = c.flen[s];
    n.w = (int32_t)c.w[s];
    n.epos = pos_e[s];
    n.slot = s;
    node[u] = n;
    ue[n.epos] = (uint32_t)u;
}

// Tier 2's results by slot.
__global__ void k_node_results(const Node2 *node, uint64_t na, const uint32_t *nlive,
                               const int32_t *score_s, const uint32_t *pred_s, int64_t *score,
                               uint32_t *pred) {
    const uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= na || u >= *nlive) return;
    const uint32_t s = node[u].slot, p = pred_s[u];
    score[s] = score_s[u];
    pred[s] = p == NONE32 ? NONE32 : node[p].slot;
}

// Most nodes of one region (entries between consecutive region bounds).
__global__ void k_max_span(const uint32_t *bnd, uint32_t nr, uint32_t *out) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < nr) atomicMax(out, bnd[r + 1] - bnd[r]);
}

// pos_e[nodes_e[v]] = v: the end-order entry of every node slot.
__global__ void k_invert(const uint32_t *nodes_e, uint64_t na, uint32_t *pos_e) {
    const uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < na) pos_e[nodes_e[v]] = (uint32_t)v;
}

// Keys of the node entries: pass 0 by end (region, ex, ey); pass 1 and 2
// the extraction order, y first (stable), then (region, score descending,
// x).  Entries past the live nodes of every region sort last.
__global__ void k_node_keys2(const uint32_t *nodes, uint64_t na, const uint32_t *nlive,
                             const uint32_t *reg_of_slot, const Chains1 c, const int64_t *score,
                             int pass, const uint32_t *perm, uint64_t *key, uint32_t *val) {
    const uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= na) return;
    const uint32_t e = perm ? perm[u] : (uint32_t)u;  // entry of `nodes`
    const uint32_t s = nodes[e];
    const bool live = e < *nlive;
    const uint32_t r = reg_of_slot[s];
    if (pass == 0) {
        key[u] = live ? (((uint64_t)r << 42) | ((uint64_t)c.cex[s] << 21) | c.cey[s]) : ~0ull;
        val[u] = s;
    } else if (pass == 1) {
        key[u] = live ? c.cy[s] : ~0ull;
        val[u] = e;
    } else {
        // scores lie in (-2^20, 2^20]: shifted by 2^20 they fit 22 bits
        const uint64_t inv = (1ull << 22) - 1 - (uint64_t)(score[s] + (1ll << 20));
        key[u] = live ? (((uint64_t)r << 42) | (inv << 20) | c.cx[s]) : ~0ull;
        val[u] = s;
    }
}

// 4c. the final chains: a region's entries from nbnd[r] on.
__global__ void k_finals(const uint32_t *reg_of_slot, const uint32_t *nbnd, uint64_t na,
                         const uint32_t *nlive, const uint32_t *flag, const uint32_t *pre,
                         const uint64_t *first, Final fin) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= na || !flag[j]) return;
    const uint32_t i = pre[j];
    const uint32_t lo = nbnd[reg_of_slot[fin.member[j]]], at = lo + (i - pre[lo]);
    fin.start[at] = (uint32_t)j;
    fin.end[at] = i + 1 < pre[na] ? (uint32_t)first[i + 1] : *nlive;
}

// Final chain g (global, in region order) as (region, entry).
__device__ __forceinline__ void final_of(const uint64_t *foff, uint32_t nr, uint64_t g,
                                         const uint32_t *nbnd, uint32_t &r, uint32_t &e) {
    r = region_of(foff, nr, g);
    e = nbnd[r] + (uint32_t)(g - foff[r]);
}

// Calls visit(anchor) for the anchors of final chain entry e, in order.
template <class F>
__device__ __forceinline__ void walk_anchors(const Chains1 &c, const Final &fin, uint32_t e,
                                             F &&visit) {
    for (uint32_t s = fin.start[e]; s < fin.end[e]; s++) {
        const uint32_t node = fin.member[s];
        for (uint32_t m = c.start[node]; m < c.end[node]; m++) visit(c.member[m]);
    }
}

// A stretch between consecutive anchors of a final chain.
struct Seg {
    uint32_t chain;   // final chain (global id)
    uint32_t region;
    uint32_t qx, ty;  // start of the stretch on Q and T'
    uint32_t dx, dy;
    uint32_t keep;    // bases of the anchor after it, past the anchor's cut
    uint32_t _pad;
    uint64_t cells;   // offset of its traceback bytes
    uint64_t ops;     // offset of its column operations
    uint64_t rows;    // offset of its rolling score rows
};

__device__ __forceinline__ uint64_t seg_cells(uint32_t dx, uint32_t dy) {
    const uint64_t c = (uint64_t)(dx + 1) * (dy + 1);
    return c <= DP_CELLS ? c : 0;  // 0: the diagonal stand-in, no table
}

// Traceback tables hold one byte per cell, line by line, each line padded to
// a multiple of 8 bytes (tables start at multiples of 8 too), so that eight
// cells of a line are written with one 8-byte store.  A line is a row (query
// base i), except in the wave aligner's tables of stretches with dx > dy,
// whose lines are columns (target base j); room for either.
__device__ __forceinline__ uint32_t tb_pitch(uint32_t d) { return (d + 1 + 7) & ~7u; }
__device__ __forceinline__ uint64_t seg_tb_bytes(uint32_t dx, uint32_t dy) {
    if (!seg_cells(dx, dy)) return 0;
    const uint64_t rows = (uint64_t)(dx + 1) * tb_pitch(dy);
    const uint64_t cols = (uint64_t)(dy + 1) * tb_pitch(dx);
    return dx > dy && cols > rows ? cols : rows;
}

// Stretches of at least `wave_cells` cells are aligned by one 64-lane
// workgroup each (k_align_wave), which holds the shorter side in its
// registers: at most 1,024 of its DP_CELLS cells' lines, WAVE_S per lane.  The
// others are aligned by one thread each (k_align_segs).
constexpr uint32_t WAVE_S = 16;
static_assert((uint64_t)(64 * WAVE_S) * (64 * WAVE_S) >= DP_CELLS, "the shorter side fits");
__device__ __forceinline__ bool seg_wave(uint32_t dx, uint32_t dy, uint32_t wave_cells) {
    const uint64_t c = seg_cells(dx, dy);
    return c && c >= wave_cells;
}
// Rolling score cells a stretch needs in memory: the thread aligner's.
__device__ __forceinline__ uint64_t seg_rows(uint32_t dx, uint32_t dy, uint32_t wave_cells) {
    return seg_cells(dx, dy) && !seg_wave(dx, dy, wave_cells) ? 3ull * (dy + 1) : 0;
}

// 5a. per final chain: stretches, traceback bytes, column operations
__global__ void k_seg_count(const Anchors an, const Chains1 c, const Final fin,
                            const uint64_t *foff, uint32_t nr, const uint32_t *nbnd, uint64_t nf,
                            uint32_t wave_cells, uint32_t *nseg, uint64_t *ncell, uint64_t *nops,
                            uint64_t *nrow) {
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nf) return;
    uint32_t r, e;
    final_of(foff, nr, g, nbnd, r, e);
    uint32_t ns = 0, px = 0, py = 0;
    uint64_t cells = 0, ops = 0, rows = 0;
    bool first = true;
    walk_anchors(c, fin, e, [&](uint32_t a) {
        if (!first) {
            uint32_t o = 0, dx = 0, dy = 0;
            link_trim(px, py, an.x[a], an.y[a], an.len[a], o, dx, dy);
            ns++;
            cells += seg_tb_bytes(dx, dy);
            ops += (uint64_t)dx + dy;
            rows += seg_rows(dx, dy, wave_cells);
        }
        first = false;
        px = an.x[a] + an.len[a];
        py = an.y[a] + an.len[a];
    });
    nseg[g] = ns;
    ncell[g] = cells;
    nops[g] = ops;
    nrow[g] = rows;
}

__global__ void k_seg_emit(const Anchors an, const Chains1 c, const Final fin,
                           const uint64_t *foff, uint32_t nr, const uint32_t *nbnd, uint64_t nf,
                           const uint64_t *soff, const uint64_t *coff, const uint64_t *ooff,
                           const uint64_t *roff, uint32_t wave_cells, Seg *seg,
                           uint32_t *fanchor) {
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nf) return;
    uint32_t r, e;
    final_of(foff, nr, g, nbnd, r, e);
    uint64_t s = soff[g], cells = coff[g], ops = ooff[g], rows = roff[g];
    uint32_t *const first3 = fanchor + 3 * g;  // the chain's first anchor: x, y, length
    uint32_t px = 0, py = 0;
    bool first = true;
    walk_anchors(c, fin, e, [&](uint32_t a) {
        if (!first) {
            uint32_t o = 0;
            Seg x;
            x.chain = (uint32_t)g;
            x.region = r;
            x.qx = px;
            x.ty = py;
            link_trim(px, py, an.x[a], an.y[a], an.len[a], o, x.dx, x.dy);
            x.keep = an.len[a] - o;
            x._pad = 0;
            x.cells = cells;
            x.ops = ops;
            x.rows = rows;
            seg[s++] = x;
            cells += seg_tb_bytes(x.dx, x.dy);
            ops += (uint64_t)x.dx + x.dy;
            rows += seg_rows(x.dx, x.dy, wave_cells);
        } else {  // the chain's first anchor, kept whole
            first3[0] = an.x[a];
            first3[1] = an.y[a];
            first3[2] = an.len[a];
        }
        first = false;
        px = an.x[a] + an.len[a];
        py = an.y[a] + an.len[a];
    });
}

// States of the recurrence, the higher preferred among equal scores: in the
// table (M), in a gap of the target (I), in a gap of the query (D).
enum : uint32_t { ST_D = 0, ST_I = 1, ST_M = 2 };

// Traceback byte of a cell (i, j): bits 0-1 the best state before a
// diagonal step, 2-3 the source of the query-gap state, 4-5 of the
// target-gap state, and TB_EQ when query base i - 1 equals target base j - 1
// (neither an N), so that the traceback reads no bases.
constexpr uint8_t TB_EQ = 64;

// Scores are held as 4 * score + state, so that one maximum of three picks the
// best score, settles ties (M, then I, then D) and says which state it was.
// Cells outside the table, and states that cannot be reached, hold values near
// NEG: they stay far below every reachable score (a step moves a value by 24
// at most and a stretch has fewer than 2^21 steps, so they stay within
// 5.1e7 of NEG = -4e8, and reachable values above -5.1e7), so they never win
// against a reachable state and need no test of their own; the traceback
// never enters them.
constexpr int NEG = -400000000;
__device__ __forceinline__ int max3(int a, int b, int c) { return max(max(a, b), c); }

// One cell of the three-state recurrence (match 2, mismatch -4, a gap of L
// bases -(4 + 2 L)) from its diagonal (p*), upper (u*) and left (l*)
// neighbours: M, I, D and the traceback byte.
__device__ __forceinline__ uint32_t cell(int pm, int pi, int pd, int um, int ui, int ud, int lm,
                                         int li, int ld, bool eq, int &m, int &ii, int &dd) {
    constexpr int OPEN = -4 * 6, EXT = -4 * 2, MA = 4 * 2, MI = -4 * 4;
    const int b = max3(pm, pi, pd);
    m = (b | 3) + (eq ? MA - 1 : MI - 1);  // 4 * score + ST_M
    const int x = max3(um + OPEN, ui + EXT, ud + OPEN);
    ii = (x | 3) - 2;                      // + ST_I
    const int y = max3(lm + OPEN, li + OPEN, ld + EXT);
    dd = y & ~3;                           // + ST_D
    return ((uint32_t)b & 3u) | (((uint32_t)x & 3u) << 2) | (((uint32_t)y & 3u) << 4) |
           (eq ? TB_EQ : 0);
}

// The traceback of a filled stretch (table rows P bytes apart) from its end
// state st: column operations written to out in order; returns their number.
__device__ uint32_t trace_back(const Seg &S, const uint8_t *T, uint32_t P, uint32_t st,
                               uint8_t *out) {
    uint32_t i = S.dx, j = S.dy, n = 0;
    while (i > 0 || j > 0) {
        const uint8_t code = T[(uint64_t)i * P + j];
        if (st == ST_M) {
            out[n++] = (code & TB_EQ) ? OP_EQ : OP_X;
            st = code & 3;
            i--;
            j--;
        } else if (st == ST_I) {
            out[n++] = OP_I;
            st = (code >> 2) & 3;
            i--;
        } else {
            out[n++] = OP_D;
            st = (code >> 4) & 3;
            j--;
        }
    }
    // columns were written end first: reverse them
    for (uint32_t a = 0, b = n; a + 1 < b; a++, b--) {
        const uint8_t x = out[a];
        out[a] = out[b - 1];
        out[b - 1] = x;
    }
    return n;
}

// The stretches by the aligner that takes them (a stable sort on the class:
// the thread aligner's first, in chain order, whose neighbours share cache
// lines; then the wave aligner's, those with the most lines per lane first, as
// they take longest).  count: the thread aligner's.  (Ordering the thread
// aligner's stretches by size, for alike work per wave, was slower: it
// scatters the lanes' memory.)
__global__ void k_seg_order(const Seg *seg, uint64_t ns, uint32_t wave_cells, uint32_t *key,
                            uint32_t *val, unsigned long long *count) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool thread = false;
    if (t < ns) {
        const Seg S = seg[t];
        thread = !seg_wave(S.dx, S.dy, wave_cells);
        const uint32_t side = min(S.dx, S.dy);
        key[t] = thread ? 0u : side >= 512 ? 1u : side >= 256 ? 2u : side >= 64 ? 3u : 4u;
        val[t] = (uint32_t)t;
    }
    const uint64_t b = __ballot(thread);  // one atomic per wave
    if (b && (threadIdx.x % 64) == (uint32_t)__builtin_ctzll(b))
        atomicAdd(count, (unsigned long long)__popcll(b));
}

// 5b. one thread per stretch: the three-state affine recurrence (match 2,
// mismatch -4, a gap of L bases -(4 + 2 L)) over two rolling rows, one
// traceback byte per cell (bits 0-1: best state before a diagonal step,
// bits 2-3: source of the query-gap state, bits 4-5: of the target-gap
// state; ties to M, then I, then D), then the columns written backwards
// (op codes, one byte each, dx + dy of them at most).
__global__ void k_align_segs(const IndexView ix, const ARegion *reg, const Seg *seg,
                             const uint32_t *order, uint64_t ns, uint8_t *tb, int *rows,
                             uint8_t *cols, uint32_t *ncol) {
    const uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= ns) return;
    const uint32_t t = order[u];  // the stretch (k_seg_order's thread-aligner part)
    const Seg S = seg[t];
    const uint32_t dx = S.dx, dy = S.dy;
    const ARegion R = reg[S.region];
    uint8_t *out = cols + S.ops;
    if (!seg_cells(dx, dy)) {  // the diagonal stand-in
        const uint32_t m = dx < dy ? dx : dy;
        uint32_t n = 0;
        for (uint32_t i0 = 0; i0 < m; i0 += 16) {  // 16 base pairs read before any op is written
            uint8_t v[16];
#pragma unroll
            for (uint32_t q = 0; q < 16; q++) {
                const uint32_t i = i0 + q;
                const uint32_t a = i < m ? base_at(ix, R.q0 + S.qx + i) : 4u;
                const uint32_t b = i < m ? t_base(ix, R, S.ty + i) : 4u;
                v[q] = (a < 4 && a == b) ? OP_EQ : OP_X;
            }
#pragma unroll
            for (uint32_t q = 0; q < 16; q++)
                if (i0 + q < m) out[n++] = v[q];
        }
        for (uint32_t i = m; i < dx; i++) out[n++] = OP_I;
        for (uint32_t j = m; j < dy; j++) out[n++] = OP_D;
        ncol[t] = n;
        return;
    }
    const uint32_t W = dy + 1, P = tb_pitch(dy);
    uint8_t *T = tb + S.cells;
    int *Mr = rows + S.rows, *Ir = Mr + W, *Dr = Ir + W;  // row i - 1, then row i in place
    constexpr uint32_t CH = 8;  // cells whose loads are issued before any of them is written,
                                // and whose traceback bytes go out in one 8-byte store
    for (uint32_t i = 0; i <= dx; i++) {
        const uint32_t qa = i ? base_at(ix, R.q0 + S.qx + i - 1) : 4u;
        int pm = NEG, pi = NEG, pd = NEG;  // row i - 1, column j - 1
        int lm = NEG, li = NEG, ld = NEG;  // row i, column j - 1
        for (uint32_t j0 = 0; j0 <= dy; j0 += CH) {
            int um[CH], ui[CH], ud[CH];  // row i - 1, column j (i > 0)
            uint32_t tbv[CH];            // target base j - 1 (j > 0)
#pragma unroll
            for (uint32_t q = 0; q < CH; q++) {
                const uint32_t j = j0 + q;
                const bool in = j <= dy;
                um[q] = in && i ? Mr[j] : NEG;
                ui[q] = in && i ? Ir[j] : NEG;
                ud[q] = in && i ? Dr[j] : NEG;
                tbv[q] = in && i && j ? t_base(ix, R, S.ty + j - 1) : 4u;
            }
            uint64_t codes = 0;  // the chunk's traceback bytes (0 past the row)
#pragma unroll
            for (uint32_t q = 0; q < CH; q++) {
                const uint32_t j = j0 + q;
                if (j > dy) break;
                int m, ii, dd;
                const uint32_t code = cell(pm, pi, pd, um[q], ui[q], ud[q], lm, li, ld,
                                          qa < 4 && qa == tbv[q], m, ii, dd);
                if (i == 0 && j == 0) m = ST_M;
                pm = um[q];
                pi = ui[q];
                pd = ud[q];
                lm = m;
                li = ii;
                ld = dd;
                Mr[j] = m;
                Ir[j] = ii;
                Dr[j] = dd;
                codes |= (uint64_t)code << (8 * q);
            }
            *reinterpret_cast<uint64_t *>(T + (uint64_t)i * P + j0) = codes;
        }
    }
    const uint32_t st = (uint32_t)max3(Mr[dy], Ir[dy], Dr[dy]) & 3u;  // end state
    ncol[t] = trace_back(S, T, P, st, out);
}

// v of the lane before (lane 0: `first`).
__device__ __forceinline__ int lane_before(int v, int first) {
    return __builtin_amdgcn_update_dpp(first, v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}

// The table of one stretch, filled by a wave (k_align_wave): a lane holds SW
// lines of the shorter side (na + 1 lines in all; rows when ROWS, else
// columns) and walks the longer one (positions 0..nb), position s - lane at
// step s.  T: line a's traceback bytes at T + a * P, eight to a store.
// Returns the end state.
template <uint32_t SW, bool ROWS>
__device__ __forceinline__ uint32_t fill_wave(const IndexView &ix, const ARegion &R, const Seg &S,
                                              uint32_t na, uint32_t nb, uint8_t *T, uint32_t P) {
    const uint32_t lane = threadIdx.x, a0 = lane * SW;
    // base d - 1 of the lanes' side and of the walked side
    const auto line_base = [&](uint32_t d) {
        return ROWS ? base_at(ix, R.q0 + S.qx + d - 1) : t_base(ix, R, S.ty + d - 1);
    };
    const auto walk_base = [&](uint32_t d) {
        return d == 0 || d > nb ? 4u
               : ROWS           ? t_base(ix, R, S.ty + d - 1)
                                : base_at(ix, R.q0 + S.qx + d - 1);
    };
    uint32_t lb[SW];                 // 5 where nothing matches: no walked base is 5
    int M[SW], I[SW], D[SW];         // position b - 1 of each line, then b in place
    uint32_t lo[SW], hi[SW];         // each line's last eight traceback bytes
#pragma unroll
    for (uint32_t k = 0; k < SW; k++) {
        const uint32_t a = a0 + k;
        lb[k] = a >= 1 && a <= na ? line_base(a) : 5u;
        if (lb[k] == 4) lb[k] = 5;
        M[k] = I[k] = D[k] = NEG;
        lo[k] = hi[k] = 0;
    }
    // the last line of the lane at its last position, and (position b - 1, the
    // line before the lane's first), which for cell (0, 0) stands for a
    // mismatch away from score 0
    int oM = NEG, oI = NEG, oD = NEG;
    int gM = lane == 0 ? 4 * 4 + (int)ST_M : NEG, gI = NEG, gD = NEG;
    uint32_t wb = 4, ahead = walk_base(lane);
    const uint32_t steps = nb + 1 + na / SW;
    for (uint32_t s0 = 0; s0 < steps; s0 += 64) {
        const uint32_t now = ahead;  // lane l: walked base of position s0 + l
        ahead = walk_base(s0 + 64 + lane);
        const uint32_t su = min(64u, steps - s0);
        for (uint32_t u = 0; u < su; u++) {
            const uint32_t b = s0 + u - lane;  // wraps below 0
            wb = (uint32_t)lane_before((int)wb, __builtin_amdgcn_readlane((int)now, (int)u));
            const int iM = lane_before(oM, NEG), iI = lane_before(oI, NEG),
                      iD = lane_before(oD, NEG);
            if (b <= nb) {
                int pm = gM, pi = gI, pd = gD;  // position b - 1, the line before
                int cm = iM, ci = iI, cd = iD;  // position b, the line before
#pragma unroll
                for (uint32_t k = 0; k < SW; k++) {
                    const int vm = M[k], vi = I[k], vd = D[k];
                    const uint32_t code =
                        ROWS ? cell(pm, pi, pd, cm, ci, cd, vm, vi, vd, wb == lb[k], M[k], I[k],
                                    D[k])
                             : cell(pm, pi, pd, vm, vi, vd, cm, ci, cd, wb == lb[k], M[k], I[k],
                                    D[k]);
                    lo[k] = __builtin_amdgcn_alignbyte(hi[k], lo[k], 1);
                    hi[k] = __builtin_amdgcn_alignbyte(code, hi[k], 1);
                    pm = vm;
                    pi = vi;
                    pd = vd;
                    cm = M[k];
                    ci = I[k];
                    cd = D[k];
                }
                oM = cm;
                oI = ci;
                oD = cd;
                if ((b & 7) == 7 || b == nb) {
                    const uint32_t sh = 8 * (7 - (b & 7));
                    uint8_t *at = T + (uint64_t)a0 * P + (b & ~7u);
#pragma unroll
                    for (uint32_t k = 0; k < SW; k++, at += P)
                        if (a0 + k <= na)
                            *reinterpret_cast<uint64_t *>(at) =
                                (((uint64_t)hi[k] << 32) | lo[k]) >> sh;
                }
            }
            gM = iM;
            gI = iI;
            gD = iD;
        }
    }
    int end = 0;
#pragma unroll
    for (uint32_t k = 0; k < SW; k++)
        if (a0 + k == na) end = max3(M[k], I[k], D[k]);
    return (uint32_t)__builtin_amdgcn_readlane(end, (int)(na / SW)) & 3u;
}

// The traceback of a table filled by a wave from its end state st: column
// operations to out (room for dx + dy), in order; returns their number.
// Cell (i, j) is at T + i * pi + j * pj.  The lanes look at the next 64 cells
// of a run in one state at once: as the run goes on where the state's source
// is the state itself, the first lane whose cell came from another one ends it.
__device__ uint32_t trace_wave(uint32_t dx, uint32_t dy, const uint8_t *T, uint32_t pi,
                               uint32_t pj, uint32_t st, uint8_t *out) {
    const uint32_t lane = threadIdx.x, room = dx + dy;
    uint32_t i = dx, j = dy, n = 0;
    while (i > 0 || j > 0) {
        const uint32_t most = st == ST_M ? min(i, j) : st == ST_I ? i : j;
        if (most == 0) {  // never so in a filled table; the walk ends in any case
            st = i ? ST_I : ST_D;
            continue;
        }
        const uint32_t ci = i - (st == ST_D ? 0u : lane), cj = j - (st == ST_I ? 0u : lane);
        uint32_t code = 0, src = 0;
        if (lane < most) {
            code = T[(uint64_t)ci * pi + (uint64_t)cj * pj];
            src = (code >> (2 * (ST_M - st))) & 3u;
        }
        const uint64_t stop = __ballot(lane >= most || src != st);
        uint32_t run = stop ? (uint32_t)__builtin_ctzll(stop) + 1 : 64u;
        run = min(run, most);
        if (lane < run)
            out[room - 1 - n - lane] =
                st == ST_M ? ((code & TB_EQ) ? OP_EQ : OP_X) : st == ST_I ? OP_I : OP_D;
        if (st != ST_D) i -= run;
        if (st != ST_I) j -= run;
        n += run;
        st = (uint32_t)__builtin_amdgcn_readlane((int)src, (int)(run - 1));
    }
    // to the front of the room
    __syncthreads();
    if (n < room)
        for (uint32_t a = lane; a - lane < n; a += 64) {
            const uint8_t v = a < n ? out[room - n + a] : (uint8_t)0;
            if (a < n) out[a] = v;
        }
    return n;
}

// 5c. one 64-lane workgroup per large stretch, the same recurrence and tie
// rules as k_align_segs.  A step hands the last line of each lane to the next
// lane (a move within the registers), so a stretch takes one step per position
// of its longer side and one per lane in use; bound by the instructions of its
// cells (about 25 each).  Rows in registers instead of 53 KB of LDS (three
// waves per CU) or, past 4,096 columns, global memory; codes stored by eights;
// and the traceback a run at a time by all lanes instead of a base at a time
// by one: 39.8 -> 4.3 ms for the stretches from 2,048 cells of 50 Mbp's
// regions.
__global__ __launch_bounds__(64) void k_align_wave(const IndexView ix, const ARegion *reg,
                                                   const Seg *seg, const uint32_t *order,
                                                   uint64_t ns, uint8_t *tb, uint8_t *cols,
                                                   uint32_t *ncol) {
    if (blockIdx.x >= ns) return;
    const uint32_t t = order[blockIdx.x];  // the stretch (k_seg_order's wave part)
    const Seg S = seg[t];
    const ARegion R = reg[S.region];
    uint8_t *T = tb + S.cells;
    const uint32_t dx = S.dx, dy = S.dy;
    const auto fill = [&](auto rows) {
        constexpr bool ROWS = decltype(rows)::value;
        const uint32_t na = ROWS ? dx : dy, nb = ROWS ? dy : dx, P = tb_pitch(nb);
        if (na < 64) return fill_wave<1, ROWS>(ix, R, S, na, nb, T, P);
        if (na < 128) return fill_wave<2, ROWS>(ix, R, S, na, nb, T, P);
        if (na < 256) return fill_wave<4, ROWS>(ix, R, S, na, nb, T, P);
        if (na < 512) return fill_wave<8, ROWS>(ix, R, S, na, nb, T, P);
        return fill_wave<WAVE_S, ROWS>(ix, R, S, na, nb, T, P);
    };
    const bool rows = dx <= dy;
    const uint32_t st = rows ? fill(std::true_type()) : fill(std::false_type());
    __syncthreads();  // the table is written
    const uint32_t n = trace_wave(dx, dy, T, rows ? tb_pitch(dy) : 1u, rows ? 1u : tb_pitch(dx),
                                  st, cols + S.ops);
    if (threadIdx.x == 0) ncol[t] = n;
}

// What a final chain's share - the stretch before an anchor and the anchor's
// '=' run - adds to its chain.
struct Share {
    uint32_t runs;  // merged runs, the last always '='; FIRST_EQ: so is the first
    uint32_t match, mism, opens, ts, tv;
};
constexpr uint32_t FIRST_EQ = 1u << 31;

// A final chain's counts.
struct ChainStats {
    uint32_t match, mism, ins, del, opens, ts, tv, nops;
    uint32_t x0, y0, ex, ey;
};

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return v;
}

// One share (n column ops at col, starting at (qi, ti), then `keep` equal bases)
// walked by a lane: calls run(op, len) for its runs in order (equal ops next to
// each other merged) and, when COUNT, adds its columns to c.
template <bool COUNT, class F>
__device__ __forceinline__ void walk_share(const IndexView &ix, const ARegion &R, const uint8_t *col,
                                           uint32_t n, uint32_t qi, uint32_t ti, uint32_t keep,
                                           Share &c, F &&run) {
    uint32_t cur = 0xFFu, len = 0;
    const auto op1 = [&](uint32_t op) {
        if constexpr (COUNT) {
            if (op == OP_EQ) {  // the aligners write it for equal bases only
                c.match++;
                qi++;
                ti++;
            } else if (op == OP_X) {  // unequal bases, or an N on either side
                const uint32_t x = base_at(ix, R.q0 + qi), y = t_base(ix, R, ti);
                c.mism++;
                if (x < 4 && y < 4) {
                    if ((x ^ y) == 2) c.ts++; else c.tv++;
                }
                qi++;
                ti++;
            } else {
                if (cur != op) c.opens++;
                if (op == OP_I) qi++; else ti++;
            }
        }
        if (op == cur) {
            len++;
        } else {
            if (len) run(cur, len);
            cur = op;
            len = 1;
        }
    };
    // 16 column ops at a time, all loaded before any is used
    for (uint32_t u0 = 0; u0 < n; u0 += 16) {
        uint8_t cb[16];
#pragma unroll
        for (uint32_t q = 0; q < 16; q++) cb[q] = u0 + q < n ? col[u0 + q] : 0;
#pragma unroll
        for (uint32_t q = 0; q < 16; q++)
            if (u0 + q < n) op1(cb[q]);
    }
    if (cur == OP_EQ) {
        len += keep;
    } else {
        if (len) run(cur, len);
        cur = OP_EQ;
        len = keep;
    }
    if constexpr (COUNT) c.match += keep;
    run(cur, len);
}

// The same by a whole wave, 64 columns at a time: chunk(op, starts, valid) for
// each, with every lane's op, the lanes at which a run starts and the lanes in
// use.  Returns the last op (0xFF for none).
template <class F>
__device__ __forceinline__ uint32_t walk_wave(const uint8_t *col, uint32_t n, F &&chunk) {
    const uint32_t lane = threadIdx.x % 64;
    uint32_t last = 0xFFu;
    for (uint32_t u0 = 0; u0 < n; u0 += 64) {
        const uint32_t m = min(64u, n - u0);
        const uint32_t op = lane < m ? (uint32_t)col[u0 + lane] : 0u;
        const uint32_t prev = (uint32_t)lane_before((int)op, (int)last);
        chunk(op, __ballot(lane < m && op != prev), m == 64 ? ~0ull : (1ull << m) - 1);
        last = lane_u32(op, m - 1);
    }
    return last;
}

// Shares of at least this many columns are walked by their wave together: a
// lane alone takes over 1 us per 16 columns, and its wave waits for it.
constexpr uint32_t SHARE_WAVE = 96;

// 6a. the shares, one lane each (long ones by the wave), and how many more runs
// than its predecessors' a share brings to its chain's CIGAR: a first run of
// equal bases lengthens the run before it.
// (Before, one wave walked a whole chain, 64 shares at a time, merging them one
// by one, once for the counts and once for the CIGAR: 16.6 ms for 50 Mbp's
// regions, where the four kernels now take 3.4.)
__global__ __launch_bounds__(256) void k_shares(const IndexView ix, const ARegion *reg,
                                                const Seg *seg, uint64_t ns, const uint8_t *cols,
                                                const uint32_t *ncol, Share *share,
                                                uint32_t *more) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t lane = threadIdx.x % 64;
    Seg S{};
    uint32_t n = 0;
    if (t < ns) {
        S = seg[t];
        n = ncol[t];
    }
    Share c{};
    if (t < ns && n < SHARE_WAVE) {
        uint32_t first = 0xFFu;
        walk_share<true>(ix, reg[S.region], cols + S.ops, n, S.qx, S.ty, S.keep, c,
                         [&](uint32_t op, uint32_t) {
                             if (!c.runs) first = op;
                             c.runs++;
                         });
        if (first == OP_EQ) c.runs |= FIRST_EQ;
    }
    for (uint64_t todo = __ballot(n >= SHARE_WAVE); todo; todo &= todo - 1) {
        const uint32_t l = (uint32_t)__builtin_ctzll(todo);
        const Seg W = seg[t - lane + l];
        const ARegion R = reg[W.region];
        const uint8_t *col = cols + W.ops;
        uint32_t qi = W.qx, ti = W.ty;
        Share w{};
        const uint32_t last = walk_wave(col, lane_u32(n, l), [&](uint32_t op, uint64_t starts,
                                                                uint64_t valid) {
            const uint64_t eq = __ballot(op == OP_EQ), x = __ballot(op == OP_X);
            const uint64_t ins = __ballot(op == OP_I), del = __ballot(op == OP_D);
            const uint64_t below = (1ull << lane) - 1;
            bool ts = false, tv = false;
            if (op == OP_X) {
                const uint32_t a =
                    base_at(ix, R.q0 + qi + (uint32_t)__popcll(valid & ~del & below));
                const uint32_t b = t_base(ix, R, ti + (uint32_t)__popcll(valid & ~ins & below));
                if (a < 4 && b < 4) {
                    ts = (a ^ b) == 2;
                    tv = !ts;
                }
            }
            w.runs += (uint32_t)__popcll(starts);
            w.match += (uint32_t)__popcll(eq);
            w.mism += (uint32_t)__popcll(x);
            w.opens += (uint32_t)__popcll(starts & (ins | del));
            w.ts += (uint32_t)__popcll(__ballot(ts));
            w.tv += (uint32_t)__popcll(__ballot(tv));
            qi += (uint32_t)__popcll(valid & ~del);
            ti += (uint32_t)__popcll(valid & ~ins);
        });
        w.match += W.keep;
        if (last != OP_EQ) w.runs++;
        if (col[0] == OP_EQ) w.runs |= FIRST_EQ;
        if (lane == l) c = w;
    }
    if (t >= ns) return;
    share[t] = c;
    more[t] = (c.runs & ~FIRST_EQ) - (c.runs & FIRST_EQ ? 1u : 0u);
}

// 6b. the chains' counts from their shares and which are reported.  Most
// chains have a share or two: a lane each; the wave goes through the long ones
// together.
__global__ __launch_bounds__(256) void k_chain_counts(const uint64_t *soff, uint64_t nf,
                                                      const Seg *seg, const Share *share,
                                                      const uint64_t *moff,
                                                      const uint32_t *fanchor, uint32_t min_len,
                                                      double delta, ChainStats *stats,
                                                      uint32_t *nops_out, uint32_t *pass_out) {
    constexpr uint64_t LONG = 8;
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t lane = threadIdx.x % 64;
    const uint64_t s0 = g < nf ? soff[g] : 0, s1 = g < nf ? soff[g + 1] : 0;
    const auto add = [&](ChainStats &st, uint64_t s) {
        const Share c = share[s];
        const uint32_t dx = seg[s].dx, dy = seg[s].dy, keep = seg[s].keep;
        const uint32_t both = c.match - keep + c.mism;  // columns of the stretch on both sides
        st.match += c.match;
        st.mism += c.mism;
        st.ins += dx - both;
        st.del += dy - both;
        st.opens += c.opens;
        st.ts += c.ts;
        st.tv += c.tv;
    };
    ChainStats st = {};
    if (s1 - s0 <= LONG)
        for (uint64_t s = s0; s < s1; s++) add(st, s);
    for (uint64_t todo = __ballot(s1 - s0 > LONG); todo; todo &= todo - 1) {
        const uint32_t l = (uint32_t)__builtin_ctzll(todo);
        const uint64_t a = soff[g - lane + l], b = soff[g - lane + l + 1];
        ChainStats w = {};
#pragma unroll 2
        for (uint64_t s = a + lane; s < b; s += 64) add(w, s);
        w.match = wave_sum_u32(w.match);
        w.mism = wave_sum_u32(w.mism);
        w.ins = wave_sum_u32(w.ins);
        w.del = wave_sum_u32(w.del);
        w.opens = wave_sum_u32(w.opens);
        w.ts = wave_sum_u32(w.ts);
        w.tv = wave_sum_u32(w.tv);
        if (lane == l) st = w;
    }
    if (g >= nf) return;
    const uint32_t l0 = fanchor[3 * g + 2];
    st.match += l0;
    st.nops = 1 + (uint32_t)(moff[s1] - moff[s0]);
    st.x0 = fanchor[3 * g];
    st.y0 = fanchor[3 * g + 1];
    st.ex = st.x0 + l0;
    st.ey = st.y0 + l0;
    if (s1 > s0) {  // the end of the last stretch's anchor
        const Seg S = seg[s1 - 1];
        st.ex = S.qx + S.dx + S.keep;
        st.ey = S.ty + S.dy + S.keep;
    }
    stats[g] = st;
    const uint32_t aln = st.match + st.mism + st.ins + st.del;
    const bool ok = aln >= min_len && (double)(st.mism + st.opens) <= delta * (double)aln;
    pass_out[g] = ok ? 1u : 0u;
    nops_out[g] = ok ? st.nops : 0u;
}

// 6c. the CIGARs of the reported chains, share by share (cigar zeroed
// beforehand, the chain's first anchor's run added by k_records): run i of a
// share goes to the chain's place for it; a length that grows from several
// places is added up.
__global__ __launch_bounds__(256) void k_cigars(const IndexView ix, const ARegion *reg,
                                                const Seg *seg, uint64_t ns, const uint8_t *cols,
                                                const uint32_t *ncol, const Share *share,
                                                const uint64_t *soff, const uint64_t *moff,
                                                const uint32_t *pass, const uint64_t *op_off,
                                                uint32_t *cigar) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t lane = threadIdx.x % 64;
    Seg S{};
    uint32_t n = 0;
    bool on = false, merged = false;  // merged: the first run lengthens the one before
    uint64_t at = 0;                  // where the share's run 0 goes
    if (t < ns) {
        S = seg[t];
        on = pass[S.chain] != 0;
        if (on) {
            n = ncol[t];
            merged = (share[t].runs & FIRST_EQ) != 0;
            at = op_off[S.chain] + 1 + (moff[t] - moff[soff[S.chain]]) - (merged ? 1u : 0u);
        }
    }
    if (on && n < SHARE_WAVE) {
        const uint32_t runs = share[t].runs & ~FIRST_EQ;
        uint32_t i = 0;
        Share unused;
        walk_share<false>(ix, reg[S.region], cols + S.ops, n, S.qx, S.ty, S.keep, unused,
                          [&](uint32_t op, uint32_t len) {
                              const uint32_t v = (len << 4) | (i == 0 && merged ? 0u : op);
                              if (i == 0 || i + 1 == runs)
                                  atomicAdd(cigar + at + i, v);
                              else
                                  cigar[at + i] = v;
                              i++;
                          });
    }
    for (uint64_t todo = __ballot(on && n >= SHARE_WAVE); todo; todo &= todo - 1) {
        const uint32_t l = (uint32_t)__builtin_ctzll(todo);
        const Seg W = seg[t - lane + l];
        const bool wm = lane_u32(merged, l) != 0;
        uint32_t *const cig =
            cigar + (((uint64_t)lane_u32((uint32_t)(at >> 32), l) << 32) | lane_u32((uint32_t)at, l));
        uint32_t runs = 0;  // runs started so far
        const uint32_t last = walk_wave(cols + W.ops, lane_u32(n, l), [&](uint32_t op, uint64_t starts,
                                                                          uint64_t valid) {
            // the columns that go on the run before
            const uint32_t m = (uint32_t)__popcll(valid);
            const uint32_t on0 = starts ? (uint32_t)__builtin_ctzll(starts) : m;
            if (lane == 0 && on0) atomicAdd(cig + runs - 1, on0 << 4);
            if ((starts >> lane) & 1) {
                const uint64_t later = lane == 63 ? 0ull : starts >> (lane + 1);
                const uint32_t len = later ? (uint32_t)__builtin_ctzll(later) + 1 : m - lane;
                const uint32_t i = runs + (uint32_t)__popcll(starts & ((1ull << lane) - 1));
                const uint32_t v = (len << 4) | (i == 0 && wm ? 0u : op);
                if (later && i)
                    cig[i] = v;
                else
                    atomicAdd(cig + i, v);
            }
            runs += (uint32_t)__popcll(starts);
        });
        if (lane == 0) {
            if (last == OP_EQ)
                atomicAdd(cig + runs - 1, W.keep << 4);
            else
                atomicAdd(cig + runs, (W.keep << 4) | OP_EQ);
        }
    }
}

// 6d. the records of the reported chains
__global__ void k_records(const IndexView ix, const ARegion *reg, const uint64_t *foff, uint32_t nr,
                          uint64_t nf, const ChainStats *stats, const uint32_t *fanchor,
                          const uint32_t *pass, const uint64_t *wr_off, const uint64_t *op_off,
                          sdf_sd *sd, uint32_t *cigar) {
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nf || !pass[g]) return;
    const uint32_t r = region_of(foff, nr, g);
    const ARegion R = reg[r];
    const ChainStats st = stats[g];
    atomicAdd(cigar + op_off[g], (fanchor[3 * g + 2] << 4) | OP_EQ);
    sdf_sd d;
    d.region = r;
    d.strand = R.o;
    d.q_seq = R.qseq;
    d.t_seq = R.tseq;
    d._pad = 0;
    const uint64_t qo = ix.off[R.qseq], to = ix.off[R.tseq];
    d.q_begin = R.q0 + st.x0 - qo;
    d.q_end = R.q0 + st.ex - qo;
    if (R.o == 0) {
        d.t_begin = R.t0 + st.y0 - to;
        d.t_end = R.t0 + st.ey - to;
    } else {
        d.t_begin = R.t1 - st.ey - to;
        d.t_end = R.t1 - st.y0 - to;
    }
    d.aln_len = st.match + st.mism + st.ins + st.del;
    d.matches = st.match;
    d.mismatches = st.mism;
    d.ins = st.ins;
    d.dels = st.del;
    d.gap_opens = st.opens;
    d.transitions = st.ts;
    d.transversions = st.tv;
    const double al = (double)(st.match + st.mism);
    const double P = al > 0 ? st.ts / al : 0.0, Q = al > 0 ? st.tv / al : 0.0;
    const double a1 = 1.0 - 2.0 * P - Q, a2 = 1.0 - 2.0 * Q;
    d.k2p = (al > 0 && a1 > 0 && a2 > 0) ? -0.5 * log(a1) - 0.25 * log(a2) : -1.0;
    const double p = al > 0 ? st.mism / al : 0.0, a3 = 1.0 - 4.0 * p / 3.0;
    d.jc = (al > 0 && a3 > 0) ? -0.75 * log(a3) : -1.0;
    d.cigar_off = op_off[g];
    d.cigar_len = st.nops;
    sd[wr_off[g]] = d;
}

__global__ void k_u32_to_u64(const uint32_t *a, uint64_t n, uint64_t *b) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) b[t] = a[t];
}

unsigned nb(uint64_t n, unsigned t = 256) { return (unsigned)std::max<uint64_t>(1, (n + t - 1) / t); }

// launch(first, blocks) for n workgroups of `threads` threads, in parts of fewer
// than the 2^32 threads a launch may have.
template <class F>
void by_parts(uint64_t n, uint64_t threads, F &&launch) {
    const uint64_t most = ((1ull << 32) - 1) / threads;
    for (uint64_t first = 0; first < n; first += most) {
        launch(first, (unsigned)std::min(most, n - first));
        SDF_HIP(hipGetLastError());
    }
}

// Chains taken out by score (see k_own_init): the members of all chains, chain
// after chain (member), the chains' heads (flag), the chains before each
// position (pre, na + 1) and each chain's first position (first).  order, list:
// the entries in extraction and in start order, the first *nlive of them (all
// na without); most: the most entries of a region.
void take_chains(const uint32_t *order, const uint32_t *list, const uint32_t *pred, uint64_t na,
                 const uint32_t *nlive, uint32_t most, uint32_t *member, uint32_t *flag,
                 uint32_t *pre, uint64_t *first, hipStream_t st) {
    DevBuf<uint32_t> key(na);
    if (na <= OWN_SMALL) {
        k_own_small<<<1, 1024, 0, st>>>(order, list, (uint32_t)na, nlive, pred, most, key.p, member);
        SDF_HIP(hipGetLastError());
    } else {
        DevBuf<uint32_t> own(na), ja(na), jb(na);
        k_own_init<<<nb(na), 256, 0, st>>>(order, na, nlive, pred, own.p, ja.p);
        SDF_HIP(hipGetLastError());
        uint32_t *jin = ja.p, *jout = jb.p;
        for (uint64_t reach = 1; reach < most; reach *= 2) {
            k_own_double<<<nb(na), 256, 0, st>>>(list, na, nlive, own.p, jin, jout);
            SDF_HIP(hipGetLastError());
            std::swap(jin, jout);
        }
        k_own_keys<<<nb(na), 256, 0, st>>>(list, na, nlive, own.p, key.p, member);
        SDF_HIP(hipGetLastError());
    }
    int bits = 1;
    while ((1ull << bits) <= na) bits++;
    radix_sort_u32(key.p, member, na, bits, st);
    k_own_heads<<<nb(na), 256, 0, st>>>(key.p, na, nlive, flag);
    SDF_HIP(hipGetLastError());
    scan_u32(flag, pre, na, st);
    k_run_first<<<nb(na), 256, 0, st>>>(flag, pre, na, first);
    SDF_HIP(hipGetLastError());
}

template <class T>
T read1(const T *d, hipStream_t st) {
    T h{};
    Readback rb(st);
    rb.add(&h, d, sizeof(T));
    rb.wait();
    return h;
}

}  // namespace

void sd_align(const IndexView &ix, const uint64_t *h_off, const sdf_region *regions, uint64_t n,
              uint32_t k, uint32_t min_len, double delta, SdResult &res, hipStream_t st) {
    res.nsd = 0;
    res.nops = 0;
    if (n == 0) return;
    // regions with global sides; per-region offsets of T' and Q positions
    std::vector<ARegion> hr(n);
    std::vector<uint64_t> hto(n + 1), hqo(n + 1);
    hto[0] = hqo[0] = 0;
    for (uint64_t r = 0; r < n; r++) {
        const sdf_region &x = regions[r];
        ARegion a;
        a.q0 = h_off[x.q_seq] + x.q_begin;
        a.q1 = h_off[x.q_seq] + x.q_end;
        a.t0 = h_off[x.t_seq] + x.t_begin;
        a.t1 = h_off[x.t_seq] + x.t_end;
        a.o = x.strand;
        a.qseq = x.q_seq;
        a.tseq = x.t_seq;
        a._pad = 0;
        hr[r] = a;
        hto[r + 1] = hto[r] + (a.t1 - a.t0);
        hqo[r + 1] = hqo[r] + (a.q1 - a.q0);
    }
    const uint32_t nr = (uint32_t)n;
    DevBuf<ARegion> dreg(n);
    DevBuf<uint64_t> qoff(n + 1);
    SDF_HIP(hipMemcpyAsync(dreg.p, hr.data(), n * sizeof(ARegion), hipMemcpyHostToDevice, st));
    SDF_HIP(hipMemcpyAsync(qoff.p, hqo.data(), (n + 1) * 8, hipMemcpyHostToDevice, st));
    // the regions by falling size: one workgroup or wave takes a region in the
    // chaining kernels, and the largest take longest, so they start first
    std::vector<uint32_t> hl(n);
    for (uint64_t r = 0; r < n; r++) hl[r] = (uint32_t)r;
    std::stable_sort(hl.begin(), hl.end(), [&](uint32_t a, uint32_t b) {
        return (hto[a + 1] - hto[a]) + (hqo[a + 1] - hqo[a]) > (hto[b + 1] - hto[b]) + (hqo[b + 1] - hqo[b]);
    });
    DevBuf<uint32_t> large(n);
    SDF_HIP(hipMemcpyAsync(large.p, hl.data(), n * 4, hipMemcpyHostToDevice, st));
    const uint64_t QT = hqo[n];
    // key bits of a region number: every region number stays below 2^rbits - 1, so
    // no key of a region has all of its bits set like the sentinel ~0
    int rbits = 1;
    while ((1ull << rbits) <= (uint64_t)n) rbits++;
    std::optional<Range> stage;
    stage.emplace("sdf final SDs: seeds");
    // 1. matches per query position, their offsets, the matches sorted
    // Query positions per workgroup: every part of a large side builds the target's
    // buckets anew, so parts are as long as leave some 2,048 workgroups (50 Mbp:
    // 10.1, 8.9, 9.0 ms for the counts with at most 32,768, 65,536, 131,072).
    const uint64_t xpart =
        std::clamp<uint64_t>(QT / 2048 / SEED_XLO * SEED_XLO, SEED_XLO, SEED_XHI);
    std::vector<SeedWork> hw;
    for (const uint32_t r : hl)
        for (uint64_t nq = hqo[r + 1] - hqo[r], x = 0; x < nq; x += xpart)
            hw.push_back(SeedWork{r, (uint32_t)x, (uint32_t)std::min(nq, x + xpart)});
    DevBuf<SeedWork> work(hw.size() + 1);
    DevBuf<uint32_t> qcnt(QT + 1);
    DevBuf<uint64_t> moff(QT + 1);
    if (QT) {
        SDF_HIP(hipMemcpyAsync(work.p, hw.data(), hw.size() * sizeof(SeedWork),
                               hipMemcpyHostToDevice, st));
        by_parts(hw.size(), SEED_THREADS, [&](uint64_t first, unsigned blocks) {
            k_seeds<false><<<blocks, SEED_THREADS, 0, st>>>(ix, dreg.p, work.p + first, qoff.p, k,
                                                            qcnt.p, nullptr, nullptr);
        });
    }
    scan_u32_to_u64(qcnt.p, moff.p, QT, st);
    const uint64_t M = read1(moff.p + QT, st);
    DevBuf<uint64_t> mkey(M + 1);
    if (M) {
        by_parts(hw.size(), SEED_THREADS, [&](uint64_t first, unsigned blocks) {
            k_seeds<true><<<blocks, SEED_THREADS, 0, st>>>(ix, dreg.p, work.p + first, qoff.p, k,
                                                           qcnt.p, moff.p, mkey.p);
        });
        // (region, diagonal): the matches are made in x order within a region
        sort_keys_u64_bits(mkey.p, M, 20, 41 + rbits, st);
    }
    // 2. anchors
    stage.emplace("sdf final SDs: anchors");
    DevBuf<uint32_t> flag(M + 1), fpre(M + 1);
    if (M) {
        k_run_starts<<<nb(M), 256, 0, st>>>(mkey.p, M, flag.p);
        SDF_HIP(hipGetLastError());
    }
    scan_u32(flag.p, fpre.p, M, st);
    const uint64_t A = read1(fpre.p + M, st);
    if (A == 0) return;
    DevBuf<uint32_t> areg(A), ax(A), ay(A), alen(A);
    Anchors an{areg.p, ax.p, ay.p, alen.p};
    DevBuf<uint64_t> rfirst(A);
    k_run_first<<<nb(M), 256, 0, st>>>(flag.p, fpre.p, M, rfirst.p);
    SDF_HIP(hipGetLastError());
    k_anchor_emit<<<nb(A), 256, 0, st>>>(mkey.p, M, rfirst.p, A, k, an);
    SDF_HIP(hipGetLastError());
    mkey.reset();
    rfirst.reset();
    // orders by (region, x, y) and by (region, end x, end y)
    DevBuf<uint64_t> kxy(A), kend(A), kbuf(A);
    DevBuf<uint32_t> byxy(A), byend(A), byscore(A), perm(A);
    k_order_keys<<<nb(A), 256, 0, st>>>(an, A, 0, kxy.p, byxy.p);
    k_order_keys<<<nb(A), 256, 0, st>>>(an, A, 1, kend.p, byend.p);
    SDF_HIP(hipGetLastError());
    radix_sort_u64(kxy.p, byxy.p, A, 42 + rbits, st);
    radix_sort_u64(kend.p, byend.p, A, 42 + rbits, st);
    DevBuf<uint32_t> bnd(n + 1);
    k_region_bounds<<<nb(n + 1), 256, 0, st>>>(kxy.p, A, 42, nr, bnd.p);
    SDF_HIP(hipGetLastError());
    // 3. tier 1
    stage.emplace("sdf final SDs: tier 1");
    const double dM = delta < 0.15 ? delta : 0.15, dG = delta - dM;
    uint32_t G1 = (uint32_t)std::ceil((double)min_len * dG);
    if (G1 < 1) G1 = 1;
    DevBuf<int64_t> s1(A);
    DevBuf<uint32_t> p1(A);
    Tier1 t1{s1.p, p1.p};
    uint32_t most_anchors = 0;  // anchors of the largest region
    {
        DevBuf<uint32_t> elen(A), pos_e(A);
        DevBuf<int64_t> s1e(A);
        k_end_order<<<nb(A), 256, 0, st>>>(an, byend.p, A, elen.p, pos_e.p);
        SDF_HIP(hipGetLastError());
        // LDS block ends for up to T2_BLOCKS blocks of 64 anchors a region (align_lds_blocks)
        DevBuf<uint32_t> most(1);
        fill_u32(most.p, 0u, 1, st);
        k_max_span<<<nb(n), 256, 0, st>>>(bnd.p, nr, most.p);
        SDF_HIP(hipGetLastError());
        most_anchors = read1(most.p, st);
        const uint32_t nblk =
            std::min<uint32_t>(std::min(knob(tuning().align_lds_blocks, T2_BLOCKS), T2_BLOCKS),
                               (most_anchors + 63) / 64);
        k_tier1<<<nr, 64 * T1_WAVES, 4 * nblk, st>>>(kxy.p, byxy.p, an.len, kend.p, byend.p,
                                                     elen.p, pos_e.p, bnd.p, nr, G1, t1, s1e.p,
                                                     nblk, large.p);
        SDF_HIP(hipGetLastError());
    }
    // score order: y first (stable), then (region, score descending, x)
    k_score_keys<<<nb(A), 256, 0, st>>>(an, A, t1, 0, kbuf.p, perm.p, nullptr);
    SDF_HIP(hipGetLastError());
    radix_sort_u64(kbuf.p, perm.p, A, 20, st);
    k_score_keys<<<nb(A), 256, 0, st>>>(an, A, t1, 1, kbuf.p, byscore.p, perm.p);
    SDF_HIP(hipGetLastError());
    radix_sort_u64(kbuf.p, byscore.p, A, 41 + rbits, st);
    DevBuf<uint32_t> mem1(A), cst(A), cend(A), ccount(n), cx(A), cy(A), cex(A), cey(A), cfl(A);
    DevBuf<int64_t> cw(A);
    Chains1 c{mem1.p, cst.p, cend.p, ccount.p, cx.p, cy.p, cex.p, cey.p, cw.p, cfl.p};
    DevBuf<uint32_t> cpre(A + 1);  // chains before each member position
    DevBuf<uint64_t> cfirst(A);    // each chain's first
    take_chains(byscore.p, byxy.p, t1.pred, A, nullptr, most_anchors, c.member, flag.p, cpre.p,
                cfirst.p, st);
    k_chain_count<<<nb(n), 256, 0, st>>>(bnd.p, nr, cpre.p, c.count);
    k_nodes1<<<nb(A), 256, 0, st>>>(an, bnd.p, A, flag.p, cpre.p, cfirst.p, t1.score, c);
    SDF_HIP(hipGetLastError());
    // nodes ordered by (region, x, y)
    DevBuf<uint32_t> rslot(A), nodes(A), nbnd(n + 1);
    k_slot_regions<<<nb(A), 256, 0, st>>>(an, byxy.p, A, rslot.p);
    k_node_keys<<<nb(A), 256, 0, st>>>(bnd.p, rslot.p, A, c, kbuf.p, nodes.p);
    SDF_HIP(hipGetLastError());
    radix_sort_u64(kbuf.p, nodes.p, A, 42 + rbits, st);
    k_region_bounds<<<nb(n + 1), 256, 0, st>>>(kbuf.p, A, 42, nr, nbnd.p);
    SDF_HIP(hipGetLastError());
    // 4. tier 2: nodes by end, scores, extraction order, final chains
    stage.emplace("sdf final SDs: tier 2");
    DevBuf<uint32_t> nodes_e(A), order(A);
    DevBuf<uint64_t> ekey(A);
    DevBuf<int64_t> s2(A);
    DevBuf<uint32_t> p2(A), fmem(A), fst(A), fend(A), fcount(n + 1);
    k_node_keys2<<<nb(A), 256, 0, st>>>(nodes.p, A, nbnd.p + nr, rslot.p, c, s2.p, 0, nullptr,
                                        ekey.p, nodes_e.p);
    SDF_HIP(hipGetLastError());
    radix_sort_u64(ekey.p, nodes_e.p, A, 42 + rbits, st);
    uint32_t most_nodes = 0;  // nodes of the largest region
    {
        DevBuf<uint32_t> pos_e(A), ue(A), p2s(A);
        DevBuf<Node2> node2(A);
        DevBuf<int32_t> s2s(A), s2e(A);
        k_invert<<<nb(A), 256, 0, st>>>(nodes_e.p, A, pos_e.p);
        k_node_starts<<<nb(A), 256, 0, st>>>(nodes.p, A, nbnd.p + nr, pos_e.p, c, node2.p, ue.p);
        SDF_HIP(hipGetLastError());
        // LDS bounds for up to T2_BLOCKS blocks of 64 nodes per region (align_lds_blocks)
        DevBuf<uint32_t> most(1);
        fill_u32(most.p, 0u, 1, st);
        k_max_span<<<nb(n), 256, 0, st>>>(nbnd.p, nr, most.p);
        SDF_HIP(hipGetLastError());
        most_nodes = read1(most.p, st);
        const uint32_t nblk =
            std::min<uint32_t>(std::min(knob(tuning().align_lds_blocks, T2_BLOCKS), T2_BLOCKS),
                               (most_nodes + 63) / 64);
        k_tier2<<<nr, 64 * T2_WAVES, 8 * nblk, st>>>(nbnd.p, nr, node2.p, ekey.p, ue.p, s2s.p,
                                                     s2e.p, p2s.p, nblk, large.p);
        k_node_results<<<nb(A), 256, 0, st>>>(node2.p, A, nbnd.p + nr, s2s.p, p2s.p, s2.p, p2.p);
        SDF_HIP(hipGetLastError());
    }
    k_node_keys2<<<nb(A), 256, 0, st>>>(nodes.p, A, nbnd.p + nr, rslot.p, c, s2.p, 1, nullptr,
                                        kbuf.p, perm.p);
    SDF_HIP(hipGetLastError());
    radix_sort_u64(kbuf.p, perm.p, A, 20, st);
    k_node_keys2<<<nb(A), 256, 0, st>>>(nodes.p, A, nbnd.p + nr, rslot.p, c, s2.p, 2, perm.p,
                                        kbuf.p, order.p);
    SDF_HIP(hipGetLastError());
    radix_sort_u64(kbuf.p, order.p, A, 42 + rbits, st);
    Final fin{fmem.p, fst.p, fend.p, fcount.p};
    take_chains(order.p, nodes.p, p2.p, A, nbnd.p + nr, most_nodes, fin.member, flag.p, cpre.p,
                cfirst.p, st);
    k_chain_count<<<nb(n), 256, 0, st>>>(nbnd.p, nr, cpre.p, fin.count);
    k_finals<<<nb(A), 256, 0, st>>>(rslot.p, nbnd.p, A, nbnd.p + nr, flag.p, cpre.p, cfirst.p, fin);
    SDF_HIP(hipGetLastError());
    DevBuf<uint64_t> foff(n + 1);
    scan_u32_to_u64(fcount.p, foff.p, n, st);
    const uint64_t NF = read1(foff.p + n, st);
    if (NF == 0) return;
    // 5. stretches between anchors, aligned
    stage.emplace("sdf final SDs: alignment");
    DevBuf<uint32_t> nseg(NF + 1);
    DevBuf<uint64_t> ncell(NF + 1), nops(NF + 1), nrow(NF + 1);
    // Stretches a thread takes: a thread needs about 0.25 us per cell whatever
    // else runs, so a call of few stretches waits for its longest; a wave is
    // idle in most lanes on a small one (50 Mbp, all regions: 85.5, 79.4, 75.0,
    // 73.5, 73.2, 73.3, 73.9, 74.9 ms from 4,096, 2,048, 1,024, 512, 256, 128,
    // 64, 1 cells up; 3 Mbp: 4.53, 3.90, 3.42, 3.20, 3.10, 3.05, 3.02, 2.98 ms).
    const uint32_t wave_cells = knob(tuning().align_wave_cells, 1u << 8);
    k_seg_count<<<nb(NF), 256, 0, st>>>(an, c, fin, foff.p, nr, nbnd.p, NF, wave_cells, nseg.p,
                                        ncell.p, nops.p, nrow.p);
    SDF_HIP(hipGetLastError());
    DevBuf<uint64_t> soff(NF + 1), coff(NF + 1), ooff(NF + 1), roff(NF + 1);
    scan_u32_to_u64(nseg.p, soff.p, NF, st);
    scan_u64(ncell.p, coff.p, NF, st);
    scan_u64(nops.p, ooff.p, NF, st);
    scan_u64(nrow.p, roff.p, NF, st);
    uint64_t NS = 0, NC = 0, NO = 0, NRW = 0;
    {
        Readback rb(st);
        rb.add(&NS, soff.p + NF, 8);
        rb.add(&NC, coff.p + NF, 8);
        rb.add(&NO, ooff.p + NF, 8);
        rb.add(&NRW, roff.p + NF, 8);
        rb.wait();
    }
    DevBuf<Seg> seg(NS + 1);
    DevBuf<uint8_t> tb(NC + 1), cols(NO + 1);
    DevBuf<int> rows(NRW + 1);
    DevBuf<uint32_t> ncol(NS + 1);
    DevBuf<uint32_t> fanchor(3 * NF);
    k_seg_emit<<<nb(NF), 256, 0, st>>>(an, c, fin, foff.p, nr, nbnd.p, NF, soff.p, coff.p, ooff.p,
                                       roff.p, wave_cells, seg.p, fanchor.p);
    SDF_HIP(hipGetLastError());
    if (NS) {
        DevBuf<uint32_t> okey(NS), order(NS);
        DevBuf<unsigned long long> tcount(1);
        fill_u32(reinterpret_cast<uint32_t *>(tcount.p), 0u, 2, st);
        k_seg_order<<<nb(NS, 256), 256, 0, st>>>(seg.p, NS, wave_cells, okey.p, order.p, tcount.p);
        SDF_HIP(hipGetLastError());
        radix_sort_u32(okey.p, order.p, NS, 3, st);
        const uint64_t nthread = read1(tcount.p, st);
        if (nthread)
            k_align_segs<<<nb(nthread, 64), 64, 0, st>>>(ix, dreg.p, seg.p, order.p, nthread, tb.p,
                                                        rows.p, cols.p, ncol.p);
        SDF_HIP(hipGetLastError());
        by_parts(NS - nthread, 64, [&](uint64_t first, unsigned blocks) {
            k_align_wave<<<blocks, 64, 0, st>>>(ix, dreg.p, seg.p, order.p + nthread + first, blocks,
                                                tb.p, cols.p, ncol.p);
        });
    }
    // 6. records and CIGAR
    stage.emplace("sdf final SDs: records");
    DevBuf<uint32_t> aops(NF + 1), apass(NF + 1);
    DevBuf<Share> share(NS + 1);
    DevBuf<uint32_t> more(NS + 1);
    DevBuf<uint64_t> mroff(NS + 1);
    DevBuf<ChainStats> stats(NF);
    if (NS) {
        k_shares<<<nb(NS, 256), 256, 0, st>>>(ix, dreg.p, seg.p, NS, cols.p, ncol.p, share.p,
                                              more.p);
        SDF_HIP(hipGetLastError());
    }
    scan_u32_to_u64(more.p, mroff.p, NS, st);
    k_chain_counts<<<nb(NF), 256, 0, st>>>(soff.p, NF, seg.p, share.p, mroff.p, fanchor.p,
                                                min_len, delta, stats.p, aops.p, apass.p);
    SDF_HIP(hipGetLastError());
    DevBuf<uint64_t> woff(NF + 1), opoff(NF + 1);
    scan_u32_to_u64(apass.p, woff.p, NF, st);
    scan_u32_to_u64(aops.p, opoff.p, NF, st);
    uint64_t NSD = 0, NOPS = 0;
    {
        Readback rb(st);
        rb.add(&NSD, woff.p + NF, 8);
        rb.add(&NOPS, opoff.p + NF, 8);
        rb.wait();
    }
    res.sd.alloc(NSD + 1);
    res.cigar.alloc(NOPS + 1);
    if (NSD) {
        fill_u32(res.cigar.p, 0u, NOPS, st);
        if (NS) {
            k_cigars<<<nb(NS, 256), 256, 0, st>>>(ix, dreg.p, seg.p, NS, cols.p, ncol.p, share.p,
                                                  soff.p, mroff.p, apass.p, opoff.p, res.cigar.p);
            SDF_HIP(hipGetLastError());
        }
        k_records<<<nb(NF), 256, 0, st>>>(ix, dreg.p, foff.p, nr, NF, stats.p, fanchor.p, apass.p,
                                          woff.p, opoff.p, res.sd.p, res.cigar.p);
        SDF_HIP(hipGetLastError());
    }
    SDF_HIP(hipStreamSynchronize(st));
    res.nsd = NSD;
    res.nops = NOPS;
}

}  // namespace sdf
