// Extension of regions by the winnowed MinHash estimate (Section 3.2).
//
// A region pairs G_i = [q0, q1) with G_j = [t0, t1) in orientation o.  Both
// grow by one base per step, first forward (query right end; target right end
// for o = 0, left end for o = 1), then backward from the forward result
// (query left end; target left end for o = 0, right end for o = 1).  A phase
// stops at the first step that leaves a sequence, makes a side longer than
// max_len, makes the two sides intersect (same sequence), or gives a state
// whose estimate m / s is below tau; it keeps the state before that step.
//
// The state is the ordered set L of Section 3.1: the distinct hashes of
// W(G_i) u W(G_j) in ascending order, each with the strands it has on either
// side.  s = |W(G_i)|, and m counts the hashes among the s smallest of L that
// occur on both sides with strands a, b, a xor b = o.  Every minimizer whose
// k-mer lies in a side belongs to it (masked and palindromic ones too).
//
// One workgroup takes one region:
//  1. the minimizers of both start windows and of every position a phase can
//     reach within a horizon H are gathered (six contiguous ranges of the
//     position-sorted minimizer array) and ranked by hash: bucketed on the
//     top 11 hash bits, each run of buckets sorted by one wave in registers,
//     equal hashes sharing a rank, so L becomes an array of 4-bit cells by rank;
//  2. the start windows' minimizers are set, and s, the rank v of the s-th
//     smallest element of L, and m are counted in parallel;
//  3. the minimizers that enter are taken in step order, s, v and m kept up to
//     date (an insertion moves v at most one element of L, to its successor or
//     predecessor) and m >= ceil(tau s) checked after each step; steps at which
//     no minimizer enters keep the previous state and its outcome.  Up to 256
//     minimizers per side are tried at once: the state after each step follows
//     from prefix sums over them and from the elements of L next to v, so all
//     their steps are checked together, and they are inserted up to the first
//     step refused.
// The horizon of one attempt is max(h0, longer side) steps per phase, half of
// that, and again half, while the minimizers within it are more than the scratch
// or a hash bucket holds.  A phase that runs through it stops at its last step; the next attempt
// gathers and ranks again around the region reached and continues the same
// phase from there (the state is a function of the region, so nothing is
// repeated).
//
// Bound by the slowest region, whose entering minimizers form one chain
// (430 kbp a side on the 50 Mbp workload, about 200,000 of them: chance
// matches hold a large region's estimate just above the threshold, so nearly
// every step has to be checked) and whose ranks are sorted again by every
// attempt.  9,157 regions of that workload: 30 ms with one wave trying 128
// events under a slack bound and the ranks sorted in LDS by the workgroup (its
// slowest region 29 ms), 12.3 ms now (8 ms).
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "extend.h"
#include "search.h"
#include "wave.h"

namespace sdf {

namespace {

constexpr int XT = 256;                 // threads per workgroup
// Every parity run of this kernel used 256-thread workgroups.  A build with
// 512 threads stopped answering once on the GPU and its cause is unknown
// (the block scans, chunk bounds, bitonic loops and barriers read
// correctly for any multiple of 64), so the size stays fixed until that
// cause is found.
static_assert(XT == 256, "k_extend is only validated with 256-thread workgroups");
constexpr uint32_t NB_BITS = 11;
constexpr uint32_t NB = 1u << NB_BITS;  // buckets over the top hash bits
constexpr uint32_t CH = 2048;           // keys sorted at once in LDS
// A chunk of several buckets holds at most 512 keys; buckets at the low end of
// the hashes (minimizers crowd there) up to 1,024 are a wave's too.
constexpr uint32_t HALF = 256;
constexpr int XW = XT / 64;
constexpr int UN = 8;                   // elements per thread and round while gathering
constexpr uint64_t HB_DIV = 4;          // backward horizon: at least a quarter of the longer side
constexpr uint32_t TAGS = 2048;         // tags of a batch's events
constexpr uint32_t LDS_WORDS = NB + 1 + (NB + 2) / 2 + 2 * CH + 1;  // the sort area, as words
constexpr uint64_t INF = 1ull << 62;

enum { C_Q0 = 1, C_Q1 = 2, C_T0 = 4, C_T1 = 8 };
enum { STOP_BOUND = 1, STOP_CAP = 2, STOP_OVERLAP = 3, STOP_ESTIMATE = 4 };
constexpr uint32_t RANK_REP = 1u << 31;
enum { XE_CAP = 1, XE_HASH = 2, XE_STATE = 4 };

struct ExtArgs {
    IndexView ix;
    const sdf_region *in;
    uint64_t n;
    sdf_region *out;
    double tau;
    uint64_t max_len;
    uint64_t h0;            // horizon per attempt: max(h0, longer side / hdiv) steps
    uint32_t *work;         // region counter
    uint64_t *tmp;          // per workgroup: ecap keys
    uint32_t *rank;         // per workgroup: ecap
    uint32_t *gnib;         // per workgroup: ecap / 8 + 1
    uint64_t ecap;
    uint32_t lds_words;     // cells kept in LDS up to 8 * lds_words ranks
    uint32_t batches;       // 0: one step at a time
    uint32_t hdiv;          // horizon per attempt: at least the longer side / hdiv
    uint64_t hb0;           // backward horizon while the forward phase is pending (0: same)
    uint32_t *err;
    unsigned long long *stats;  // [0] insertions, [1] continued attempts, [2] ranks,
                                // [3] ranking ticks, [4] event-loop ticks, [5] slowest region,
                                // [6] buckets ranked through the hash set
};

struct Shared {
    union {
        struct {
            uint32_t bs[NB + 1];    // bucket starts
            uint16_t cl[NB + 2];    // first bucket of each chunk
            uint64_t ck[CH];        // cursors; the hash set of a large bucket
        };
        uint32_t w[LDS_WORDS];      // afterwards: the cells of L
    };
    uint32_t red[2 * XW];
    uint32_t estep[2][XT];      // held events of both sides: step (NONE32 past the last),
    uint32_t ecell[2][XT];      // rank << 4 | cell bit,
    uint32_t epre[2][XT];       // inclusive prefix sums of what they change
    uint32_t wsum[2][XW];
    uint16_t tag[TAGS];         // event named for each slot of ranks
    uint32_t near[2][64];       // elements of L above v, and from v down: rank << 1 | shared
    uint32_t nn[2];
    int32_t nr[2];              // ranks that near[] describes completely: nr[1] .. nr[0]
    uint64_t nsh[2];            // bit i: near[][i] is shared
    uint32_t dark, refused;     // first step of a batch not told, refused
    uint64_t uq, ut, last;      // events consumed per side, steps taken
    uint32_t ok, code, nq, nt;
    uint64_t mlo[6], mhi[6];
    uint32_t base[7];
    uint32_t region;
    uint32_t nchunk, cnt;
    int32_t v;
    uint32_t s, m;
    uint32_t flag;
};

// First minimizer with pos >= x, searched by 16 neighbouring lanes with the
// same x: 16 probes per round.  Every lane of the wave takes part.
__device__ __forceinline__ uint64_t lower_pos16(const IndexView &ix, uint64_t x) {
    const uint32_t lane = threadIdx.x & 63, sub = lane & 15, sh = lane & 48;
    uint64_t lo = 0, hi = ix.nm;  // the answer lies in [lo, hi]
    while (__ballot(hi > lo)) {
        const uint64_t step = (hi - lo + 15) / 16;
        const uint64_t pr = lo + sub * step;
        const bool below = pr < hi && (uint64_t)ix.mpos[pr] < x;  // a prefix of the 16
        const uint32_t c = (uint32_t)__popcll((__ballot(below) >> sh) & 0xFFFFull);
        const uint64_t nhi = min(hi, lo + (uint64_t)c * step);
        lo = c ? lo + (uint64_t)(c - 1) * step + 1 : lo;
        hi = c ? nhi : lo;
    }
    return lo;
}

// Cell bits present per nibble (bit 0 of each nibble set).
__device__ __forceinline__ uint32_t nz_mask(uint32_t w) {
    return (w | (w >> 1) | (w >> 2) | (w >> 3)) & 0x11111111u;
}
__device__ __forceinline__ uint32_t q_mask(uint32_t w) {
    return (w | (w >> 1)) & 0x11111111u;
}
__device__ __forceinline__ uint32_t shared_mask(uint32_t w, uint32_t o) {
    if (o == 0) {
        const uint32_t x = w & (w >> 2) & 0x33333333u;
        return (x | (x >> 1)) & 0x11111111u;
    }
    return ((w & (w >> 3)) | ((w >> 1) & (w >> 2))) & 0x11111111u;
}
__device__ __forceinline__ bool cell_shared(uint32_t c, uint32_t o) {
    return shared_mask(c, o) != 0;
}

__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v);

// Exclusive block scan of one value per thread; returns the total.  One
// barrier: two sets of wave totals take turns.
__device__ __forceinline__ uint32_t block_scan(Shared &L, uint32_t v, uint32_t &excl, uint32_t &turn) {
    const uint32_t incl = wave_incl_sum(v), w = threadIdx.x >> 6;
    uint32_t *red = L.red + turn * XW;
    turn ^= 1;
    if ((threadIdx.x & 63) == 63) red[w] = incl;
    __syncthreads();
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (uint32_t t = 0; t < (uint32_t)XW; t++) {
        if (t < w) before += red[t];
        tot += red[t];
    }
    excl = before + incl - v;
    return tot;
}

__device__ __forceinline__ uint32_t block_sum(Shared &L, uint32_t v, uint32_t &turn) {
    uint32_t e;
    return block_scan(L, v, e, turn);
}

// Region geometry of one phase: which ends grow.
struct Phase {
    uint32_t ql, qr, tl, tr;  // growth per step of q0 (down), q1 (up), t0 (down), t1 (up)
};
__device__ __forceinline__ Phase phase_of(int dir, uint32_t o) {
    Phase p;
    p.ql = dir; p.qr = 1 - dir;
    p.tl = dir == 0 ? o : 1 - o;
    p.tr = 1 - p.tl;
    return p;
}

// Steps a phase may take before a sequence end, the length cap or an
// overlap, and the stop code of the first refused step.
__device__ void phase_limit(const uint64_t r[4], uint64_t qlo, uint64_t qhi, uint64_t tlo,
                            uint64_t thi, bool same_seq, const Phase &p, uint64_t max_len,
                            uint64_t &lim, uint32_t &code) {
    uint64_t lb = INF;
    if (p.ql) lb = std::min(lb, r[0] - qlo);
    if (p.qr) lb = std::min(lb, qhi - r[1]);
    if (p.tl) lb = std::min(lb, r[2] - tlo);
    if (p.tr) lb = std::min(lb, thi - r[3]);
    const uint64_t lc = max_len - std::max(r[1] - r[0], r[3] - r[2]);
    uint64_t lo = INF;
    if (same_seq) {
        if (r[1] <= r[2]) {  // query before target
            const uint64_t c = p.qr + p.tl;
            lo = c ? (r[2] - r[1]) / c : INF;
        } else if (r[3] <= r[0]) {  // target before query
            const uint64_t c = p.ql + p.tr;
            lo = c ? (r[0] - r[3]) / c : INF;
        } else {
            lo = 0;
        }
    }
    lim = std::min(lb, std::min(lc, lo));
    code = lb == lim ? STOP_BOUND : (lc == lim ? STOP_CAP : STOP_OVERLAP);
}

struct Est {
    int32_t v;  // rank of the s-th smallest element of L (-1 when s = 0)
    uint32_t s, m;
};

__device__ __forceinline__ bool passes(const Est &e, double tau) {
    return e.s > 0 && e.m >= (uint32_t)ceil(tau * (double)e.s);
}

__device__ __forceinline__ uint32_t cell_at(const uint32_t *nib, int32_t r) {
    return (nib[r >> 3] >> ((r & 7) * 4)) & 15u;
}

// Smallest rank > v holding an element (one exists by construction), and
// its cell; the wave probes 64 cell words per step.
__device__ __forceinline__ int32_t succ_rank(const uint32_t *nib, int32_t v, uint32_t nw,
                                             uint32_t &cell) {
    const int32_t r = v + 1;
    if ((uint32_t)r >= nw * 8) return -2;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t w0 = (uint32_t)r >> 3;
    const uint32_t first_mask = 0xFFFFFFFFu << ((r & 7) * 4);
    for (uint32_t base = w0; base < nw; base += 64) {
        const uint32_t w = base + lane;
        uint32_t word = w < nw ? nib[w] : 0u;
        if (w == w0) word &= first_mask;
        const uint32_t u = nz_mask(word);
        const uint64_t hit = __ballot(u != 0);
        if (hit) {
            const uint32_t l = (uint32_t)__builtin_ctzll(hit);
            const uint32_t ul = __builtin_amdgcn_readlane(u, l);
            const uint32_t wl = __builtin_amdgcn_readlane(word, l);
            const uint32_t nib_i = (uint32_t)__builtin_ctz(ul) >> 2;
            cell = (wl >> (nib_i * 4)) & 15u;
            return (int32_t)((base + l) * 8 + nib_i);
        }
    }
    return -2;
}

// Largest rank < v holding an element (one exists by construction), and its
// cell; the wave probes 64 cell words per step, downwards.
__device__ __forceinline__ int32_t pred_rank(const uint32_t *nib, int32_t v, uint32_t &cell) {
    const int32_t r = v - 1;
    if (r < 0) return -2;
    const uint32_t lane = threadIdx.x & 63;
    const int32_t w0 = r >> 3;
    const uint32_t first_mask = (r & 7) == 7 ? 0xFFFFFFFFu : ((1u << (((r & 7) + 1) * 4)) - 1u);
    for (int32_t top = w0; top >= 0; top -= 64) {
        const int32_t w = top - (int32_t)lane;
        uint32_t word = w >= 0 ? nib[w] : 0u;
        if (w == w0) word &= first_mask;
        const uint32_t u = nz_mask(word);
        const uint64_t hit = __ballot(u != 0);
        if (hit) {
            const uint32_t l = (uint32_t)__builtin_ctzll(hit);  // nearest word below
            const uint32_t ul = __builtin_amdgcn_readlane(u, l);
            const uint32_t wl = __builtin_amdgcn_readlane(word, l);
            const uint32_t nib_i = (31u - (uint32_t)__builtin_clz(ul)) >> 2;
            cell = (wl >> (nib_i * 4)) & 15u;
            return (top - (int32_t)l) * 8 + (int32_t)nib_i;
        }
    }
    return -2;
}

struct Undo {  // at most two cells change per step
    uint32_t n;
    uint32_t w0, old0, w1, old1;
};

// Adds `bit` to the cell of rank r and updates (s, v, m).  Returns false
// when the structure is inconsistent (never for a valid state).
__device__ __forceinline__ bool insert(uint32_t *nib, uint32_t nw, uint32_t r, uint32_t bit, uint32_t o, Est &e,
                       Undo &u) {
    const uint32_t wi = r >> 3, sh = (r & 7) * 4;
    const uint32_t word = nib[wi];
    const uint32_t c = (word >> sh) & 15u, c2 = c | bit;
    if (c2 == c) return true;
    if (u.n == 0) { u.w0 = wi; u.old0 = word; } else { u.w1 = wi; u.old1 = word; }
    u.n++;
    nib[wi] = word | (bit << sh);
    const bool was_u = c != 0;
    const bool new_q = (bit & 3u) && !(c & 3u);
    const bool gain = !cell_shared(c, o) && cell_shared(c2, o);
    const int32_t ri = (int32_t)r;
    if (new_q) {
        e.s++;
        if (!was_u && ri < e.v) return true;  // enters below v: v stays the s-th
        if (was_u && ri <= e.v && gain) e.m++;
        uint32_t cv;
        const int32_t vn = succ_rank(nib, e.v, nw, cv);
        if (vn < 0) return false;
        if (cell_shared(cv, o)) e.m++;
        e.v = vn;
    } else if (!was_u) {
        if (ri < e.v) {  // a new target-side element pushes v out of the s smallest
            if (cell_shared(cell_at(nib, e.v), o)) e.m--;
            uint32_t cv;
            const int32_t vn = pred_rank(nib, e.v, cv);
            if (vn < 0) return false;
            e.v = vn;
        }
    } else if (ri <= e.v && gain) {
        e.m++;
    }
    return true;
}

__device__ __forceinline__ void undo(uint32_t *nib, const Undo &u) {
    if (u.n > 1) nib[u.w1] = u.old1;
    if (u.n > 0) nib[u.w0] = u.old0;
}

// One list of entering minimizers: the minimizer array range [lo, hi),
// walked upwards (step = pos + k - ref) or downwards (step = ref - pos).
struct EvList {
    uint64_t lo, hi;
    bool up;
    uint64_t ref;
    uint32_t side;  // C_Q0 or C_T0
    uint32_t base;  // element id of index lo
};

// Inclusive prefix sum over the lanes of the wave, with DPP moves (register
// to register, no trip through the LDS crossbar): prefix within each row of
// 16 lanes, then the last lane of row 0 and of row 2 into rows 1 and 3, then
// lane 31 into rows 2 and 3.  Lanes without a source add 0.
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v) {
    constexpr int ROW_SHR = 0x110, ROW_BCAST15 = 0x142, ROW_BCAST31 = 0x143;
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_SHR + 1, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_SHR + 2, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_SHR + 4, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_SHR + 8, 0xf, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_BCAST15, 0xa, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ROW_BCAST31, 0xc, 0xf, false);
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    return __builtin_amdgcn_readlane(wave_incl_sum(v), 63);
}

// Keys [b, e) of src (whole buckets, so no hash continues outside, and at most
// 64 N): one wave sorts them in registers (bitonic, key t * 64 + lane in x[t])
// and gives every element its rank, equal hashes sharing one.  Ranks of the
// chunk start at b: they have gaps where hashes repeat, but keep the order.
// RANK_REP marks the elements of a hash that occurs more than once.  Sorted
// are the hash, less the chunk's first (hbase), over ten bits of index: in 32
// bits where the chunk's hashes allow, half the instructions per exchange.
template <int N, class K>
__device__ __forceinline__ void rank_chunk(const uint64_t *src, uint32_t b, uint32_t e, uint32_t hbase,
                                           uint32_t *rank) {
    const uint32_t lane = threadIdx.x & 63;
    K x[N];
#pragma unroll
    for (int t = 0; t < N; t++) {
        const uint32_t i = t * 64 + lane;
        x[t] = b + i < e ? ((K)((uint32_t)(src[b + i] >> 32) - hbase) << 10) | i : (K)~(K)0;
    }
    wave_sort_keys<K, N>(x, lane);
    uint32_t eid[N];
#pragma unroll
    for (int t = 0; t < N; t++)
        eid[t] = b + t * 64 + lane < e ? (uint32_t)src[b + (uint32_t)(x[t] & 1023)] : 0u;
    uint32_t heads = 0;  // distinct hashes before register t
    uint32_t before = 0;
    const uint64_t le = lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1;
#pragma unroll
    for (int t = 0; t < N; t++) {
        const uint32_t h = (uint32_t)(x[t] >> 10);
        const uint32_t up = (uint32_t)__shfl_up((int)h, 1, 64), dn = (uint32_t)__shfl_down((int)h, 1, 64);
        const uint32_t p = lane ? up : before;
        before = (uint32_t)__builtin_amdgcn_readlane((int)h, 63);
        const uint32_t next = t + 1 < N ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x[t + 1 < N ? t + 1 : t] >> 10)) : 0u;
        const bool head = (t == 0 && lane == 0) || p != h;
        const uint64_t hm = __ballot(head);
        const bool tail = b + t * 64 + lane + 1 >= e || (lane == 63 ? next : dn) != h;
        if (b + t * 64 + lane < e)
            rank[eid[t]] = (b + heads + (uint32_t)__popcll(hm & le) - 1) | (head && tail ? 0u : RANK_REP);
        heads += (uint32_t)__popcll(hm);
    }
}

// The same for a bucket of 64 * 16 to CH keys, by the whole workgroup in LDS.
__device__ void rank_block(Shared &L, const uint64_t *src, uint32_t b, uint32_t e, uint32_t *rank,
                           uint32_t &turn) {
    uint64_t *ck = L.ck;
    const uint32_t cnt = e - b;
    uint32_t P = 1;
    while (P < cnt) P <<= 1;
    for (uint32_t i = threadIdx.x; i < P; i += XT) ck[i] = i < cnt ? src[b + i] : ~0ull;
    __syncthreads();
    for (uint32_t size = 2; size <= P; size <<= 1) {
        for (uint32_t stride = size >> 1, sh = (uint32_t)__builtin_ctz(size) - 1; stride > 0;
             stride >>= 1, sh--) {
            for (uint32_t i = threadIdx.x; i < P / 2; i += XT) {
                const uint32_t lo = ((i >> sh) << (sh + 1)) | (i & (stride - 1)), hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const uint64_t x = ck[lo], y = ck[hi];
                if ((x > y) == asc) { ck[lo] = y; ck[hi] = x; }
            }
            __syncthreads();
        }
    }
    const uint32_t seg = (cnt + XT - 1) / XT;
    const uint32_t s0 = std::min(cnt, threadIdx.x * seg), s1 = std::min(cnt, s0 + seg);
    uint32_t heads = 0;
    for (uint32_t i = s0; i < s1; i++)
        heads += (i == 0 || (ck[i] >> 32) != (ck[i - 1] >> 32)) ? 1u : 0u;
    uint32_t excl;
    block_scan(L, heads, excl, turn);
    uint32_t r = b + excl;
    for (uint32_t i = s0; i < s1; i++) {
        const bool head = i == 0 || (ck[i] >> 32) != (ck[i - 1] >> 32);
        const bool tail = i + 1 == cnt || (ck[i] >> 32) != (ck[i + 1] >> 32);
        if (head) r++;
        rank[(uint32_t)ck[i]] = (r - 1) | (head && tail ? 0u : RANK_REP);
    }
    __syncthreads();
}

// A bucket of more than CH keys (in practice one hash repeated many times,
// as in a tandem array): collect its distinct hashes in an LDS hash set,
// sort them, and rank each key by binary search.  More than BIGD distinct
// hashes in one bucket is reported as an error.
constexpr uint32_t BIGT = CH / 2;  // hash set slots (u64, tagged)
constexpr uint32_t BIGD = CH / 4;  // distinct hashes allowed
constexpr uint32_t BIGT_BITS = __builtin_ctz(BIGT);
__device__ bool rank_big(Shared &L, const uint64_t *src, uint64_t b, uint64_t e, uint32_t *rank) {
    uint64_t *set = L.ck;           // BIGT slots: (1 << 32) | hash, 0 = empty
    uint64_t *list = L.ck + BIGT;   // BIGT sorted distinct hashes
    for (uint32_t i = threadIdx.x; i < BIGT; i += XT) set[i] = 0;
    if (threadIdx.x == 0) { L.cnt = 0; L.flag = 0; }
    __syncthreads();
    for (uint64_t i = b + threadIdx.x; i < e; i += XT) {
        const uint32_t h = (uint32_t)(src[i] >> 32);
        const uint64_t tag = (1ull << 32) | h;
        uint32_t slot = (h * 0x9E3779B1u) >> (32 - BIGT_BITS);  // multiplicative hash
        for (uint32_t probe = 0;; probe++) {
            if (probe >= BIGT || L.cnt > BIGD) { L.flag = 1; break; }
            const uint64_t prev = atomicCAS((unsigned long long *)&set[slot], 0ull,
                                            (unsigned long long)tag);
            if (prev == 0) { atomicAdd(&L.cnt, 1u); break; }
            if (prev == tag) break;
            slot = (slot + 1) & (BIGT - 1);
        }
    }
    __syncthreads();
    const bool over = L.flag || L.cnt > BIGD;
    const uint32_t D = L.cnt;
    __syncthreads();  // every thread has read the count before it is reset
    if (over) return false;
    uint32_t P = 1;
    while (P < D) P <<= 1;
    if (threadIdx.x == 0) L.cnt = 0;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < BIGT; i += XT)
        if (set[i]) list[atomicAdd(&L.cnt, 1u)] = set[i] & 0xFFFFFFFFull;
    __syncthreads();
    for (uint32_t i = D + threadIdx.x; i < P; i += XT) list[i] = ~0ull;
    __syncthreads();
    for (uint32_t size = 2; size <= P; size <<= 1) {
        for (uint32_t stride = size >> 1, sh = (uint32_t)__builtin_ctz(size) - 1; stride > 0;
             stride >>= 1, sh--) {
            for (uint32_t i = threadIdx.x; i < P / 2; i += XT) {
                const uint32_t lo = ((i >> sh) << (sh + 1)) | (i & (stride - 1)), hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const uint64_t x = list[lo], y = list[hi];
                if ((x > y) == asc) { list[lo] = y; list[hi] = x; }
            }
            __syncthreads();
        }
    }
    for (uint64_t i = b + threadIdx.x; i < e; i += XT) {
        const uint64_t key = src[i];
        const uint64_t h = key >> 32;
        uint32_t lo = 0, hi = D;  // first index with list[index] >= h
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (list[mid] < h) lo = mid + 1; else hi = mid;
        }
        rank[(uint32_t)key] = ((uint32_t)b + lo) | RANK_REP;
    }
    __syncthreads();
    return true;
}

// The elements of L next to v into near[]: those above it by one wave (dir 0),
// from v itself down by another (dir 1), at most `most`.
__device__ __forceinline__ void near_v(Shared &L, const uint32_t *nib, uint32_t nw, int32_t v,
                                       uint32_t most, uint32_t o, int dir) {
    const uint32_t lane = threadIdx.x & 63;
    const int32_t w0 = (dir == 0 ? v + 1 : v) >> 3;
    const int32_t w = dir == 0 ? w0 + (int32_t)lane : w0 - (int32_t)lane;
    uint32_t c = w >= 0 && w < (int32_t)nw ? nib[w] : 0u;
    if (lane == 0) {
        if (dir == 0) c &= 0xFFFFFFFFu << (((v + 1) & 7) * 4);
        else c &= (v & 7) == 7 ? 0xFFFFFFFFu : (1u << (((v & 7) + 1) * 4)) - 1u;
    }
    uint32_t nz = nz_mask(c);
    const uint32_t sh = shared_mask(c, o);
    const uint32_t incl = wave_incl_sum(__popc(nz)), tot = __builtin_amdgcn_readlane(incl, 63);
    const uint32_t n = std::min(most, tot);
    for (uint32_t i = incl - __popc(nz); nz && i < n; i++) {
        const uint32_t b = dir == 0 ? (uint32_t)__builtin_ctz(nz) : 31u - (uint32_t)__builtin_clz(nz);
        nz &= ~(1u << b);
        L.near[dir][i] = (((uint32_t)w * 8 + (b >> 2)) << 1) | ((sh >> b) & 1u);
    }
    __asm__ volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // writes of other lanes before reads
    const uint32_t e = lane < n ? L.near[dir][lane] : 0u;
    const uint64_t shared = __ballot(e & 1u);
    // a list cut short describes the ranks up to its last element, any other
    // all that was read
    const int32_t end = dir == 0 ? (w0 + 64) * 8 - 1 : max(0, (w0 - 63) * 8);
    const int32_t far = tot > n ? (int32_t)(__builtin_amdgcn_readlane(e, n - 1) >> 1) : end;
    if (lane == 0) {
        L.nn[dir] = n;
        L.nr[dir] = far;
        L.nsh[dir] = shared;
    }
}

struct PhaseIn {
    uint64_t qlo, qhi, tlo, thi;
    bool same;
    uint32_t o;
    uint64_t Hf, Hb;
    uint64_t start[4];  // the region the lists were gathered for
};

// The first step of the held events from (iq, it) on by itself, on wave 0:
// inserts, checks, and undoes a refused step.
__device__ __forceinline__ void one_step(const ExtArgs &a, Shared &L, uint32_t *nib, uint32_t nw,
                                         uint32_t iq, uint32_t it, uint32_t o,
                                         unsigned long long &applied) {
    Est e{L.v, L.s, L.m};
    const Est prev = e;
    const uint32_t sq = iq < XT ? L.estep[0][iq] : NONE32, st = it < XT ? L.estep[1][it] : NONE32;
    const uint32_t te = std::min(sq, st);
    bool ok = L.ok != 0, bad = false;
    uint64_t last = L.last;
    uint32_t code = 0, nq = 0, nt = 0;
    if (te > last + 1 && !ok) {  // steps without an entering minimizer keep the state
        code = STOP_ESTIMATE;
    } else {
        Undo u;
        u.n = 0;
        if (sq == te) {
            const uint32_t c = L.ecell[0][iq];
            bad |= !insert(nib, nw, c >> 4, c & 15u, o, e, u);
            nq = 1;
        }
        if (st == te) {
            const uint32_t c = L.ecell[1][it];
            bad |= !insert(nib, nw, c >> 4, c & 15u, o, e, u);
            nt = 1;
        }
        applied += nq + nt;
        if (passes(e, a.tau)) {
            ok = true;
            last = te;
        } else {
            undo(nib, u);
            e = prev;
            code = STOP_ESTIMATE;
            last = te - 1;
        }
    }
    if (threadIdx.x == 0) {
        L.v = e.v; L.s = e.s; L.m = e.m;
        L.uq += nq;
        L.ut += nt;
        L.last = last;
        L.ok = ok;
        L.code = code;
        if (bad) L.flag |= 4u;
    }
}

// Number of the sorted steps [0, XT) up to `step`.
__device__ __forceinline__ uint32_t upto(const uint32_t *steps, uint32_t step) {
    uint32_t lo = 0, hi = XT;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (steps[mid] <= step) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// One phase, by the workgroup.  Up to XT entering minimizers per side are held,
// in step order, and the steps up to S (every event of which is held) are
// tried together while the state passes: after an event's step, with all events
// up to it, s has grown by the hashes new to the query side (dS), the elements
// new below v (nB) have moved v by d = dS - nB elements up or down, and m
// follows the elements that became shared at or below v (gB) and the shared
// ones among those d elements: prefix sums over the two lists and the elements
// next to v.  Events that change elements next to v, and a v that leaves them,
// end what can be told; the batch is applied up to the first step refused or
// not told, which is then done by itself.  Leaves the steps taken in L.last and
// the stop code in L.code (0: the events ran out before the phase could stop,
// a larger horizon is needed).
__device__ __forceinline__ void run_phase(const ExtArgs &a, Shared &L, uint32_t *nib, uint32_t nw,
                                          const uint32_t *rank, const EvList &lq, const EvList &lt,
                                          uint64_t known, uint64_t lim, uint32_t lim_code, uint32_t o,
                                          unsigned long long &applied) {
    const uint32_t tid = threadIdx.x, wave = tid >> 6;
    const uint64_t count[2] = {lq.hi - lq.lo, lt.hi - lt.lo};
    if (tid == 0) {
        L.uq = L.ut = L.last = 0;
        L.code = 0;
        L.ok = passes(Est{L.v, L.s, L.m}, a.tau);
    }
    for (;;) {
        __syncthreads();  // the state of the last round
        if (L.code || (L.flag & 4u)) return;
        const uint64_t used[2] = {L.uq, L.ut};
        uint32_t step[2], cell[2];
#pragma unroll
        for (int d = 0; d < 2; d++) {
            const EvList &l = d ? lt : lq;
            const uint64_t u = used[d] + tid;
            step[d] = NONE32;
            cell[d] = 0;
            if (u < count[d]) {
                const uint64_t mi = l.up ? l.lo + u : l.hi - 1 - u;
                const uint64_t pos = a.ix.mpos[mi];
                step[d] = (uint32_t)(l.up ? pos + a.ix.k - l.ref : l.ref - pos);
                const uint32_t r = rank[l.base + (uint32_t)(mi - l.lo)];
                cell[d] = (r & RANK_REP) | ((r & ~RANK_REP) << 4) | (l.side << (a.ix.mflags[mi] & 1));
            }
            L.estep[d][tid] = step[d];
            L.ecell[d][tid] = cell[d] & ~RANK_REP;
        }
        const int32_t v = L.v;
        const uint32_t s0 = L.s, m0 = L.m;
        const bool batch = L.ok && s0 > 0 && a.batches;
        if (tid == 0) L.dark = L.refused = NONE32;
        if (batch && wave < 2)
            near_v(L, nib, nw, v, s0 < 512 ? 8u : s0 < 8192 ? 16u : s0 < 32768 ? 32u : 63u, o, (int)wave);
        __syncthreads();
        const uint64_t te = std::min(L.estep[0][0], L.estep[1][0]);
        if (te > known) break;  // (no event: NONE32, which no step reaches)
        uint64_t S = known;
        if (used[0] + XT < count[0]) S = std::min<uint64_t>(S, L.estep[0][XT - 1]);
        if (used[1] + XT < count[1]) S = std::min<uint64_t>(S, L.estep[1][XT - 1]);
        if (!batch) {
            if (wave == 0) one_step(a, L, nib, nw, 0, 0, o, applied);
            continue;
        }
        // ---- what each event changes, given those before it ----
        bool held[2];
        uint32_t r[2], bit[2], c0[2];
#pragma unroll
        for (int d = 0; d < 2; d++) {
            held[d] = (uint64_t)step[d] <= S;
            r[d] = (cell[d] & ~RANK_REP) >> 4;
            bit[d] = cell[d] & 15u;
            c0[d] = held[d] ? cell_at(nib, (int32_t)r[d]) : 0u;
        }
        // events of one rank see the bits of those before them (by step, query side
        // first): round by round one event of each slot of ranks is named, and all
        // events of the slot look at it (rounds: the most events in a slot)
        bool todo[2];
#pragma unroll
        for (int d = 0; d < 2; d++) todo[d] = held[d] && (cell[d] & RANK_REP);
        const bool rep[2] = {todo[0], todo[1]};
        while (__syncthreads_or(todo[0] || todo[1])) {
#pragma unroll
            for (int d = 0; d < 2; d++)
                if (todo[d]) L.tag[r[d] % TAGS] = (uint16_t)(d * XT + tid);
            __syncthreads();
#pragma unroll
            for (int d = 0; d < 2; d++) {
                if (!rep[d]) continue;
                const uint32_t id = L.tag[r[d] % TAGS];
                const uint32_t od = id / XT, oc = L.ecell[od][id % XT], os = L.estep[od][id % XT];
                if ((oc >> 4) == r[d] && (os < step[d] || (os == step[d] && od < (uint32_t)d)))
                    c0[d] |= oc & 15u;
                if (id == d * XT + tid) todo[d] = false;
            }
        }
        // dS, nB, gB of an event in ten bits each, and whether it is next to v
        const int32_t ra = L.nr[1], rb = L.nr[0];
        uint32_t f[2];
        bool close[2];
#pragma unroll
        for (int d = 0; d < 2; d++) {
            const uint32_t c1 = c0[d] | bit[d];
            const bool ch = held[d] && c1 != c0[d];
            close[d] = ch && (int32_t)r[d] >= ra && (int32_t)r[d] <= rb;
            f[d] = !ch ? 0u
                       : (uint32_t)(!(c0[d] & 3u) && (c1 & 3u)) |
                             ((c0[d] == 0 && (int32_t)r[d] < v) ? 1u << 10 : 0u) |
                             (((int32_t)r[d] <= v && !cell_shared(c0[d], o) && cell_shared(c1, o)) ? 1u << 20 : 0u);
        }
        const uint32_t i0 = wave_incl_sum(f[0]), i1 = wave_incl_sum(f[1]);
        if ((tid & 63) == 63) {
            L.wsum[0][wave] = i0;
            L.wsum[1][wave] = i1;
        }
        __syncthreads();
        uint32_t pre[2] = {i0, i1};
#pragma unroll
        for (uint32_t w = 0; w < (uint32_t)XW; w++)
            if (w < wave) {
                pre[0] += L.wsum[0][w];
                pre[1] += L.wsum[1][w];
            }
        L.epre[0][tid] = pre[0];
        L.epre[1][tid] = pre[1];
        __syncthreads();
        // ---- the state after each event's step ----
        const uint64_t su = L.nsh[0], sd = L.nsh[1];
        const int32_t nu = (int32_t)L.nn[0], nd = (int32_t)L.nn[1];
        auto m_of = [&](uint32_t p, int32_t &d) {  // m after the events counted in p
            d = (int32_t)(p & 1023u) - (int32_t)((p >> 10) & 1023u);
            const uint32_t x = (uint32_t)std::min(d < 0 ? -d : d, 63);
            const uint32_t c = (uint32_t)__popcll((d < 0 ? sd : su) & ((1ull << x) - 1));
            return (int32_t)m0 + (int32_t)(p >> 20) + (d < 0 ? -(int32_t)c : (int32_t)c);
        };
#pragma unroll
        for (int d = 0; d < 2; d++) {
            bool dark = false, refused = false;
            if (held[d]) {
                const uint32_t n = upto(L.estep[1 - d], step[d]);
                const uint32_t p = pre[d] + (n ? L.epre[1 - d][n - 1] : 0u);
                int32_t dv;
                const int32_t m = m_of(p, dv);
                dark = close[d] || dv > nu || -dv >= nd;
                refused = m < (int32_t)(uint32_t)ceil(a.tau * (double)(s0 + (p & 1023u)));
            }
            // (steps ascend with the lanes: the first is the least)
            const uint64_t md = __ballot(dark), mr = __ballot(refused);
            if ((tid & 63) == 0) {
                if (md) atomicMin(&L.dark, L.estep[d][(tid & ~63u) + (uint32_t)__builtin_ctzll(md)]);
                if (mr) atomicMin(&L.refused, L.estep[d][(tid & ~63u) + (uint32_t)__builtin_ctzll(mr)]);
            }
        }
        __syncthreads();
        const uint32_t dark = L.dark, refused = L.refused, cut = std::min(dark, refused);
#pragma unroll
        for (int d = 0; d < 2; d++)
            if (held[d] && step[d] < cut) atomicOr(&nib[r[d] >> 3], bit[d] << ((r[d] & 7) * 4));
        __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // written before the barrier
        if (tid == 0) {
            const uint32_t end = (uint32_t)std::min<uint64_t>((uint64_t)cut - 1, S);  // the last step taken
            const uint32_t tq = upto(L.estep[0], end), tt = upto(L.estep[1], end);
            const uint32_t p = (tq ? L.epre[0][tq - 1] : 0u) + (tt ? L.epre[1][tt - 1] : 0u);
            int32_t d;
            L.m = (uint32_t)m_of(p, d);
            L.s = s0 + (p & 1023u);
            if (d > 0) L.v = (int32_t)(L.near[0][d - 1] >> 1);
            if (d < 0) L.v = (int32_t)(L.near[1][-d] >> 1);
            L.uq += tq;
            L.ut += tt;
            L.last = std::max<uint64_t>(L.last, end);
            applied += tq + tt;
            if (refused < dark) L.code = STOP_ESTIMATE;
            L.nq = tq;
            L.nt = tt;
        }
        if (dark <= refused && dark != NONE32) {  // the next step, which is held, by itself
            __syncthreads();
            if (wave == 0) one_step(a, L, nib, nw, L.nq, L.nt, o, applied);
        }
    }
    // no event up to `known` is left
    __syncthreads();
    if (tid == 0) {
        if (L.last < known && !L.ok) {
            L.code = STOP_ESTIMATE;
        } else {
            L.last = std::max<uint64_t>(L.last, known);
            if (known >= lim) {
                L.code = lim_code;
                L.last = lim;
            }
        }
    }
    __syncthreads();
}

// The phases from `dir0` on, from the state L.v, L.s, L.m of region r.
// Returns 0 when both phases stopped (r, codes final), 2 (forward) / 8
// (backward) when a phase ran through its horizon: r and the state are then
// what it reached, which the next attempt continues from; 4 for an
// inconsistent set.  Inlined once with L in LDS and once in global memory.
__device__ __forceinline__ uint32_t phases(const ExtArgs &a, Shared &L, uint32_t *nib,
                                           uint32_t nw, const uint32_t *rank, const PhaseIn &pi,
                                           int dir0, uint64_t r[4], uint32_t codes[2],
                                           unsigned long long &app) {
    const uint32_t o = pi.o;
    if (threadIdx.x == 0) L.flag = 0;
    for (int dir = dir0; dir < 2; dir++) {
        const Phase p = phase_of(dir, o);
        uint64_t lim;
        uint32_t lcode;
        phase_limit(r, pi.qlo, pi.qhi, pi.tlo, pi.thi, pi.same, p, a.max_len, lim, lcode);
        const uint64_t known = std::min(dir == 0 ? pi.Hf : pi.Hb, lim);
        EvList lq, lt;
        const int iq = dir == 0 ? 2 : 4, it = dir == 0 ? 3 : 5;
        lq.lo = L.mlo[iq]; lq.hi = L.mhi[iq]; lq.base = L.base[iq]; lq.side = C_Q0;
        lt.lo = L.mlo[it]; lt.hi = L.mhi[it]; lt.base = L.base[it]; lt.side = C_T0;
        if (dir == 0) {
            lq.up = true; lq.ref = pi.start[1];
            lt.up = o == 0; lt.ref = o == 0 ? pi.start[3] : pi.start[2];
        } else {
            lq.up = false; lq.ref = pi.start[0];
            lt.up = o == 1; lt.ref = o == 0 ? pi.start[2] : pi.start[3];
        }
        run_phase(a, L, nib, nw, rank, lq, lt, known, lim, lcode, o, app);
        const uint64_t t = L.last;
        const uint32_t code = L.code;
        const bool bad = (L.flag & 4u) != 0;
        __syncthreads();  // read by all before the next phase
        r[0] -= p.ql * t; r[1] += p.qr * t; r[2] -= p.tl * t; r[3] += p.tr * t;
        if (bad) return 4u;
        if (code == 0) return dir == 0 ? 2u : 8u;
        codes[dir] = code;
    }
    return 0;
}

}  // namespace

__global__ void __launch_bounds__(XT) __attribute__((amdgpu_waves_per_eu(3)))
k_extend(ExtArgs a) {
    __shared__ Shared L;
    const IndexView &ix = a.ix;
    const uint32_t k = ix.k;
    const uint64_t blk = blockIdx.x;
    uint64_t *tmp = a.tmp + blk * a.ecap;
    uint32_t *rank = a.rank + blk * a.ecap;
    uint32_t *gnib = a.gnib + blk * (a.ecap / 8 + 1);
    const uint32_t hbits = 2 * k;
    const uint32_t shift = hbits > NB_BITS ? hbits - NB_BITS : 0;
    const uint32_t nbk = 1u << (hbits - shift);
    constexpr uint32_t PER = NB / XT;
    uint32_t turn = 0;  // set of wave totals that the next block scan uses

    for (;;) {
        if (threadIdx.x == 0) L.region = atomicAdd(a.work, 1u);
        __syncthreads();
        const uint32_t id = L.region;
        __syncthreads();
        if (id >= a.n) break;
        const uint64_t t_region = wall_clock64();
        const sdf_region R = a.in[id];
        const uint32_t o = R.strand;
        const uint64_t qlo = ix.off[R.q_seq], qhi = ix.off[R.q_seq + 1];
        const uint64_t tlo = ix.off[R.t_seq], thi = ix.off[R.t_seq + 1];
        const bool same = R.q_seq == R.t_seq;
        uint64_t r[4] = {qlo + R.q_begin, qlo + R.q_end, tlo + R.t_begin, tlo + R.t_end};
        sdf_region res = R;
        if (r[1] - r[0] > a.max_len || r[3] - r[2] > a.max_len) {
            if (threadIdx.x == 0) {
                res.m = res.s = 0;
                res.stop = STOP_CAP | (STOP_CAP << 8);
                a.out[id] = res;
            }
            continue;
        }
        unsigned long long applied = 0, t_rank = 0, t_loop = 0;
        uint32_t attempts = 0;
        uint32_t codes[2] = {0, 0};
        int dir = 0;          // the phase the next attempt continues
        uint64_t hcut = ~0ull;  // horizon cap after a scratch overflow
        bool failed = false;
        Est e{-1, 0, 0};
        for (;;) {  // attempts: gather, rank, run until both phases stop
            const uint64_t t_att = wall_clock64();
            const uint64_t longer = std::max(r[1] - r[0], r[3] - r[2]);
            const uint64_t want =
                std::max<uint64_t>(1, std::min(hcut, std::max(a.h0, longer / a.hdiv)));
            uint64_t lim_f;
            uint32_t code_f;
            phase_limit(r, qlo, qhi, tlo, thi, same, phase_of(0, o), a.max_len, lim_f, code_f);
            const uint64_t Hf = dir == 0 ? std::min(want, lim_f) : 0;
            uint64_t ub_b = std::min(r[0] - qlo, o == 0 ? r[2] - tlo : thi - r[3]);
            ub_b = std::min(ub_b, a.max_len - longer);
            // the backward phase starts from a state the forward phase has driven
            // to the threshold and seldom goes far: while the forward phase is
            // pending a shorter backward horizon is gathered (a backward phase that
            // runs through it continues in the next attempt, which ranks everything
            // again: a quarter of the longer side spares most large regions that)
            const uint64_t Hb =
                std::min(dir == 0 && a.hb0 ? std::min(want, std::max(a.hb0, longer / HB_DIV)) : want, ub_b);
            // position ranges [pa, pe] of the six element lists: both windows,
            // then the forward and the backward minimizers that can enter
            int64_t pa[6], pe[6];  // (indexed by constants only: registers)
            pa[0] = (int64_t)r[0]; pe[0] = (int64_t)r[1] - k;
            pa[1] = (int64_t)r[2]; pe[1] = (int64_t)r[3] - k;
            pa[2] = (int64_t)r[1] + 1 - k; pe[2] = (int64_t)(r[1] + Hf) - k;
            if (o == 0) { pa[3] = (int64_t)r[3] + 1 - k; pe[3] = (int64_t)(r[3] + Hf) - k; }
            else { pa[3] = (int64_t)r[2] - (int64_t)Hf; pe[3] = (int64_t)r[2] - 1; }
            pa[4] = (int64_t)r[0] - (int64_t)Hb; pe[4] = (int64_t)r[0] - 1;
            if (o == 0) { pa[5] = (int64_t)r[2] - (int64_t)Hb; pe[5] = (int64_t)r[2] - 1; }
            else { pa[5] = (int64_t)r[3] + 1 - k; pe[5] = (int64_t)(r[3] + Hb) - k; }
            if (Hf == 0) { pa[2] = pa[3] = 1; pe[2] = pe[3] = 0; }
            if (Hb == 0) { pa[4] = pa[5] = 1; pe[4] = pe[5] = 0; }
            {
                const uint32_t gp = threadIdx.x >> 4, l = min(gp >> 1, 5u);  // 16 lanes per bound
                int64_t lo_p = pa[0], hi_p = pe[0];
#pragma unroll
                for (uint32_t t = 1; t < 6; t++)
                    if (l == t) { lo_p = pa[t]; hi_p = pe[t]; }
                const bool hi_end = gp & 1;
                const int64_t x = hi_end ? hi_p + 1 : lo_p;
                uint64_t v = lower_pos16(ix, (uint64_t)std::max<int64_t>(x, 0));
                if (hi_p < lo_p) v = 0;
                if (gp < 12 && (threadIdx.x & 15) == 0) {
                    if (hi_end) L.mhi[l] = v; else L.mlo[l] = v;
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                uint32_t acc = 0;
                for (int l = 0; l < 6; l++) {
                    if (L.mhi[l] < L.mlo[l]) L.mhi[l] = L.mlo[l];
                    L.base[l] = acc;
                    const uint64_t c = L.mhi[l] - L.mlo[l];
                    acc = (uint32_t)std::min<uint64_t>((uint64_t)acc + c, 0xFFFFFFFFull);
                }
                L.base[6] = acc;
                L.flag = 0;
            }
            __syncthreads();
            const uint64_t E = L.base[6];
            if (E > a.ecap) {
                // shorten the horizon; give up when it cannot shrink
                if (want <= 1) {
                    if (threadIdx.x == 0) atomicOr(a.err, (uint32_t)XE_CAP);
                    failed = true;
                    break;
                }
                hcut = want / 2;
                continue;
            }
            attempts++;
            // 1. bucket by the top hash bits into tmp
            for (uint32_t i = threadIdx.x; i < NB + 1; i += XT) L.bs[i] = 0;
            __syncthreads();
            // (UN elements per thread and round, their loads in flight together: a
            // region's elements are taken by one workgroup alone)
            for (int l = 0; l < 6; l++) {
                const uint64_t hi = L.mhi[l];
                for (uint64_t i = L.mlo[l] + threadIdx.x; i < hi; i += XT * UN) {
                    uint32_t h[UN];
#pragma unroll
                    for (int u = 0; u < UN; u++) h[u] = ix.mhash[std::min(i + (uint64_t)u * XT, hi - 1)];
#pragma unroll
                    for (int u = 0; u < UN; u++)
                        if (i + (uint64_t)u * XT < hi) atomicAdd(&L.bs[(h[u] >> shift) & (nbk - 1)], 1u);
                }
            }
            __syncthreads();
            {
                uint32_t loc = 0;
                for (uint32_t t = 0; t < PER; t++) loc += L.bs[threadIdx.x * PER + t];
                uint32_t ex;
                block_scan(L, loc, ex, turn);
                for (uint32_t t = 0; t < PER; t++) {
                    const uint32_t c = L.bs[threadIdx.x * PER + t];
                    L.bs[threadIdx.x * PER + t] = ex;
                    ex += c;
                }
                if (threadIdx.x == 0) L.bs[NB] = (uint32_t)E;
                __syncthreads();
            }
            {
                uint32_t *cur = reinterpret_cast<uint32_t *>(L.ck);  // NB cursors
                for (uint32_t i = threadIdx.x; i < NB; i += XT) cur[i] = L.bs[i];
                __syncthreads();
                for (int l = 0; l < 6; l++) {
                    const uint64_t hi = L.mhi[l];
                    const uint32_t eid = L.base[l] - (uint32_t)L.mlo[l];
                    for (uint64_t i = L.mlo[l] + threadIdx.x; i < hi; i += XT * UN) {
                        uint32_t h[UN], at[UN];
#pragma unroll
                        for (int u = 0; u < UN; u++) h[u] = ix.mhash[std::min(i + (uint64_t)u * XT, hi - 1)];
#pragma unroll
                        for (int u = 0; u < UN; u++)
                            if (i + (uint64_t)u * XT < hi)
                                at[u] = atomicAdd(&cur[(h[u] >> shift) & (nbk - 1)], 1u);
#pragma unroll
                        for (int u = 0; u < UN; u++)
                            if (i + (uint64_t)u * XT < hi)
                                tmp[at[u]] = ((uint64_t)h[u] << 32) | (eid + (uint32_t)(i + (uint64_t)u * XT));
                    }
                }
                __syncthreads();
            }
            // 2. chunks of whole buckets: a bucket opens a chunk when its start
            // falls in another half-chunk window than the previous bucket's, or
            // when it or the previous bucket holds more than half a chunk; so a
            // chunk of several buckets holds at most 2 HALF keys
            {
                uint32_t flags = 0, nf = 0;
                for (uint32_t t = 0; t < PER; t++) {
                    const uint32_t bk = threadIdx.x * PER + t;
                    bool open = false;
                    if (bk < nbk) {
                        const uint32_t sz = L.bs[bk + 1] - L.bs[bk];
                        const uint32_t szp = bk ? L.bs[bk] - L.bs[bk - 1] : 0;
                        open = bk == 0 || sz > HALF || szp > HALF ||
                               (L.bs[bk] / HALF) != (L.bs[bk - 1] / HALF);
                    }
                    flags |= (open ? 1u : 0u) << t;
                    nf += open ? 1u : 0u;
                }
                uint32_t ex;
                const uint32_t nch = block_scan(L, nf, ex, turn);
                for (uint32_t t = 0; t < PER; t++)
                    if (flags & (1u << t)) L.cl[ex++] = (uint16_t)(threadIdx.x * PER + t);
                if (threadIdx.x == 0) L.nchunk = nch;
                __syncthreads();
            }
            {
                const uint32_t nch = L.nchunk;
                auto bounds = [&](uint32_t c, uint32_t &c0, uint32_t &c1) {
                    const uint32_t b1 = c + 1 < nch ? L.cl[c + 1] : nbk;
                    c0 = L.bs[L.cl[c]];
                    c1 = b1 < nbk ? L.bs[b1] : (uint32_t)E;
                };
                bool big = false;
                for (uint32_t c = threadIdx.x >> 6; c < nch; c += XW) {
                    uint32_t c0, c1;
                    bounds(c, c0, c1);
                    const uint32_t b0 = L.cl[c], b1 = c + 1 < nch ? L.cl[c + 1] : nbk;
                    const uint32_t hbase = b0 << shift;
                    if (c1 - c0 > 1024) big = true;
                    else if (((uint64_t)(b1 - b0) << shift) >= 1ull << 22) {
                        if (c1 - c0 <= 128) rank_chunk<2, uint64_t>(tmp, c0, c1, hbase, rank);
                        else if (c1 - c0 <= 512) rank_chunk<8, uint64_t>(tmp, c0, c1, hbase, rank);
                        else rank_chunk<16, uint64_t>(tmp, c0, c1, hbase, rank);
                    } else {
                        if (c1 - c0 <= 128) rank_chunk<2, uint32_t>(tmp, c0, c1, hbase, rank);
                        else if (c1 - c0 <= 256) rank_chunk<4, uint32_t>(tmp, c0, c1, hbase, rank);
                        else if (c1 - c0 <= 512) rank_chunk<8, uint32_t>(tmp, c0, c1, hbase, rank);
                        else rank_chunk<16, uint32_t>(tmp, c0, c1, hbase, rank);
                    }
                }
                if (__syncthreads_or(big))
                    for (uint32_t c = 0; c < nch; c++) {
                        uint32_t c0, c1;
                        bounds(c, c0, c1);
                        if (c1 - c0 <= 1024) continue;
                        if (c1 - c0 <= CH) {
                            rank_block(L, tmp, c0, c1, rank, turn);
                        } else if (rank_big(L, tmp, c0, c1, rank)) {
                            if (threadIdx.x == 0) atomicAdd(&a.stats[6], 1ull);
                        } else {
                            if (threadIdx.x == 0) L.flag = 1;
                            __syncthreads();
                            break;
                        }
                    }
                __syncthreads();
            }
            if (L.flag) {
                // a bucket holds too many hashes: shorten the horizon as above (the
                // backward phase's share of it had such regions refused: sides of 1 Mbp
                // with w = 64 gather 4.5 sides' minimizers instead of 4)
                if (want <= 1) {
                    if (threadIdx.x == 0) atomicOr(a.err, (uint32_t)XE_HASH);
                    failed = true;
                    break;
                }
                hcut = want / 2;
                continue;
            }
            const uint32_t nr = (uint32_t)E;  // ranks, gaps included
            const uint32_t nw = (nr + 7) / 8;
            uint32_t *nib = (nw <= a.lds_words) ? L.w : gnib;
            // 3. the state of the current region
            for (uint32_t i = threadIdx.x; i < nw; i += XT) nib[i] = 0;
            __syncthreads();
            for (int l = 0; l < 2; l++) {
                const uint64_t hi = L.mhi[l];
                const uint32_t eid = L.base[l] - (uint32_t)L.mlo[l];
                for (uint64_t i = L.mlo[l] + threadIdx.x; i < hi; i += XT * UN) {
                    uint32_t rr[UN], fl[UN];
#pragma unroll
                    for (int u = 0; u < UN; u++) {
                        const uint64_t x = std::min(i + (uint64_t)u * XT, hi - 1);
                        rr[u] = rank[eid + (uint32_t)x] & ~RANK_REP;
                        fl[u] = ix.mflags[x] & 1u;
                    }
#pragma unroll
                    for (int u = 0; u < UN; u++)
                        if (i + (uint64_t)u * XT < hi)
                            atomicOr(&nib[rr[u] >> 3], (l == 0 ? C_Q0 : C_T0) << fl[u] << ((rr[u] & 7) * 4));
                }
            }
            __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // written before the barrier
            __syncthreads();
            {
                const uint32_t seg = (nw + XT - 1) / XT;
                const uint32_t w0 = std::min(nw, threadIdx.x * seg), w1 = std::min(nw, w0 + seg);
                uint32_t qc = 0, uc = 0;
#pragma unroll 8
                for (uint32_t i = w0; i < w1; i++) {
                    const uint32_t c = nib[i];
                    qc += __popc(q_mask(c & 0x33333333u));
                    uc += __popc(nz_mask(c));
                }
                const uint32_t s = block_sum(L, qc, turn);
                uint32_t ex;
                block_scan(L, uc, ex, turn);
                if (threadIdx.x == 0) { L.v = -1; L.s = s; }
                __syncthreads();
                if (s > 0 && ex < s && s <= ex + uc) {
                    uint32_t need = s - ex;
                    for (uint32_t i = w0; i < w1; i++) {
                        uint32_t u = nz_mask(nib[i]);
                        const uint32_t c = __popc(u);
                        if (need > c) { need -= c; continue; }
                        while (--need) u &= u - 1;
                        L.v = (int32_t)(i * 8 + (__builtin_ctz(u) >> 2));
                        break;
                    }
                }
                __syncthreads();
                const int32_t v = L.v;
                uint32_t mc = 0;
#pragma unroll 8
                for (uint32_t i = w0; i < w1; i++) {
                    const int32_t left = v - (int32_t)(i * 8);  // cells [0, left] of the word count
                    const uint32_t keep = left < 0 ? 0u : left >= 7 ? 0xFFFFFFFFu : (1u << ((left + 1) * 4)) - 1u;
                    mc += __popc(shared_mask(nib[i], o) & keep);
                }
                const uint32_t m = block_sum(L, mc, turn);
                if (threadIdx.x == 0) L.m = m;
                __syncthreads();
            }
            const uint64_t t_mid = wall_clock64();
            // 4. the phases (L in LDS or in global memory)
            const PhaseIn pi{qlo, qhi, tlo, thi, same, o, Hf, Hb, {r[0], r[1], r[2], r[3]}};
            unsigned long long app = 0;
            const uint32_t fl = nw <= a.lds_words ? phases(a, L, L.w, nw, rank, pi, dir, r, codes, app)
                                                  : phases(a, L, gnib, nw, rank, pi, dir, r, codes, app);
            applied += app;
            e.v = L.v; e.s = L.s; e.m = L.m;
            __syncthreads();
            const uint64_t t_end = wall_clock64();
            t_rank += t_mid - t_att;
            t_loop += t_end - t_mid;
            if (fl & 4u) {
                if (threadIdx.x == 0) atomicOr(a.err, (uint32_t)XE_STATE);
                failed = true;
                break;
            }
            if (threadIdx.x == 0) atomicAdd(&a.stats[2], (unsigned long long)nr);
            if (!(fl & 10u)) break;
            dir = (fl & 2u) ? 0 : 1;  // continue the phase that ran out
            hcut = ~0ull;
        }
        if (threadIdx.x == 0) {
            if (failed) {
                res.m = res.s = 0;
                res.stop = 0;
            } else {
                res.q_begin = r[0] - qlo; res.q_end = r[1] - qlo;
                res.t_begin = r[2] - tlo; res.t_end = r[3] - tlo;
                res.m = e.m; res.s = e.s;
                res.stop = codes[0] | (codes[1] << 8);
            }
            a.out[id] = res;
            atomicAdd(&a.stats[0], applied);
            atomicAdd(&a.stats[1], (unsigned long long)(attempts > 0 ? attempts - 1 : 0));
            atomicAdd(&a.stats[3], t_rank);
            atomicAdd(&a.stats[4], t_loop);
            atomicMax(&a.stats[5], (unsigned long long)(wall_clock64() - t_region));
        }
        __syncthreads();
    }
}

void launch_extend(const IndexView &ix, const sdf_region *in, uint64_t n, double tau,
                   uint64_t max_len, sdf_region *out, ExtStats *stats, hipStream_t st) {
    if (stats) *stats = ExtStats{};
    if (n == 0) return;
    int dev = 0, cus = 0;
    SDF_HIP(hipGetDevice(&dev));
    SDF_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // each attempt gathers max(h0, longer side / hdiv) steps per phase; a
    // phase that runs through them continues in the next attempt.  The
    // settings may change the horizon (h0, hdiv), the cells kept in LDS (0
    // keeps L in global memory), the elements per workgroup, whether steps are
    // tried in batches and the backward horizon gathered while the forward phase
    // is pending (hb0)
    // (at least 4,096 or 16,384 steps: 13.8 and 13.6 ms a call for 9,157 regions of
    // 50 Mbp with copies of up to 50 kbp, 2.77 and 2.88 with copies of up to 4)
    const sdf_tuning &tu = tuning();
    const uint64_t h0 = knob(tu.ext_h0, 4096);
    const uint64_t ecap = std::max<uint64_t>(64, knob(tu.ext_ecap, 1u << 18));
    const uint32_t ldsw = std::min<uint32_t>(LDS_WORDS, knob(tu.ext_lds_words, LDS_WORDS));
    const uint32_t batches = knob(tu.ext_batch_min, 1);
    const uint32_t hdiv = std::max<uint32_t>(1, knob(tu.ext_hdiv, 1));
    const uint64_t hb0 = knob(tu.ext_hb0, 512);
    // as many workgroups as fit a CU's LDS; each keeps its own scratch
    const uint64_t per_cu = std::max<uint64_t>(1, (160u * 1024u) / sizeof(Shared));
    const uint64_t grid = std::min<uint64_t>(n, (uint64_t)std::max(1, cus) * per_cu);
    DevBuf<uint64_t> tmp(grid * ecap);
    DevBuf<uint32_t> rank(grid * ecap), gnib(grid * (ecap / 8 + 1));
    DevBuf<uint32_t> work(2);
    DevBuf<unsigned long long> cnt(7);
    SDF_HIP(hipMemsetAsync(work.p, 0, 8, st));
    SDF_HIP(hipMemsetAsync(cnt.p, 0, 56, st));
    ExtArgs a;
    a.ix = ix;
    a.in = in;
    a.n = n;
    a.out = out;
    a.tau = tau;
    a.max_len = max_len;
    a.h0 = h0;
    a.work = work.p;
    a.tmp = tmp.p;
    a.rank = rank.p;
    a.gnib = gnib.p;
    a.ecap = ecap;
    a.lds_words = ldsw;
    a.batches = batches;
    a.hdiv = hdiv;
    a.hb0 = hb0;
    a.err = work.p + 1;
    a.stats = cnt.p;
    k_extend<<<(unsigned)grid, XT, 0, st>>>(a);
    SDF_HIP(hipGetLastError());
    uint32_t herr = 0;
    unsigned long long hc[7] = {0, 0, 0, 0, 0, 0, 0};
    {
        Readback rb(st);
        rb.add(&herr, work.p + 1, 4);
        rb.add(hc, cnt.p, 56);
        rb.wait();
    }
    if (herr & XE_CAP)
        throw Error{SDF_EINTERNAL, "extend: a region's windows hold more minimizers than its scratch"};
    if (herr & XE_HASH)
        throw Error{SDF_EINTERNAL, "extend: more than 512 distinct hashes share 11 hash bits"};
    if (herr & XE_STATE) throw Error{SDF_EINTERNAL, "extend: inconsistent ordered set"};
    const bool print = tu.ext_stats == 1;
    if (stats || print) {
        ExtStats local;
        if (!stats) stats = &local;
        int khz = 0;
        SDF_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
        const double us = khz > 0 ? 1e3 / (double)khz : 0.0;
        stats->events = hc[0];
        stats->restarts = hc[1];
        stats->ranks = hc[2];
        stats->rank_us = (unsigned long long)((double)hc[3] * us);
        stats->loop_us = (unsigned long long)((double)hc[4] * us);
        stats->slowest_us = (unsigned long long)((double)hc[5] * us);
        if (print)
            fprintf(stderr,
                    "[sdf extend] regions=%llu insertions=%llu continued=%llu ranks=%llu "
                    "rank_ms=%.2f phase_ms=%.2f slowest_ms=%.2f big_buckets=%llu\n",
                    (unsigned long long)n, stats->events, stats->restarts, stats->ranks,
                    stats->rank_us / 1e3, stats->loop_us / 1e3, stats->slowest_us / 1e3,
                    hc[6]);
    }
}

}  // namespace sdf
