// Seeds chosen by the winnowed MinHash estimate (Section 2.2, Section 3.1).
//
// With sketch size s = |W(G_i)|, the estimate of windows i and j is
//   |S[W_i u W_j] n S[W_i] n S[W_j]| / |S[W_i u W_j]|,
// S[X] the s smallest hashes of X.  The denominator is s (the union holds
// W_i), and a hash of both windows that lies among the s smallest of the
// union lies among the s smallest of each, so the numerator m is the number
// of shared hashes (in the sense of the shared count: eligible occurrences,
// orientation o, never an occurrence with itself) among the s smallest of
// W_i u W_j.  If y hashes of W_j outside W_i fall among those s smallest,
// they are the y smallest of them, and the other s - y are the s - y
// smallest of W_i: m = #{shared hashes of rank < s - y in W_i}.
//
// A run (consecutive passing candidates of one window and orientation) is
// given by its first and last candidate; every candidate between them
// belongs to it.  One wave takes one run and emits the seed of its largest m
// (earliest j on ties) when m reaches the threshold T[s].
//
// Runs whose target minimizers fit a wave's registers: they are classified
// against the sorted query hashes and sorted by hash once, in registers.  In
// that order a candidate needs no sort of its own: the distinct outside hashes
// of its window are the lanes whose occurrence lies in it and whose previous
// occurrence does not (a compare and a ballot), the number of them below a lane
// is the popcount of the ballot below it, and y, the shared count and m are
// popcounts too.  Bound by the instructions of the two sorts and of the steps.
// A run's target minimizers are about twice its window's, so three sizes cover
// the windows in use; each launch hands the runs past its size on:
//   1. windows and runs of up to 256 minimizers (2 or 4 keys per lane);
//   2. runs of up to 512 (8 per lane);
//   3. windows of up to 512, runs of up to 1,024 (16 per lane).
// The rest (tandem arrays, longer windows) have the window of each candidate
// sorted by itself.  Whole calls over 50 Mbp with duplications (k = 12), against
// 256 as the only size with the rest left to the last launch, and against a sort
// per candidate throughout (LDS marks, a global atomic per seed):
//   min_len 1,000, w 16 ( 88 minimizers a window)   7.1 ms     7.2     15.9
//           2,000, w 16 (176)                      17.4      288      169
//           2,000, w 12 (231)                      32.1    1,521      589
//           2,000, w 12, error 0.15, k 14 (262)    61.4    2,187    1,642
#include <algorithm>
#include <cstdlib>

#include "search.h"
#include "wave.h"

namespace sdf {

constexpr int EW = 3;         // runs (waves) per workgroup
// Most runs per wave of a register launch: their seeds leave with one atomic, and
// so do the runs handed on, since a counter takes one atomic about every 12 ns
// from all CUs together (one per run: 14.2 ms for 1.2 million seeds, whatever the
// kernel did besides).
constexpr uint32_t ERUNS = 32;
constexpr uint64_t EWAVES = 4096;  // 256 CUs with four waves per SIMD
constexpr int AMAX_M = 256, TCAP_M = 64;    // minimizers held where a candidate's window is
constexpr int AMAX_L = 1024, TCAP_L = 512;  // sorted by itself: of a window, of a run
// Listed runs that the register launches leave: with a window of up to AMAX_M
// minimizers, and the others.
constexpr uint32_t RUN_MID = 1u << 30, RUN_LAST = 1u << 31;
// Runs taken at once: a launch of a wave per run stays below 2^32 threads.
constexpr uint64_t RUNS_MAX = 1ull << 25;
constexpr uint16_t TR_IN = 0x8000, TR_SHARED = 0x4000, TR_RANK = 0x3FF;

template <int AMAX, int TC>
struct EstWave {
    static constexpr int amax = AMAX, tcap = TC;
    union {
        uint64_t key[AMAX];  // query sort: hash << 32 | index in the window
        struct {             // the run's target minimizers (positions jf .. jl + n - k)
            uint32_t tp[TC], th[TC];
            uint16_t tr[TC];     // TR_IN: hash in W_i (rank in TR_RANK); TR_SHARED: pairs in o
            uint32_t out[TC];    // hashes of one target window outside W_i
            uint8_t first[TC];   // first of its value among them
        } run;
        struct {             // a run too long for `run`: one target window at a time
            uint32_t out[AMAX];
            uint8_t first[AMAX];
        } big;
    } u;
    uint32_t ahash[AMAX];    // distinct query hashes, ascending (W_i)
    uint32_t acnt[AMAX];     // eligible occurrences per hash: strand 0 low 16 bits, strand 1 high
    uint64_t cbits[AMAX / 64];  // shared hashes by rank in W_i
};

// A target occurrence (minimizer index tm, strand b, hash of rank r in W_i)
// pairs in orientation o when the window holds an eligible query occurrence
// of strand b ^ o other than itself; it can be itself only for o = 0 and tm
// inside the query window's minimizer range [q0, q0 + na).
template <class W>
__device__ __forceinline__ bool pairs(const W &L, uint32_t r, uint32_t b, uint32_t o,
                                      uint64_t tm, uint64_t q0, uint32_t na) {
    const uint32_t a = b ^ o;
    const uint32_t c = (L.acnt[r] >> (16 * a)) & 0xFFFFu;
    const uint32_t self = (o == 0 && tm >= q0 && tm < q0 + na) ? 1u : 0u;
    return c > self;
}

__device__ __forceinline__ uint32_t e_lane() { return threadIdx.x & 63; }

// First index in [0, n) with arr[index] >= x (n if none), 64 probes per step.
__device__ uint64_t wave_lower_bound(const uint32_t *arr, uint64_t n, uint64_t x) {
    const uint32_t lane = e_lane();
    uint64_t lo = 0, hi = n;  // the answer lies in [lo, hi]
    while (hi - lo > 64) {
        const uint64_t step = (hi - lo + 63) / 64;
        const uint64_t pr = lo + lane * step;
        const bool below = pr < hi && (uint64_t)arr[pr] < x;
        const uint32_t c = (uint32_t)__popcll(__ballot(below));  // probes below x form a prefix
        if (c == 0) return lo;
        const uint64_t last_below = lo + (uint64_t)(c - 1) * step;
        const uint64_t next = lo + (uint64_t)c * step;
        lo = last_below + 1;
        if (next < hi) hi = next;
    }
    const bool below = lo + lane < hi && (uint64_t)arr[lo + lane] < x;
    return lo + (uint64_t)__popcll(__ballot(below));
}

// Ascending bitonic sort of key[0, m) by one wave; m is a power of two.
__device__ void wave_bitonic(uint64_t *key, uint32_t m) {
    for (uint32_t k = 2; k <= m; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t t = e_lane(); t < m; t += 64) {
                const uint32_t u = t ^ j;
                if (u > t) {
                    const bool up = (t & k) == 0;
                    const uint64_t a = key[t], b = key[u];
                    if ((a > b) == up) {
                        key[t] = b;
                        key[u] = a;
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Number of hashes in ahash[0, s) below h.
__device__ __forceinline__ uint32_t rank_below(const uint32_t *ahash, uint32_t s, uint32_t h) {
    uint32_t lo = 0, hi = s;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ahash[mid] < h) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// From the shared marks (cbits) and the nb hashes of W_j outside W_i in
// out[0, nb): c when it cannot beat `beat`, else m.
template <class W>
__device__ uint32_t estimate_finish(W &L, const uint32_t *out, uint8_t *first, uint32_t s,
                                    uint32_t nb, bool have, uint32_t beat, uint32_t reg_cap) {
    const uint32_t lane = e_lane();
    const uint32_t nw = (s + 63) >> 6;
    __builtin_amdgcn_wave_barrier();
    uint32_t c = 0;  // shared count (every lane reads the nw words: LDS broadcasts)
    for (uint32_t w = 0; w < nw; w++) c += (uint32_t)__popcll(L.cbits[w]);
    if (have && c <= beat) return c;
    // y: distinct outside hashes among the s smallest of the union: b is one
    // iff (distinct outside hashes below b) + (hashes of W_i below b) < s
    uint32_t y = 0;
    if (nb <= reg_cap) {  // reg_cap <= 128
        // two per lane in registers (element lane and lane + 64), sorted by a
        // bitonic network over the wave; then a value is the first of its
        // kind when it differs from the one before it, and its rank among the
        // distinct outside hashes is a popcount of those firsts
        uint32_t x0 = lane < nb ? out[lane] : 0xFFFFFFFFu;
        uint32_t x1 = lane + 64 < nb ? out[lane + 64] : 0xFFFFFFFFu;
#pragma unroll
        for (uint32_t k = 2; k <= 128; k <<= 1) {
#pragma unroll
            for (uint32_t j = k >> 1; j > 0; j >>= 1) {
                if (j == 64) {  // k = 128: elements lane and lane + 64, ascending
                    const uint32_t lo = min(x0, x1), hi = max(x0, x1);
                    x0 = lo;
                    x1 = hi;
                } else {
                    const uint32_t y0 = lane_xor(x0, j);
                    const uint32_t y1 = lane_xor(x1, j);
                    const bool lower = (lane & j) == 0;
                    const bool asc0 = (lane & k) == 0, asc1 = ((lane + 64) & k) == 0;
                    x0 = (lower == asc0) ? min(x0, y0) : max(x0, y0);
                    x1 = (lower == asc1) ? min(x1, y1) : max(x1, y1);
                }
            }
        }
        // padding (all ones) sorts last, so elements [0, nb) are the values
        const uint32_t p0 = (uint32_t)__shfl_up((int)x0, 1, 64);
        // (shifted by all lanes: a shift by the lanes past the first alone finds
        // nothing in the first)
        const uint32_t s1 = (uint32_t)__shfl_up((int)x1, 1, 64);
        const uint32_t p1 = lane ? s1 : (uint32_t)__builtin_amdgcn_readlane((int)x0, 63);
        const bool f0 = lane < nb && (lane == 0 || p0 != x0);
        const bool f1 = lane + 64 < nb && p1 != x1;
        const uint64_t fm0 = __ballot(f0), fm1 = __ballot(f1);
        const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
        const uint32_t dr0 = (uint32_t)__popcll(fm0 & lt);
        const uint32_t dr1 = (uint32_t)__popcll(fm0) + (uint32_t)__popcll(fm1 & lt);
        const bool in0 = f0 && dr0 + rank_below(L.ahash, s, x0) < s;
        const bool in1 = f1 && dr1 + rank_below(L.ahash, s, x1) < s;
        y = (uint32_t)__popcll(__ballot(in0)) + (uint32_t)__popcll(__ballot(in1));
    } else {
        for (uint32_t x = lane; x < nb; x += 64) {
            const uint32_t h = out[x];
            bool f = true;
            for (uint32_t t = 0; t < x; t++)
                if (out[t] == h) {
                    f = false;
                    break;
                }
            first[x] = f ? 1 : 0;
        }
        __builtin_amdgcn_wave_barrier();
        for (uint32_t x0 = 0; x0 < nb; x0 += 64) {
            const uint32_t x = x0 + lane;
            bool in = false;
            if (x < nb && first[x]) {
                const uint32_t h = out[x];
                uint32_t below = rank_below(L.ahash, s, h);
                for (uint32_t t = 0; t < nb && below < s; t++)
                    below += (first[t] && out[t] < h) ? 1u : 0u;
                in = below < s;
            }
            y += (uint32_t)__popcll(__ballot(in));
        }
    }
    // m: shared hashes of rank < s - y in W_i
    const uint32_t lim = s - y;
    uint32_t m = 0;
    for (uint32_t x = 0; x < nw && x * 64 < lim; x++) {
        uint64_t w = L.cbits[x];
        if (lim < x * 64 + 64) w &= (1ull << (lim - x * 64)) - 1;
        m += (uint32_t)__popcll(w);
    }
    return m;
}


// Shared hashes among the s smallest of W_i u W_j for the target window
// starting at minimizer tj (position j).  A candidate whose shared count c
// is not above `beat` cannot win (m <= c, and ties go to the earlier j):
// then c is returned without the estimate.  Returns NONE32 when the window
// holds more minimizers outside W_i than the wave can hold.
template <class W>
__device__ uint32_t estimate_at(const IndexView &ix, W &L, uint32_t s, uint32_t o,
                                uint64_t tj, uint64_t jend, bool have, uint32_t beat,
                                uint32_t reg_cap, uint64_t q0, uint32_t na) {
    const uint32_t lane = e_lane();
    const uint64_t ltmask = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t nw = (s + 63) >> 6;
    uint32_t *out = L.u.big.out;  // hashes of W_j outside W_i
    if (lane < nw) L.cbits[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    uint32_t nb = 0;
    for (uint64_t base = tj;; base += 64) {
        // (position, hash and flags loaded together: a candidate is bound by the
        // latency of its loads)
        const uint64_t tm = base + lane, tc = min(tm, ix.nm - 1);
        const uint32_t pos = ix.mpos[tc], h = ix.mhash[tc];
        const uint8_t fl = ix.mflags[tc];
        const bool v = tm < ix.nm && (uint64_t)pos <= jend;
        bool outside = false;
        if (v) {
            const uint32_t r = rank_below(L.ahash, s, h);
            if (r < s && L.ahash[r] == h) {
                if ((fl & 2) && pairs(L, r, fl & 1, o, tm, q0, na))  // eligible and pairs
                    atomicOr(&L.cbits[r >> 6], 1ull << (r & 63));
            } else {
                outside = true;
            }
        }
        const uint64_t bm = __ballot(outside);
        const uint32_t at = nb + (uint32_t)__popcll(bm & ltmask);
        if (outside && at < W::amax) out[at] = h;
        nb += (uint32_t)__popcll(bm);
        if (__ballot(v) != ~0ull) break;
        if (nb > W::amax) break;
    }
    if (nb > W::amax) return NONE32;
    return estimate_finish(L, out, L.u.big.first, s, nb, have, beat, reg_cap);
}

// The same for the target window u.run.tp[xs, xe) of the run's minimizers held
// in LDS (classified once per run).
template <class W>
__device__ uint32_t estimate_lds(W &L, uint32_t s, uint32_t xs, uint32_t xe, bool have,
                                 uint32_t beat, uint32_t reg_cap) {
    const uint32_t lane = e_lane();
    const uint64_t ltmask = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t nw = (s + 63) >> 6;
    uint32_t *out = L.u.run.out;
    if (lane < nw) L.cbits[lane] = 0;
    __builtin_amdgcn_wave_barrier();
    uint32_t nb = 0;
    for (uint32_t x0 = xs; x0 < xe; x0 += 64) {
        const uint32_t x = x0 + lane;
        const bool v = x < xe;
        const uint16_t tr = v ? L.u.run.tr[x] : (uint16_t)0;
        if (tr & TR_SHARED) {
            const uint32_t r = tr & TR_RANK;
            atomicOr(&L.cbits[r >> 6], 1ull << (r & 63));
        }
        const bool outside = v && !(tr & TR_IN);
        const uint64_t bm = __ballot(outside);
        if (outside) out[nb + (uint32_t)__popcll(bm & ltmask)] = L.u.run.th[x];
        nb += (uint32_t)__popcll(bm);
    }
    return estimate_finish(L, out, L.u.run.first, s, nb, have, beat, reg_cap);  // nb <= W::tcap
}

// The runs of `list` marked MARK, with windows of up to AMAX minimizers (of the
// query, and outside hashes of a target window).  RUN_MID: one that does not fit
// is left to the launch of the RUN_LAST ones (the smaller form has 39 waves per CU,
// the larger nine; a run of thousands of candidates, as along a tandem array, is
// bound by their latency).
template <int AMAX, int TC, uint32_t MARK>
__global__ void __launch_bounds__(EW * 64) k_estimate_long(IndexView ix, const uint32_t *runs,
                                                            uint64_t nruns, uint32_t *list,
                                                            uint32_t n, const uint16_t *T,
                                                            uint32_t *seeds, uint64_t cap,
                                                            unsigned long long *nseeds,
                                                            uint32_t *err, uint32_t lds_cap,
                                                            uint32_t reg_cap) {
    constexpr uint32_t amax_rt = AMAX;
    using Wave = EstWave<AMAX, TC>;
    __shared__ Wave W[EW];
    const uint32_t lane = e_lane(), wv = threadIdx.x >> 6;
    Wave &L = W[wv];
    const uint64_t slot = (uint64_t)blockIdx.x * EW + wv;
    if (slot >= nruns) return;  // whole wave; no workgroup barrier below
    if (!(list[slot] & MARK)) return;
    const uint64_t r = list[slot] & ~MARK;
    const uint64_t ltmask = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t *rec = runs + r * 6;
    const uint32_t qid = rec[0], i = rec[1], jf = rec[2], o = rec[3], jl = rec[4], s = rec[5];
    const uint32_t k = ix.k;

    // ---- W_i: the query window's minimizers, sorted by hash ----
    const uint64_t q0 = wave_lower_bound(ix.mpos, ix.nm, i);
    const uint64_t qend = (uint64_t)i + n - k;
    uint32_t na = 0;
    for (;;) {
        const uint64_t m = q0 + na + lane;
        const bool v = m < ix.nm && (uint64_t)ix.mpos[m] <= qend;
        const uint64_t bv = __ballot(v);  // a prefix of the lanes
        if (v && na + lane < AMAX) L.u.key[na + lane] = ((uint64_t)ix.mhash[m] << 32) | (na + lane);
        na += (uint32_t)__popcll(bv);
        if (bv != ~0ull || na > amax_rt) break;
    }
    if (na > amax_rt || s == 0 || s > na) {
        if (lane == 0) atomicOr(err, na > amax_rt ? 1u : 2u);
        return;
    }
    uint32_t m2 = 1;
    while (m2 < na) m2 <<= 1;
    for (uint32_t t = na + lane; t < m2; t += 64) L.u.key[t] = ~0ull;
    for (uint32_t t = lane; t < na; t += 64) L.acnt[t] = 0;
    __builtin_amdgcn_wave_barrier();
    wave_bitonic(L.u.key, m2);
    // distinct hashes and their eligible occurrences per strand
    uint32_t nd = 0;
    for (uint32_t t0 = 0; t0 < na; t0 += 64) {
        const uint32_t t = t0 + lane;
        bool first = false;
        uint64_t key = 0;
        if (t < na) {
            key = L.u.key[t];
            first = t == 0 || (L.u.key[t - 1] >> 32) != (key >> 32);
        }
        const uint64_t fm = __ballot(first);
        const uint64_t le = fm & (ltmask | (1ull << lane));
        const uint32_t rk = nd + (uint32_t)__popcll(le) - 1;  // rank of the hash
        if (t < na) {
            if (first) L.ahash[rk] = (uint32_t)(key >> 32);
            const uint64_t m = q0 + (uint32_t)key;
            const uint8_t fl = ix.mflags[m];
            if (fl & 2) atomicAdd(&L.acnt[rk], (fl & 1) ? 0x10000u : 1u);
        }
        nd += (uint32_t)__popcll(fm);
        __builtin_amdgcn_wave_barrier();
    }
    __builtin_amdgcn_wave_barrier();  // the sort keys are dead: their space holds the run below
    if (nd != s) {
        if (lane == 0) atomicOr(err, 2u);
        return;
    }

    // ---- the run's candidates, in target order ----
    uint32_t best_m = 0, best_j = 0;
    bool have = false;
    const uint64_t t0 = wave_lower_bound(ix.mpos, ix.nm, jf);
    // the run's target minimizers, classified once, when they fit in LDS
    const uint64_t tend = (uint64_t)jl + n - k;
    uint32_t nt = 0;
    for (;;) {
        const uint64_t tm = t0 + nt + lane;
        const bool v = tm < ix.nm && (uint64_t)ix.mpos[tm] <= tend;
        const uint64_t bv = __ballot(v);  // a prefix of the lanes
        const uint32_t x = nt + lane;
        if (v && x < lds_cap) {
            const uint32_t pos = ix.mpos[tm], h = ix.mhash[tm];
            const uint8_t fl = ix.mflags[tm];
            const uint32_t rk = rank_below(L.ahash, s, h);
            uint16_t tr = 0;
            if (rk < s && L.ahash[rk] == h) {
                tr = (uint16_t)(TR_IN | rk);
                if ((fl & 2) && pairs(L, rk, fl & 1, o, tm, q0, na)) tr |= TR_SHARED;
            }
            L.u.run.tp[x] = pos;
            L.u.run.th[x] = h;
            L.u.run.tr[x] = tr;
        }
        nt += (uint32_t)__popcll(bv);
        if (bv != ~0ull || nt > lds_cap) break;
    }
    __builtin_amdgcn_wave_barrier();
    if (nt <= lds_cap) {
        uint32_t we = 0;  // end of the current candidate's window (non-decreasing in j)
        for (uint32_t x0 = 0; x0 < nt; x0 += 64) {
            const uint32_t x = x0 + lane;
            bool cand = false;
            if (x < nt && L.u.run.tp[x] <= jl && (L.u.run.tr[x] & TR_SHARED))
                cand = window_ok(ix, L.u.run.tp[x], n, nullptr);  // a candidate j of the run
            uint64_t cm = __ballot(cand);
            while (cm) {
                const uint32_t xc = x0 + (uint32_t)__ffsll((long long)cm) - 1;
                cm &= cm - 1;
                const uint32_t j = L.u.run.tp[xc];
                // first minimizer past j + n - k, 64 at a time from the previous end
                for (;;) {
                    const uint32_t y = we + lane;
                    const bool in = y < nt && (uint64_t)L.u.run.tp[y] <= (uint64_t)j + n - k;
                    const uint64_t im = __ballot(in);  // a prefix of the lanes
                    we += (uint32_t)__popcll(im);
                    if (im != ~0ull) break;
                }
                const uint32_t m = estimate_lds(L, s, xc, we, have, best_m, reg_cap);
                if (!have || m > best_m) {
                    best_m = m;
                    best_j = j;
                    have = true;
                }
            }
        }
    }
    for (uint64_t base = t0; nt > lds_cap; base += 64) {
        const uint64_t tm = base + lane;
        const bool v = tm < ix.nm && ix.mpos[tm] <= jl;
        bool cand = false;
        uint32_t pj = 0;
        if (v) {
            pj = ix.mpos[tm];
            const uint8_t fl = ix.mflags[tm];
            if (fl & 2) {
                const uint32_t h = ix.mhash[tm];
                const uint32_t rk = rank_below(L.ahash, s, h);
                if (rk < s && L.ahash[rk] == h)
                    cand = pairs(L, rk, fl & 1, o, tm, q0, na) && window_ok(ix, pj, n, nullptr);
            }
        }
        uint64_t cm = __ballot(cand);
        const bool more = __ballot(v) == ~0ull;
        while (cm) {
            const uint32_t l = (uint32_t)__ffsll((long long)cm) - 1;
            cm &= cm - 1;
            const uint32_t j = (uint32_t)__builtin_amdgcn_readlane((int)pj, (int)l);
            const uint32_t m =
                estimate_at(ix, L, s, o, base + l, (uint64_t)j + n - k, have, best_m, reg_cap, q0, na);
            if (m == NONE32) {
                if (lane == 0) {
                    if (MARK == RUN_MID) list[slot] = (uint32_t)r | RUN_LAST;
                    else atomicOr(err, 1u);
                }
                return;
            }
            if (!have || m > best_m) {
                best_m = m;
                best_j = j;
                have = true;
            }
        }
        if (!more) break;
    }
    if (lane == 0 && have && best_m >= T[s]) {
        const unsigned long long at = atomicAdd(nseeds, 1ull);
        if (at < cap) {
            uint32_t *d = seeds + at * 6;
            d[0] = qid; d[1] = i; d[2] = best_j; d[3] = o; d[4] = best_m; d[5] = s;
        }
    }
}

// ---------------------------------------------------- register launches --
// What a wave of a register launch holds: windows of up to AM minimizers, runs
// of up to TM.  Sort keys are a hash above the bits of an index below TM.
template <int AM, int TM>
struct EstRun {
    static constexpr int amax = AM, tmax = TM;
    static constexpr int ibits = __builtin_ctz(TM);
    uint32_t ahash[AM];  // distinct query hashes, ascending (W_i)
    uint32_t acnt[AM];   // eligible occurrences per hash: strand 0 low 16 bits, strand 1 high
    union {
        uint32_t tp[TM];    // the run's target minimizers: positions;
        uint32_t cand[TM];  // then its candidates in order: place | end of its window's places << 16
    };
    uint16_t tr[TM];     // TR_* and rank, or the hashes of W_i below it when outside
    uint16_t ord[TM];    // in hash order: place in the run | ORD_SAME
    uint32_t seeds[ERUNS * 6];
};
constexpr uint32_t ORD_SAME = 0x8000;  // the hash of the one before

// The keys before x's own in sorted order (lane 0 of register 0: 0).
template <class K, int E>
__device__ __forceinline__ K key_before(const K (&x)[E], int e, uint32_t lane) {
    K p, b = 0;
    if constexpr (sizeof(K) == 8) {
        p = ((K)(uint32_t)__shfl_up((int)(uint32_t)(x[e] >> 32), 1, 64) << 32) |
            (uint32_t)__shfl_up((int)(uint32_t)x[e], 1, 64);
        if (e) b = ((K)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x[e ? e - 1 : 0] >> 32), 63) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x[e ? e - 1 : 0], 63);
    } else {
        p = (K)__shfl_up((int)x[e], 1, 64);
        if (e) b = (K)__builtin_amdgcn_readlane((int)x[e ? e - 1 : 0], 63);
    }
    return lane == 0 ? b : p;
}

// Query hashes of a window in order: distinct ones and their eligible
// occurrences; the number of distinct ones.  Keys: hash over the index of the
// minimizer in the window.
template <class K, int E, class W>
__device__ __forceinline__ uint32_t sort_query(const IndexView &ix, W &L, uint64_t q0, uint32_t na,
                                               uint32_t lane) {
    constexpr int IB = W::ibits;
    K x[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const uint32_t t = e * 64 + lane;
        x[e] = t < na ? ((K)ix.mhash[q0 + t] << IB) | t : (K)~(K)0;
    }
    wave_sort_keys<K, E>(x, lane);
    for (uint32_t t = lane; t < na; t += 64) L.acnt[t] = 0;
    __builtin_amdgcn_wave_barrier();
    const uint64_t le = lane == 63 ? ~0ull : (1ull << (lane + 1)) - 1;
    uint32_t nd = 0;
#pragma unroll
    for (int e = 0; e < E; e++) {
        const K p = key_before<K, E>(x, e, lane);
        const uint32_t t = e * 64 + lane;
        const bool first = t < na && (t == 0 || (p >> IB) != (x[e] >> IB));
        const uint64_t fm = __ballot(first);
        const uint32_t rk = nd + (uint32_t)__popcll(fm & le) - 1;
        if (t < na) {
            if (first) L.ahash[rk] = (uint32_t)(x[e] >> IB);
            const uint8_t fl = ix.mflags[q0 + (uint32_t)(x[e] & (W::tmax - 1))];
            if (fl & 2) atomicAdd(&L.acnt[rk], (fl & 1) ? 0x10000u : 1u);
        }
        nd += (uint32_t)__popcll(fm);
    }
    __builtin_amdgcn_wave_barrier();
    return nd;
}

// The candidate of the largest m among the run's nt <= 64 E target minimizers
// [t0, t0 + nt), whose positions are in tp: best_m and its place; false: none.
template <class K, int E, class W>
__device__ __forceinline__ bool best_candidate(const IndexView &ix, W &L, uint64_t t0, uint32_t nt,
                                               uint64_t q0, uint32_t na, uint32_t s, uint32_t o,
                                               uint32_t n, uint32_t jl, uint32_t lane,
                                               uint32_t &best_m, uint32_t &best_x) {
    constexpr int IB = W::ibits;
    const uint32_t k = ix.k;
    K x[E];
    uint32_t wend[E];  // 0: no candidate
#pragma unroll
    for (int e = 0; e < E; e++) {
        const uint32_t t = e * 64 + lane;
        x[e] = (K)~(K)0;
        wend[e] = 0;
        if (t < nt) {
            const uint32_t h = ix.mhash[t0 + t], pos = L.tp[t];
            const uint8_t fl = ix.mflags[t0 + t];
            const uint32_t rk = rank_below(L.ahash, s, h);
            uint32_t tr = rk;
            if (rk < s && L.ahash[rk] == h) {
                tr |= TR_IN;
                if ((fl & 2) && pairs(L, rk, fl & 1, o, t0 + t, q0, na)) tr |= TR_SHARED;
            }
            L.tr[t] = (uint16_t)tr;
            x[e] = ((K)h << IB) | t;
            if (pos <= jl && (tr & TR_SHARED) && window_ok(ix, pos, n, nullptr)) {
                // the end of its window's minimizers
                uint32_t lo = t, hi = nt;
                const uint64_t lim = (uint64_t)pos + n - k;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if ((uint64_t)L.tp[mid] <= lim) lo = mid + 1; else hi = mid;
                }
                wend[e] = lo;
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
    uint32_t nc = 0;
#pragma unroll
    for (int e = 0; e < E; e++) {
        const uint64_t cm = __ballot(wend[e] != 0);
        if (wend[e])
            L.cand[__builtin_amdgcn_mbcnt_hi((uint32_t)(cm >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)cm, nc))] =
                (e * 64 + lane) | (wend[e] << 16);
        nc += (uint32_t)__popcll(cm);
    }
    wave_sort_keys<K, E>(x, lane);
    // each occurrence, in hash order: its place t in the run, the place of the
    // occurrence before it + 1 (of the shared one before it, if it is shared;
    // NEVER: it does not count), and its rank among the query hashes
    constexpr uint32_t NEVER = 0xFFFF;
    uint32_t at[E], prev[E], rank[E];
    uint64_t outside[E];
#pragma unroll
    for (int e = 0; e < E; e++) {
        const uint32_t y = e * 64 + lane;
        const K p = key_before<K, E>(x, e, lane);  // (by all lanes: a shift reads active ones only)
        const bool same = y > 0 && (p >> IB) == (x[e] >> IB);
        at[e] = y < nt ? (uint32_t)x[e] & (W::tmax - 1) : 0u;
        L.ord[y] = (uint16_t)(at[e] | (same ? ORD_SAME : 0u));
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int e = 0; e < E; e++) {
        const uint32_t y = e * 64 + lane;
        const uint32_t tr = y < nt ? L.tr[at[e]] : (uint32_t)TR_IN;
        uint32_t pv = 0;
        if (y < nt) {
            for (uint32_t z = y; L.ord[z] & ORD_SAME; z--) {
                const uint32_t tb = L.ord[z - 1] & (ORD_SAME - 1);
                if (!(tr & TR_SHARED) || (L.tr[tb] & TR_SHARED)) {
                    pv = tb + 1;
                    break;
                }
            }
        }
        prev[e] = (tr & TR_IN) && !(tr & TR_SHARED) ? NEVER : pv;
        rank[e] = tr & TR_RANK;
        outside[e] = __ballot(!(tr & TR_IN));
    }
    bool have = false;
    for (uint32_t c0 = 0; c0 < nc; c0 += 64) {
        const uint32_t mine = c0 + lane < nc ? L.cand[c0 + lane] : 0u, cn = min(64u, nc - c0);
        for (uint32_t u = 0; u < cn; u++) {
            const uint32_t cd = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)u);
            const uint32_t xs = cd & 0xFFFFu, len = (cd >> 16) - xs;
            uint64_t live[E];
            uint32_t c = 0;
#pragma unroll
            for (int e = 0; e < E; e++) {
                live[e] = __builtin_amdgcn_ballot_w64((at[e] - xs < len) & (prev[e] <= xs));
                c += (uint32_t)__popcll(live[e] & ~outside[e]);
            }
            // (m <= c, and ties go to the earlier candidate)
            if (have && c <= best_m) continue;
            uint32_t y = 0, below = 0;
#pragma unroll
            for (int e = 0; e < E; e++) {
                const uint64_t ob = live[e] & outside[e];
                const uint32_t d = __builtin_amdgcn_mbcnt_hi(
                    (uint32_t)(ob >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ob, below));
                y += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(d + rank[e] < s) & ob);
                below += (uint32_t)__popcll(ob);
            }
            uint32_t m = 0;
#pragma unroll
            for (int e = 0; e < E; e++)
                m += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(rank[e] < s - y) & live[e] & ~outside[e]);
            if (!have || m > best_m) {
                best_m = m;
                best_x = xs;
                have = true;
            }
        }
    }
    return have;
}

// The sizes of the register launches (the settings may lower them).
struct EstSizes {
    uint32_t a[3], t[3];  // minimizers of a window, of a run
};
// (The largest size only while the run is at most three of its windows long, as
// between copies: along a tandem array most of the registers' elements lie
// outside a candidate's window, and such runs go better with the longer ones of
// their array, whose launch waits for one of them.  1 Mbp with arrays of 30 kbp, units
// of 900 bases: 37.1 -> 31.4 ms a call.)
__device__ __forceinline__ uint32_t size_class(const EstSizes &z, uint32_t na, uint32_t nt) {
    return na <= z.a[0] && nt <= z.t[0] ? 0u
           : na <= z.a[1] && nt <= z.t[1] ? 1u
           : na <= z.a[2] && nt <= z.t[2] && nt <= 3 * na ? 2u
           : na <= z.a[1] ? 3u : 4u;
}

// Register launch LEVEL.  Level 0 takes all runs, and hands those past its size
// on: `over` receives the next level's from its front and the others from its
// end, with their marks (nover: how many of each, and how many of the latter are
// marked).  The later ones take the unmarked runs of `list`.
template <class K, int LEVEL, int AM, int TM>
__global__ void __launch_bounds__(EW * 64) k_estimate_runs(IndexView ix, const uint32_t *runs,
                                                            const uint32_t *list, uint64_t nruns,
                                                            uint32_t per, uint32_t n,
                                                            const uint16_t *T, uint32_t *seeds,
                                                            uint64_t cap, unsigned long long *nseeds,
                                                            uint32_t *err, EstSizes sizes,
                                                            uint32_t *over,
                                                            unsigned long long *nover) {
    using Run = EstRun<AM, TM>;
    static_assert(TM <= ORD_SAME && AM <= TR_RANK + 1 && AM <= TM, "fields of tr and ord");
    __shared__ Run W[EW];
    const uint32_t lane = e_lane(), wv = threadIdx.x >> 6;
    Run &L = W[wv];
    const uint32_t k = ix.k;
    const uint64_t r0 = ((uint64_t)blockIdx.x * EW + wv) * per;  // (no workgroup barrier below)
    const uint64_t r1 = min(r0 + per, nruns);
    uint32_t nbuf = 0;
    uint32_t handed = 0;  // lane u: size class of run r0 + u, if it is handed on
    // minimizers [first, first + count) at positions [from, to]; above `most`: most + 1
    auto count = [&](uint64_t first, uint64_t to, uint32_t most, uint32_t *pos) {
        uint32_t c = 0;
        while (c <= most) {
            const uint64_t m = first + c + lane;
            const uint32_t p = m < ix.nm ? ix.mpos[m] : 0xFFFFFFFFu;
            const bool v = m < ix.nm && (uint64_t)p <= to;
            if (pos && v && c + lane < (uint32_t)TM) pos[c + lane] = p;
            const uint64_t bv = __ballot(v);  // a prefix of the lanes
            c += (uint32_t)__popcll(bv);
            if (bv != ~0ull) return c;
        }
        return most + 1;
    };
    for (uint64_t ri = r0; ri < r1; ri++) {
        if (LEVEL > 0 && (list[ri] & (RUN_MID | RUN_LAST))) continue;
        const uint64_t r = LEVEL > 0 ? list[ri] : ri;
        const uint32_t *rec = runs + r * 6;
        const uint32_t qid = rec[0], i = rec[1], jf = rec[2], o = rec[3], jl = rec[4], s = rec[5];
        const uint64_t q0 = wave_lower_bound(ix.mpos, ix.nm, i);
        const uint32_t na = count(q0, (uint64_t)i + n - k, sizes.a[2], nullptr);
        const uint64_t t0 = wave_lower_bound(ix.mpos, ix.nm, jf);
        const uint32_t nt = na > sizes.a[2] ? 0u : count(t0, (uint64_t)jl + n - k, sizes.t[2], L.tp);
        if constexpr (LEVEL == 0) {
            const uint32_t cls = size_class(sizes, na, nt);
            if (cls) {
                handed = lane == (uint32_t)(ri - r0) ? cls : handed;
                continue;
            }
        }
        __builtin_amdgcn_wave_barrier();
        uint32_t nd;
        if (LEVEL < 2 && na <= 128) nd = sort_query<K, 2>(ix, L, q0, na, lane);
        else if (LEVEL < 2 || na <= 256) nd = sort_query<K, 4>(ix, L, q0, na, lane);
        else nd = sort_query<K, AM / 64>(ix, L, q0, na, lane);
        if (nd != s || s == 0) {
            if (lane == 0) atomicOr(err, 2u);
            continue;
        }
        uint32_t best_m = 0, best_x = 0;
        bool have;
        if (LEVEL != 1 && nt <= (uint32_t)TM / 2)
            have = best_candidate<K, TM / 128>(ix, L, t0, nt, q0, na, s, o, n, jl, lane, best_m, best_x);
        else
            have = best_candidate<K, TM / 64>(ix, L, t0, nt, q0, na, s, o, n, jl, lane, best_m, best_x);
        if (have && best_m >= T[s]) {
            const uint32_t best_j = ix.mpos[t0 + best_x];
            if (lane < 6)
                L.seeds[nbuf * 6 + lane] =
                    lane == 0 ? qid : lane == 1 ? i : lane == 2 ? best_j : lane == 3 ? o : lane == 4 ? best_m : s;
            nbuf++;
        }
    }
    if constexpr (LEVEL == 0) {
        const uint64_t next = __ballot(handed == 1), rest = __ballot(handed > 1);
        const uint64_t marked = __ballot(handed > 2);
        if (next | rest) {
            unsigned long long f = 0, b = 0;
            if (lane == 0) {
                if (next) f = atomicAdd(nover, (unsigned long long)__popcll(next));
                if (rest) b = atomicAdd(nover + 1, (unsigned long long)__popcll(rest));
                if (marked) atomicAdd(nover + 2, (unsigned long long)__popcll(marked));
            }
            f = __shfl(f, 0, 64);
            b = __shfl(b, 0, 64);
            const uint64_t lt = (1ull << lane) - 1;
            const uint32_t r = (uint32_t)r0 + lane;
            if (handed == 1) over[f + (uint32_t)__popcll(next & lt)] = r;
            if (handed > 1)
                over[nruns - 1 - (b + (uint32_t)__popcll(rest & lt))] = r | (handed == 3 ? RUN_MID : handed == 4 ? RUN_LAST : 0u);
        }
    }
    if (nbuf == 0) return;
    unsigned long long at = 0;
    if (lane == 0) at = atomicAdd(nseeds, (unsigned long long)nbuf);
    at = __shfl(at, 0, 64);
    __builtin_amdgcn_wave_barrier();
    for (uint32_t t = lane; t < nbuf * 6; t += 64)
        if (at + t / 6 < cap) seeds[at * 6 + t] = L.seeds[t];
}

static void estimate_part(const IndexView &ix, const uint32_t *runs, uint64_t nruns, uint32_t n,
                          const uint16_t *T, uint32_t *seeds, uint64_t cap,
                          unsigned long long *nseeds, uint32_t *err, hipStream_t st) {
    // the settings may lower the sizes held in LDS and registers (0 sends
    // every run down the general paths) and the window size of the register
    // launches (0 hands every run to the last)
    const sdf_tuning &tu = tuning();
    const uint32_t lds_cap = knob(tu.est_lds_cap, 1024), first = knob(tu.est_first_amax, 512);
    const uint32_t reg_cap = std::min<uint32_t>(128, knob(tu.est_reg_cap, 128));
    EstSizes z;
    const uint32_t am[3] = {256, 256, 512}, tm[3] = {256, 512, 1024};
    for (int l = 0; l < 3; l++) {
        z.a[l] = std::min(am[l], first);
        z.t[l] = std::min(tm[l], lds_cap);
    }
    DevBuf<uint32_t> over(nruns);
    DevBuf<unsigned long long> nover(3);
    SDF_HIP(hipMemsetAsync(nover.p, 0, 24, st));
    // a run takes its wave some 14 us, so few runs are spread over the waves the
    // chip holds before any takes several (0.8 Mbp: 1,377 us a call with 32 runs
    // per wave, 471 spread)
    const auto launch = [&](auto kernel, const uint32_t *list, uint64_t m) {
        const uint32_t per = (uint32_t)std::clamp<uint64_t>((m + EWAVES - 1) / EWAVES, 1, ERUNS);
        kernel<<<(unsigned)((m + EW * per - 1) / (EW * per)), EW * 64, 0, st>>>(
            ix, runs, list, m, per, n, T, seeds, cap, nseeds, err, z, over.p, nover.p);
        SDF_HIP(hipGetLastError());
    };
    // hash and index in 32 bits where they fit: half the instructions per exchange of
    // a sort
    const uint32_t hbits = 2 * ix.k;
    launch(hbits + 8 <= 32 ? k_estimate_runs<uint32_t, 0, 256, 256> : k_estimate_runs<uint64_t, 0, 256, 256>,
           nullptr, nruns);
    unsigned long long no[3] = {0, 0, 0};
    {
        Readback rb(st);
        rb.add(no, nover.p, 24);
        rb.wait();
    }
    if (no[0])
        launch(hbits + 9 <= 32 ? k_estimate_runs<uint32_t, 1, 256, 512> : k_estimate_runs<uint64_t, 1, 256, 512>,
               over.p, no[0]);
    uint32_t *const rest = over.p + (nruns - no[1]);
    if (no[1] > no[2])
        launch(hbits + 10 <= 32 ? k_estimate_runs<uint32_t, 2, 512, 1024> : k_estimate_runs<uint64_t, 2, 512, 1024>,
               rest, no[1]);
    if (no[2]) {
        const unsigned grid = (unsigned)((no[1] + EW - 1) / EW);
        k_estimate_long<AMAX_M, TCAP_M, RUN_MID><<<grid, EW * 64, 0, st>>>(
            ix, runs, no[1], rest, n, T, seeds, cap, nseeds, err, std::min<uint32_t>(TCAP_M, lds_cap), reg_cap);
        SDF_HIP(hipGetLastError());
        k_estimate_long<AMAX_L, TCAP_L, RUN_LAST><<<grid, EW * 64, 0, st>>>(
            ix, runs, no[1], rest, n, T, seeds, cap, nseeds, err, std::min<uint32_t>(TCAP_L, lds_cap), reg_cap);
        SDF_HIP(hipGetLastError());
    }
    if (no[0] + no[1]) SDF_HIP(hipStreamSynchronize(st));  // `over` is released on return
}

void launch_estimate_runs(const IndexView &ix, const uint32_t *runs, uint64_t nruns, uint32_t n,
                          const uint16_t *T, uint32_t *seeds, uint64_t cap,
                          unsigned long long *nseeds, uint32_t *err, hipStream_t st) {
    for (uint64_t r = 0; r < nruns; r += RUNS_MAX)
        estimate_part(ix, runs + 6 * r, std::min(RUNS_MAX, nruns - r), n, T, seeds, cap, nseeds, err, st);
}

}  // namespace sdf
