// Seed search (Section 3.1): for every query window [i, i+n) of a span, the
// hits C = {(j, x) in I_G : x in W(G_i)} are gathered from the reverse
// index and the target windows [j, j+n) that share at least tau * s_i
// minimizers are found; the best j of each run of consecutive passing
// targets is a seed.
//
// One workgroup owns a tile: up to `core` consecutive minimizers of the span
// as window starts plus the halo of minimizers the last window reaches.  All
// hits of the tile stay on chip:
//   1. gather: every hit (p, p', o) is loaded once, increments a small counter
//      for its (orientation, target bin of 2^SB >= n bases) in an LDS table
//      indexed by the bin modulo the table size, and the first ones of a lane
//      stay in registers;
//   2. the counters become flags: a slot is hot when some pair of adjacent
//      bins around it holds at least T_min hits;
//   3. a hit is kept only if its slot is hot.  Bins that share a slot only
//      raise counts, so no hit that could matter is dropped (lossless);
//   4. kept hits are sorted in LDS by (o, p', q); exact raw counts decide the
//      target starts x that could pass for some window of the tile, and the
//      hits within 2n of such an x are kept;
//   5. each wave takes windows and walks their candidates in target order,
//      with every window's count of distinct shared hashes kept up to date as
//      hits enter and leave the target window, and runs the run/argmax logic.
// Large tiles split the target coordinate range into partitions processed
// in order (run state of every window is kept across partitions).
//
// What bounds it: on dense indexes (3.1 Gbp: 185 hits per minimizer, 39 G per
// search) the gather's loads and the LDS counters, on sparse ones the latency
// of the phase sequence.  Counters have 4 bits while the tile has many hits
// (131,072 slots in 64 KiB: fewer chance hits in a slot than 16-bit counters
// in a quarter of the slots, so the whole tile fits one partition and every
// list is searched once, in one piece), 8 bits when it has few or when a 4-bit
// counter overflows, 16 bits when an 8-bit one does.  An overflow shows in
// the sum of the counters, taken while they become flags: it equals the
// number of hits counted exactly when none wrapped.
//
// Measured against 16-bit counters in 32 KiB, partitions of 16,384 hits, a
// search per hit for its list and hits gathered twice (tile kernel): 3.1 Gbp
// all-vs-all 538 -> 170 ms, 4,096 spans on 250 Mbp 4.06 -> 1.38 ms, 50 Mbp
// 1.31 -> 0.84 ms.
//
// The file is compiled twice, for two workgroup layouts (SDF_TILE_THREADS):
// 1,024 threads, one workgroup per CU, and 512 threads with 80 KB of LDS, two
// per CU, whose barrier waits overlap each other's work.
#include "kmer.h"
#include "sdf_impl.h"
#include "search.h"

#ifndef SDF_TILE_THREADS
#define SDF_TILE_THREADS 1024
#endif

namespace sdf {
#if SDF_TILE_THREADS == 1024
namespace tile1024 {
constexpr int TB = 1024;        // threads per tile workgroup
constexpr int QCAP = 1280;      // query minimizers per tile (core + halo)
constexpr int CMAX = 1024;      // window starts per tile core
constexpr int CB = 2048;        // kept hits per partition
constexpr uint32_t TLOG = 16;   // bin table of 2^TLOG bytes
constexpr uint32_t HCAP = 65535;  // hits per partition
#elif SDF_TILE_THREADS == 512
namespace tile512 {
constexpr int TB = 512;
constexpr int QCAP = 1024;      // holds any window of up to 1,023 + k bases
constexpr int CMAX = 512;
constexpr int CB = 1024;
constexpr uint32_t TLOG = 15;
constexpr uint32_t HCAP = 32767;
#else
#error "SDF_TILE_THREADS must be 512 or 1024"
#endif
#define SDF_TILE_WAVES_PER_EU 4  // 16 waves per CU: at most 128 VGPRs
constexpr int NWAVES = TB / 64;
constexpr uint32_t TBYTES = 1u << TLOG;
constexpr uint32_t TWORDS = TBYTES / 4;
constexpr uint32_t NCHUNK = (HCAP + 1) / 64;  // 64-hit chunks per partition
constexpr int SBUF = 32;        // seeds buffered per wave before one global atomic
constexpr int STACK = 40;
static_assert(CMAX <= TB && CB % TB == 0 && TBYTES % (16 * TB) == 0, "one pass per thread");

enum : uint32_t { EF_CAND = 1 };
// Packed per kept hit after compaction: its query minimizer, whether it is a
// candidate j owned by the partition with a valid target window, and whether
// the kept hit before it has the same orientation and position.
constexpr uint32_t EI_Q = 0x7FFu;        // bits 0-10
constexpr uint32_t EI_CAND = 1u << 11;
constexpr uint32_t EI_SAMEP = 1u << 12;
static_assert(QCAP <= 2048, "EI_Q field width");
// Flags of a query minimizer: strand and eligibility from the index, whether
// its hits are in the partition's lists, and its mode while a partition covers
// a single window.  Minimizers of one window that share hash and strand have
// the same hits except each one's own position, so their union is the full
// list: the first one stands for all of them with its self-hit kept (union),
// the others are left out (skip).
enum : uint32_t { QF_STRAND = 1, QF_ELIG = 2, QF_LISTED = 4, QF_UNION = 8, QF_SKIP = 16 };
enum : uint32_t {
    ERR_COLLECT = 2,     // (a partition keeps more than CB hits: split, or listed as dense)
    ERR_HITS = 4,        // (a partition has more than HCAP hits: split, or listed as dense)
    ERR_STACK = 8,       // partition splits nested deeper than the stack
    ERR_DENSE_FULL = 16  // more dense windows than the list holds
};

// Kept hits after the gather, over the bin table.
struct PostLds {
    uint32_t hot[CB];       // last hot start at or before an entry, + 1
    uint32_t pref[CB + 1];
    uint32_t etb[CB];       // start of the candidate's sequence
    uint32_t einfo[CB];     // EI_* fields of each kept hit
    uint16_t rng_end[CB];
    uint8_t relf[CB];
    int16_t qnext[QCAP];    // next minimizer of the tile with the same hash, or -1
    uint32_t seeds[NWAVES * SBUF * 6];
};
static_assert(sizeof(PostLds) <= TBYTES, "kept-hit arrays exceed the table area");

struct TileLds {
    union {
        uint4 vec[TBYTES / 16];
        uint32_t table[TWORDS];
        PostLds post;
    } u;
    uint64_t coll[CB];      // kept hits; before the gather: minimizers whose hash repeats
    // the partition's hits in the order of its non-empty lists (one per query
    // minimizer: strand 0, then strand 1): list l holds the hits [h0, h1), at
    // epos[base + e] for hit e (strand 1 at epos[base1 + e] when the strands'
    // pieces are not adjacent)
    uint2 rec[QCAP];        // base, meta: q (11 bits) | strand of q << 11 | first hit of strand 1 << 12
    uint32_t rec1[QCAP];    // base1
    uint64_t marks[NCHUNK]; // bit h0 - 1 of every list but the first
    uint16_t pre[NCHUNK];   // list of the chunk's first hit
    uint32_t qpos[QCAP + 1];
    int16_t qprev[QCAP];    // previous minimizer of the tile with the same hash, or -1
    uint16_t qT[QCAP];      // smallest threshold among the windows holding q (0xFFFF: none)
    uint16_t win_qend[CMAX];
    uint16_t win_s[CMAX];   // sketch size, 0 where no window starts
    uint32_t run_prev[2 * CMAX], run_best[2 * CMAX];  // run state between partitions
    uint16_t run_c[2 * CMAX];                         // 0: no run open
    uint8_t qfl[QCAP];
    uint16_t Tblk[CMAX / 32];     // smallest threshold per 32 window starts
    uint32_t stackA[STACK], stackB[STACK], stackW[STACK];  // W: first window | end << 16
    uint64_t wtmp[NWAVES + 1];
    uint32_t wmin[NWAVES];
    uint64_t ph[PH_N];
    uint32_t tile, ntiles, c0, c1, C, nwin, ncoll, nraw, ndup, dup, csum, nself;
    uint32_t obeg[2], oend[2];
    uint32_t sp;
    uint32_t err;
    uint32_t skip;
    uint32_t qid, qtb;         // query, start of its sequence
    uint32_t next_tile, next_c0, next_c1, next_qid, next_qtb;
    uint64_t next_ge;
    SpanDesc span;             // the span of the tile fetched last,
    uint32_t span_end;         // the first tile past it
    uint32_t span_tb;          // and the start of its sequence
    // work counters of this workgroup, added to the global ones once at exit
    // (global atomics on a handful of shared addresses from every CU serialise)
    unsigned long long cnt[CNT_N];
    uint32_t wseeds[NWAVES];   // seeds buffered per wave, then their offsets
    unsigned long long seed_base;
};
static_assert(sizeof(TileLds) <= (TB == 512 ? 81920 : 163840), "LDS of the workgroups of a CU");

// ----------------------------------------------------------- block helpers --
constexpr int DPP_ROW_SHR = 0x110;      // + n: lane reads lane - n of its row of 16
constexpr int DPP_WAVE_SHR1 = 0x138;    // lane reads lane - 1 of the wave
constexpr int DPP_ROW_BCAST15 = 0x142;  // last lane of each row feeds the next row
constexpr int DPP_ROW_BCAST31 = 0x143;  // lane 31 feeds rows 2 and 3

// Inclusive max-scan over the 64 lanes of a wave with DPP moves: prefix
// within each row of 16, then row 0 into row 1 and row 2 into row 3, then
// rows 0-1 into rows 2-3.  Lanes with no source keep 0, the identity.
__device__ __forceinline__ uint32_t wave_max_scan(uint32_t x) {
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 1, 0xf, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 2, 0xf, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 4, 0xf, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 8, 0xf, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_BCAST15, 0xa, 0xf, false));
    x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_BCAST31, 0xc, 0xf, false));
    return x;
}

// Inclusive sum-scan over the 64 lanes of a wave, the same DPP pattern.
__device__ __forceinline__ uint32_t wave_sum_scan(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 1, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 2, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 4, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_SHR + 8, 0xf, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_BCAST15, 0xa, 0xf, false);
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_ROW_BCAST31, 0xc, 0xf, false);
    return x;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

// In-place exclusive sum over arr[0, n) (n <= 4 * TB); arr[n] = total.
__device__ uint32_t block_scan_u32(uint32_t *arr, int n, uint64_t *wtmp) {
    const int per = (n + TB - 1) / TB;
    const int b = threadIdx.x * per;
    uint32_t s = 0;
    for (int t = 0; t < per; t++)
        if (b + t < n) s += arr[b + t];
    const uint32_t x = wave_sum_scan(s);
    if (lane_id() == 63) wtmp[wave_id()] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t acc = 0;
        for (int w = 0; w < NWAVES; w++) {
            uint64_t t = wtmp[w];
            wtmp[w] = acc;
            acc += t;
        }
        wtmp[NWAVES] = acc;
    }
    __syncthreads();
    uint32_t pre = (uint32_t)wtmp[wave_id()] + x - s;
    for (int t = 0; t < per; t++) {
        if (b + t < n) {
            uint32_t v = arr[b + t];
            arr[b + t] = pre;
            pre += v;
        }
    }
    uint32_t total = (uint32_t)wtmp[NWAVES];
    __syncthreads();
    if (threadIdx.x == 0) arr[n] = total;
    __syncthreads();
    return total;
}

// Inclusive max-scan over arr[0, n) (n <= 2 * TB).
__device__ void block_maxscan_u32(uint32_t *arr, int n, uint64_t *wtmp) {
    const int per = (n + TB - 1) / TB;
    const int b = threadIdx.x * per;
    uint32_t m = 0;
    for (int t = 0; t < per; t++)
        if (b + t < n) m = arr[b + t] > m ? arr[b + t] : m;
    const uint32_t x = wave_max_scan(m);
    if (lane_id() == 63) wtmp[wave_id()] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t acc = 0;
        for (int w = 0; w < NWAVES; w++) {
            uint64_t t = wtmp[w];
            wtmp[w] = acc;
            acc = t > acc ? t : acc;
        }
    }
    __syncthreads();
    uint32_t pre = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, DPP_WAVE_SHR1, 0xf, 0xf, false);
    pre = (uint32_t)wtmp[wave_id()] > pre ? (uint32_t)wtmp[wave_id()] : pre;
    for (int t = 0; t < per; t++) {
        if (b + t < n) {
            pre = arr[b + t] > pre ? arr[b + t] : pre;
            arr[b + t] = pre;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m, 64);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m, 64);
    return ((uint64_t)hi << 32) | lo;
}

// Ascending sort of one key per lane across the wave (bitonic network in
// registers; no barrier).
__device__ __forceinline__ uint64_t wave_sort_u64(uint64_t x) {
    const int lane = lane_id();
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            const uint64_t y = shfl_xor_u64(x, j);
            const bool up = (lane & k) == 0;     // this lane's block of k ascends
            const bool lower = (lane & j) == 0;  // this lane is the lower of its pair
            x = (lower == up) ? (x < y ? x : y) : (x < y ? y : x);
        }
    }
    return x;
}

// Ascending sort of keys[0, n) (n <= CB, keys distinct and below ~0): the
// waves sort runs of 64 keys in registers, then every key is written at its
// rank, its place in its own run plus the keys below it in each other run
// (binary searches in LDS).  Three barriers, against one per stage of a
// bitonic sort over the whole array.  keys[n, 64 ceil(n/64)) is overwritten
// with ~0.
__device__ void block_sort_runs(uint64_t *keys, uint32_t n) {
    const int lane = lane_id(), wave = wave_id();
    const uint32_t R = (n + 63) / 64;
    for (uint32_t r = (uint32_t)wave; r < R; r += NWAVES) {
        const uint32_t e = r * 64 + (uint32_t)lane;
        const uint64_t x = wave_sort_u64(e < n ? keys[e] : ~0ull);
        keys[e] = x;
    }
    __syncthreads();
    constexpr int PER = (CB + TB - 1) / TB;
    uint64_t kv[PER];
    uint32_t rk[PER];
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const uint32_t e = threadIdx.x + (uint32_t)u * TB;
        rk[u] = NONE32;
        kv[u] = 0;
        if (e < n) {
            const uint64_t x = keys[e];
            const uint32_t own = e >> 6;
            uint32_t rank = e & 63u;
            for (uint32_t r = 0; r < R; r++) {
                if (r == own) continue;
                const uint64_t *run = keys + r * 64;
                uint32_t lo = 0, hi = 64;
                while (lo < hi) {
                    const uint32_t m = (lo + hi) >> 1;
                    if (run[m] < x) lo = m + 1; else hi = m;
                }
                rank += lo;
            }
            kv[u] = x;
            rk[u] = rank;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; u++)
        if (rk[u] != NONE32) keys[rk[u]] = kv[u];
    __syncthreads();
}

// Entries of I_G^{-1} for a hash: strand 0 at [lo, mid), strand 1 at [mid, hi).
__device__ __forceinline__ void lookup(const IndexView &ix, uint32_t hash, uint32_t &lo,
                                       uint32_t &mid, uint32_t &hi) {
    const uint64_t key = (uint64_t)hash << 1;
    const uint64_t d = key >> ix.dir_shift;
    lo = ix.dir[d];
    mid = ix.dir[d + 1];
    if (ix.dir_shift == 0) {
        hi = ix.dir[d + 2];
        return;
    }
    // both keys share the directory entry: their low bits within it
    const uint32_t low = (uint32_t)(key & ((1ull << ix.dir_shift) - 1));
    const uint32_t end = mid;
    auto first = [&](uint32_t from, uint32_t bits) {  // first entry >= bits
        uint32_t a = from, b = end;
        while (a < b) {
            const uint32_t m = (a + b) >> 1;
            if (ix.ekeylo[m] < bits) a = m + 1; else b = m;
        }
        return a;
    };
    lo = first(lo, low);
    mid = first(lo, low + 1);
    hi = first(mid, low + 2);
}

// First entries of the ascending positions epos[lo, hi) that are >= x0 and
// >= x1.  The index keeps every ESAMP-th position (esamp[s] = epos[ESAMP s],
// one 128-byte line of epos per sample), so a search finds its line among
// the samples inside [lo, hi) and then its entry inside that line: two lines
// read from memory, the other probes hit the first-level cache.  The two
// searches are interleaved so that their loads overlap.
__device__ __forceinline__ void lower_pos2(const IndexView &ix, uint32_t lo, uint32_t hi,
                                           uint64_t x0, uint64_t x1, uint32_t &r0, uint32_t &r1) {
    const uint32_t s_lo = (lo + ESAMP - 1) / ESAMP, s_hi = (hi + ESAMP - 1) / ESAMP;
    uint32_t a0 = s_lo, b0 = s_hi, a1 = s_lo, b1 = s_hi;  // first sample >= x
    while (a0 < b0 || a1 < b1) {
        const uint32_t m0 = (a0 + b0) >> 1, m1 = (a1 + b1) >> 1;
        const uint32_t v0 = a0 < b0 ? ix.esamp[m0] : 0u;
        const uint32_t v1 = a1 < b1 ? ix.esamp[m1] : 0u;
        if (a0 < b0) {
            if ((uint64_t)v0 < x0) a0 = m0 + 1; else b0 = m0;
        }
        if (a1 < b1) {
            if ((uint64_t)v1 < x1) a1 = m1 + 1; else b1 = m1;
        }
    }
    // the entry lies after the last sample below x and up to the first
    // sample at or above it
    uint32_t c0 = a0 > s_lo ? (a0 - 1) * ESAMP + 1 : lo;
    uint32_t d0 = min(hi, a0 * ESAMP);
    uint32_t c1 = a1 > s_lo ? (a1 - 1) * ESAMP + 1 : lo;
    uint32_t d1 = min(hi, a1 * ESAMP);
    while (c0 < d0 || c1 < d1) {
        const uint32_t m0 = (c0 + d0) >> 1, m1 = (c1 + d1) >> 1;
        const uint32_t v0 = c0 < d0 ? ix.epos[m0] : 0u;
        const uint32_t v1 = c1 < d1 ? ix.epos[m1] : 0u;
        if (c0 < d0) {
            if ((uint64_t)v0 < x0) c0 = m0 + 1; else d0 = m0;
        }
        if (c1 < d1) {
            if ((uint64_t)v1 < x1) c1 = m1 + 1; else d1 = m1;
        }
    }
    r0 = c0;
    r1 = c1;
}

// Packed kept-hit key: o (1 bit) | p' (32 bits) | q (11 bits).
__device__ __forceinline__ uint64_t ckey(uint32_t o, uint32_t p, uint32_t q) {
    return ((uint64_t)o << 43) | ((uint64_t)p << 11) | q;
}
__device__ __forceinline__ uint32_t ck_o(uint64_t k) { return (uint32_t)(k >> 43); }
__device__ __forceinline__ uint32_t ck_p(uint64_t k) { return (uint32_t)(k >> 11); }
__device__ __forceinline__ uint32_t ck_q(uint64_t k) { return (uint32_t)(k & 2047); }
__device__ __forceinline__ uint64_t ck_op(uint64_t k) { return k >> 11; }

__device__ __forceinline__ uint32_t lanes_below(uint64_t m, uint32_t add) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, add));
}
__device__ __forceinline__ uint32_t uni(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint32_t lane_read(uint32_t x, uint32_t l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, (int)l);
}

// A value the compiler does not see through: addresses made from it are
// computed where they are used, not hoisted out of the tile loop and spilled.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// The kernel's arguments, read again from where this is called (scalar loads
// that hit the constant cache): held in registers over the whole tile loop they
// spill.  They are the kernel's first and only parameter.
__device__ __forceinline__ const SearchArgs &kernel_args() {
    auto p = (const __attribute__((address_space(4))) SearchArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const SearchArgs *)p;
}

// The list of hit e (marks and pre of its chunk): lists that start at or
// before it, less one.
__device__ __forceinline__ uint32_t list_of(const TileLds &L, uint32_t e) {
    const uint64_t m = L.marks[e >> 6] & ((1ull << (e & 63)) - 1);
    return L.pre[e >> 6] + (uint32_t)__popcll(m);
}

constexpr int HU = 8;  // chunks gathered per round: their loads are all in flight together
// Rounds whose hits stay in registers (24 per lane); those of later rounds are
// gathered again.  More of them spill: 6 rounds wrote 224 GB of scratch per
// 3.1 Gbp search (tile kernel 206, 197, 176, 170, 173 ms at 6, 5, 4, 3, 2
// rounds; 4,096 spans 1.63, 1.61, 1.51, 1.38, 1.48 ms; 50 Mbp 0.95, 0.95, 0.90,
// 0.84, 0.85 ms).
constexpr int SG = 3;

// Hits of the chunks [c, c + HU): pv = target position, bit u of the result =
// orientation.  Lists and chunks are exact, so every load is in range; lanes
// past the last hit repeat it.
__device__ __forceinline__ uint32_t gather_hits(const TileLds &L, const uint32_t *epos, uint32_t H,
                                                uint32_t nch, bool pieces, uint32_t c,
                                                uint32_t lane, uint32_t (&pv)[HU]) {
    uint32_t ob = 0;
    uint32_t at[HU];
#pragma unroll
    for (int u = 0; u < HU; u++) {
        const uint32_t cc = min(c + (uint32_t)u, nch - 1);
        const uint32_t l = lanes_below(L.marks[cc], L.pre[cc]);
        const uint32_t e = min(cc * 64 + lane, H - 1);
        const uint2 r = L.rec[l];
        const uint32_t b = e >= (r.y >> 12) ? 1u : 0u;
        at[u] = (pieces && b ? L.rec1[l] : r.x) + e;
        ob |= (b ^ ((r.y >> 11) & 1)) << u;
    }
#pragma unroll
    for (int u = 0; u < HU; u++) pv[u] = epos[at[u]];
    return ob;
}

// A window the tile cannot hold goes to the list of dense windows (once)
// and takes no further part in this tile.
__device__ __forceinline__ void list_dense(const SearchArgs &a, TileLds &L, uint32_t m) {
    const unsigned long long d = atomicAdd(&a.counters[CNT_DENSE], 1ull);
    if (d < a.dense_cap) a.dense[d] = ((uint64_t)L.qid << 32) | m;
    else L.err |= ERR_DENSE_FULL;
}

// Push the halves of an over-full partition [A, B) x windows [WA, WB): by
// target while it spans more than 4n bases, else by window starts; the
// lower half goes on top.  A single window that cannot be split further is
// listed as dense.
__device__ __forceinline__ void split_partition(const SearchArgs &a, TileLds &L, uint32_t A,
                                                uint32_t B, uint32_t WA, uint32_t WB, uint32_t n) {
    if (L.sp + 2 > STACK) {
        L.err |= ERR_STACK;
    } else if ((uint64_t)B - A > 4ull * n) {
        const uint32_t mid = A + (B - A) / 2, W = WA | (WB << 16);
        L.stackA[L.sp] = mid; L.stackB[L.sp] = B; L.stackW[L.sp] = W; L.sp++;
        L.stackA[L.sp] = A; L.stackB[L.sp] = mid; L.stackW[L.sp] = W; L.sp++;
    } else if (WB - WA > 1) {
        const uint32_t mid = WA + (WB - WA) / 2;
        L.stackA[L.sp] = A; L.stackB[L.sp] = B; L.stackW[L.sp] = mid | (WB << 16); L.sp++;
        L.stackA[L.sp] = A; L.stackB[L.sp] = B; L.stackW[L.sp] = WA | (mid << 16); L.sp++;
    } else if (L.win_s[WA]) {
        list_dense(a, L, L.c0 + WA);
        L.win_s[WA] = 0;  // no candidates, no runs: its seeds come from the dense pass
    }
}

// ------------------------------------------------------------ tile kernel --
// Optional phase breakdown: thread 0 reads the wall clock after the barrier
// that ends each phase and accumulates the difference.
#define PHASE(id)                                                       \
    do {                                                                \
        if (prof) {                                                     \
            const uint64_t now_ = wall_clock64();                       \
            L.ph[id] += now_ - ph_t;                                    \
            ph_t = now_;                                                \
        }                                                               \
    } while (0)

// Per-wave seed buffer (LDS) flushed with one global atomic per batch.
struct SeedBuf {
    uint32_t *buf;  // SBUF * 6 words of this wave
    uint32_t n;     // wave-uniform
};

__device__ __forceinline__ void seeds_flush(const SearchArgs &a, SeedBuf &sb, int lane) {
    if (sb.n == 0) return;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(&a.counters[CNT_SEEDS], (unsigned long long)sb.n);
    base = __shfl(base, 0, 64);
    for (uint32_t t = lane; t < sb.n * 6; t += 64) {
        const unsigned long long idx = base + t / 6;
        if (idx < a.seed_cap) a.seeds[base * 6 + t] = sb.buf[t];
    }
    __builtin_amdgcn_wave_barrier();
    sb.n = 0;
}

// Every lane with `mine` set pushes one seed; order within the buffer does
// not matter (seeds are sorted afterwards).
__device__ __forceinline__ void seeds_push_lanes(const SearchArgs &a, SeedBuf &sb, int lane,
                                                 bool mine, uint32_t qid, uint32_t i, uint32_t j,
                                                 uint32_t o, uint32_t c, uint32_t s) {
    const uint64_t m = __ballot(mine);
    const uint32_t cnt = (uint32_t)__popcll(m);
    if (cnt == 0) return;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t rank = (uint32_t)__popcll(m & lt);
    if (sb.n + cnt > SBUF) seeds_flush(a, sb, lane);
    if (cnt > SBUF) {  // too many for the buffer: write directly
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(&a.counters[CNT_SEEDS], (unsigned long long)cnt);
        base = __shfl(base, 0, 64);
        if (mine && base + rank < a.seed_cap) {
            uint32_t *d = a.seeds + (base + rank) * 6;
            d[0] = qid; d[1] = i; d[2] = j; d[3] = o; d[4] = c; d[5] = s;
        }
        return;
    }
    if (mine) {
        uint32_t *d = sb.buf + (sb.n + rank) * 6;
        d[0] = qid; d[1] = i; d[2] = j; d[3] = o; d[4] = c; d[5] = s;
    }
    __builtin_amdgcn_wave_barrier();
    sb.n += cnt;
}

// All waves of the workgroup write their buffered seeds with one global
// atomic for the workgroup (every wave must call it: it holds barriers).
__device__ __forceinline__ void seeds_flush_block(const SearchArgs &a, TileLds &L, SeedBuf &sb,
                                                  int lane, int wave) {
    if (lane == 0) L.wseeds[wave] = sb.n;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0;
        for (int w = 0; w < NWAVES; w++) {
            const uint32_t c = L.wseeds[w];
            L.wseeds[w] = tot;
            tot += c;
        }
        L.seed_base = tot ? atomicAdd(&a.counters[CNT_SEEDS], (unsigned long long)tot) : 0ull;
    }
    __syncthreads();
    const unsigned long long base = L.seed_base + L.wseeds[wave];
    for (uint32_t t = lane; t < sb.n * 6; t += 64) {
        const unsigned long long idx = base + t / 6;
        if (idx < a.seed_cap) a.seeds[base * 6 + t] = sb.buf[t];
    }
    sb.n = 0;
}

// Hot flags of four adjacent table words at once: bit 0 of every counter field
// says whether some pair of adjacent slots among (slot - 2, slot - 1),
// (slot - 1, slot), (slot, slot + 1) sums to at least T.  pw and nw are the
// words before and after w; `sum` gains the counters of w.
__device__ __forceinline__ uint32_t hot_nibbles(uint32_t pw, uint32_t w, uint32_t nw, uint32_t T,
                                                uint32_t &sum) {
    const uint32_t K = 0x01010101u * (0x80u - T);
    const uint32_t E = w & 0x0F0F0F0Fu, O = (w >> 4) & 0x0F0F0F0Fu;
    const uint32_t Se = E + O;                                     // pairs starting at 0, 2, 4, 6
    const uint32_t So = O + ((E >> 8) | ((nw & 15u) << 24));       // at 1, 3, 5, 7
    sum = __builtin_amdgcn_sad_u8(Se, 0u, sum);
    const uint32_t he = ((Se + K) & 0x80808080u) >> 7, ho = ((So + K) & 0x80808080u) >> 7;
    const uint32_t pe = ((pw >> 28) + ((pw >> 24) & 15u)) >= T ? 1u : 0u;  // at -2
    const uint32_t po = ((pw >> 28) + (w & 15u)) >= T ? 1u : 0u;           // at -1
    const uint32_t bo = (ho << 8) | po;
    return (((he << 8) | pe) | bo | he) | ((bo | he | ho) << 4);
}
__device__ __forceinline__ uint32_t hot_bytes(uint32_t pw, uint32_t w, uint32_t nw, uint32_t T,
                                              uint32_t &sum) {
    const uint32_t K = 0x00010001u * (0x8000u - T);
    const uint32_t E = w & 0x00FF00FFu, O = (w >> 8) & 0x00FF00FFu;
    const uint32_t Se = E + O, So = O + ((E >> 16) | ((nw & 255u) << 16));
    sum = __builtin_amdgcn_sad_u8(w, 0u, sum);
    const uint32_t he = ((Se + K) & 0x80008000u) >> 15, ho = ((So + K) & 0x80008000u) >> 15;
    const uint32_t pe = ((pw >> 24) + ((pw >> 16) & 255u)) >= T ? 1u : 0u;
    const uint32_t po = ((pw >> 24) + (w & 255u)) >= T ? 1u : 0u;
    const uint32_t bo = (ho << 16) | po;
    return (((he << 16) | pe) | bo | he) | ((bo | he | ho) << 8);
}

// Table slot of position p and orientation o: the bin modulo half the table,
// so that adjacent bins are adjacent slots.  hl: log2 of the half's slots.
__device__ __forceinline__ uint32_t slot_of(uint32_t p, uint32_t o, uint32_t SB, uint32_t hl) {
    return ((p >> SB) & ((1u << hl) - 1u)) | (o << hl);
}

// Open run of a window and orientation.
struct RunState {
    uint32_t prev_j, best_j, best_c;  // best_c 0: none
};
// 64 window starts and an orientation, one window per lane: its minimizers are
// [qc, qc + len), len 0 where no window starts; together they lie in [qlo, qhi).
struct Block {
    uint32_t qlo, qhi, o;
    uint32_t qc, len, i, si, Ti;
    uint32_t near;      // X - 1 of the excluded overlaps
    bool runs_out;      // first and last candidate of each run instead of its seed
};
// A candidate: its position, the least previous candidate that a run links to
// (its sequence's start and less than n back), and for the excluded overlaps
// with the window itself |j - i| < X the range 2X - 1 (0: another sequence).
struct Cand {
    uint32_t j, lo, kx;
};
__device__ __forceinline__ Cand candidate(const SearchArgs &a, const TileLds &L, uint32_t e) {
    Cand c;
    c.j = ck_p(L.coll[e]);
    const uint32_t tb = L.u.post.etb[e];
    c.lo = max(tb, c.j >= a.n - 1 ? c.j - (a.n - 1) : 0u);
    c.kx = tb == L.qtb ? 2 * (a.n - a.max_overlap) - 1 : 0u;
    return c;
}

// Seeds of runs that ended, one per lane at most, until they are pushed
// together (most windows have one run): lanes in m hold (j, v).
struct EndedRuns {
    uint64_t m;
    uint32_t j, v;
};
__device__ __forceinline__ void push_ended(const SearchArgs &a, TileLds &L, SeedBuf &sbuf,
                                           const Block &bk, EndedRuns &er, uint32_t lane) {
    seeds_push_lanes(a, sbuf, (int)lane, (er.m >> lane) & 1, L.qid, bk.i, er.j, bk.o, er.v, bk.si);
    er.m = 0;
}

// Run logic of one candidate: a passing candidate continues the open run when
// it lies in its sequence less than n after the previous candidate; a run's
// seed is its largest count, earliest j on ties.  With runs_out a run gives
// its first and last candidate (the previous one) for the estimate.
__device__ __forceinline__ void run_step(const SearchArgs &a, TileLds &L, SeedBuf &sbuf,
                                         const Block &bk, RunState &rs, EndedRuns &er,
                                         uint32_t lane, bool mine, uint32_t cnt, uint32_t j,
                                         uint32_t lo, uint32_t kx) {
    // (& and |, not && and ||: no branches)
    const bool open = rs.best_c != 0;
    const bool pass = mine & (cnt >= bk.Ti) & (j + bk.near - bk.i >= kx);
    const bool link = pass & open & (rs.prev_j >= lo);
    const bool ends = mine & open & !link;
    const uint64_t em = __builtin_amdgcn_ballot_w64(ends);
    if (em & er.m) push_ended(a, L, sbuf, bk, er, lane);
    er.m |= em;
    er.j = ends ? rs.best_j : er.j;
    er.v = ends ? (bk.runs_out ? rs.prev_j : rs.best_c) : er.v;
    const bool upd = pass & (!link | (!bk.runs_out & (cnt > rs.best_c)));
    rs.best_c = upd ? cnt : (mine & !pass) ? 0u : rs.best_c;
    rs.best_j = upd ? j : rs.best_j;
    rs.prev_j = mine ? j : rs.prev_j;
}

// Candidates among the kept hits [ob, oe) against the windows of a block whose
// minimizers fit R per lane.  Lane l holds for each of its minimizers
// qlo + 64 r + l the last of its hits that has entered (every hit up to
// j + n - k has entered before candidate j): one at or past the candidate means
// that the minimizer has a hit in [j, j + n - k], so a ballot per r is the
// candidate's bitmask over the block's minimizers, and a window's count the
// popcount of it over the window's own.  DUP: a hash repeats within the tile.
// Each lane then looks for the earlier ones of its own minimizers (four arrays of
// 30 kbp with units of 350 bases: 148 ms a search, 319 with one look at a time,
// 199 with a wave per window); a form of its own, as other tiles ran 1.5%
// slower with it in theirs.
template <int R, bool DUP>
__device__ __forceinline__ void eval_masks(const SearchArgs &a, TileLds &L, SeedBuf &sbuf,
                                           const Block &bk, RunState &rs, EndedRuns &er,
                                           uint32_t ob, uint32_t oe,
                                           uint32_t lane, uint32_t &n_evals,
                                           uint32_t &n_scan) {
    const PostLds &F = L.u.post;
    const uint32_t qlo = bk.qlo, nq = bk.qhi - bk.qlo;
    uint64_t wm[R];  // the window's minimizers
    uint32_t last[R] = {};  // hit + 1
    uint64_t again[R] = {};  // (with repeats) minimizers with an earlier one of their hash in the block
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int from = (int)lane - 64 * r, to = (int)(lane + bk.len) - 64 * r;
        uint64_t m = from <= 0 ? ~0ull : from < 64 ? ~0ull << from : 0ull;
        if (to < 64) m = to <= 0 ? 0ull : m & ((1ull << to) - 1);
        wm[r] = m;
        const uint32_t q = lane + 64 * r;
        if (DUP) again[r] = __builtin_amdgcn_ballot_w64(q < nq && L.qprev[min(qlo + q, (uint32_t)QCAP - 1)] >= (int)qlo);
    }
    // the next hit to enter, its chunk, the chunk's minimizers and the hits of it
    // still to enter
    uint32_t next = NONE32, fc = ob & ~63u, frl = 0;
    uint64_t frel = 0;
    auto chunk_of_next = [&]() {
        for (;; fc += 64) {
            if (fc >= oe) {
                next = NONE32;
                return;
            }
            const uint32_t fx = fc + lane;
            frl = fx >= ob && fx < oe ? (F.einfo[fx] & EI_Q) - qlo : NONE32;
            frel = __builtin_amdgcn_ballot_w64(frl < nq);
            if (frel) break;
        }
        next = fc + (uint32_t)__builtin_ctzll(frel);
    };
    chunk_of_next();
    uint32_t carry_q = EI_Q;  // minimizer of the hit before the chunk
    for (uint32_t e0 = ob & ~63u; e0 < oe; e0 += 64) {
        n_scan++;
        const uint32_t ex = e0 + lane;
        const bool valid = ex >= ob && ex < oe;
        const uint32_t info = valid ? F.einfo[ex] : 0u;
        const uint32_t qx = info & EI_Q;
        const bool cand = valid && (info & EI_CAND) && qx - qlo < nq;
        uint64_t mm = __ballot(cand);
        const uint32_t pq = (uint32_t)__builtin_amdgcn_update_dpp((int)carry_q, (int)qx, DPP_WAVE_SHR1,
                                                                  0xf, 0xf, false);
        carry_q = lane_read(qx, 63);
        if (!mm) continue;
        // the window's first hit at this position: the one before lies outside it
        const uint32_t pq1 = (info & EI_SAMEP) ? pq + 1 : 0u;
        Cand c{0, 0, 0};
        uint32_t pend = 0;
        if (cand) {
            c = candidate(a, L, ex);
            pend = F.rng_end[ex];
        }
        while (mm) {
            const uint32_t bb = (uint32_t)__ffsll((long long)mm) - 1;
            mm &= mm - 1;
            const uint32_t e = e0 + bb;
            const uint32_t q = lane_read(qx, bb);
            const bool mine = (q - bk.qc < bk.len) & (bk.qc >= lane_read(pq1, bb));
            const uint64_t mb = __builtin_amdgcn_ballot_w64(mine);
            if (!mb) continue;
            n_evals += (uint32_t)__popcll(mb);
            const uint32_t re = lane_read(pend, bb);
            while (next < re) {
                const uint32_t rel = lane_read(frl, next & 63);
#pragma unroll
                for (int r = 0; r < R; r++) last[r] = lane + 64 * r == rel ? next + 1 : last[r];
                frel &= frel - 1;
                if (frel) {
                    next = fc + (uint32_t)__builtin_ctzll(frel);
                } else {
                    fc += 64;
                    chunk_of_next();
                }
            }
            uint64_t M[R];
            uint32_t cnt = 0;
#pragma unroll
            for (int r = 0; r < R; r++) {
                M[r] = __builtin_amdgcn_ballot_w64(last[r] > e);
                cnt += (uint32_t)__popc((uint32_t)M[r] & (uint32_t)wm[r]);
                cnt += (uint32_t)__popc((uint32_t)(M[r] >> 32) & (uint32_t)(wm[r] >> 32));
            }
            uint64_t rep = 0;  // (again[] is empty without repeats)
#pragma unroll
            for (int r = 0; r < R; r++) rep |= M[r] & again[r];
            if (rep) {
                // a marked minimizer that repeats the hash of an earlier marked one
                // does not count in the windows that hold the nearest such one too:
                // each lane looks for that of its own minimizers
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const uint64_t am = M[r] & again[r];
                    if (!am) continue;
                    int x = (am >> lane) & 1 ? (int)L.qprev[qlo + 64 * r + lane] : -1;
                    while (x >= (int)qlo) {
                        const uint32_t rx = (uint32_t)x - qlo, half = rx >> 5;
                        uint32_t m = 0;
#pragma unroll
                        for (int v = 0; v < 2 * R; v++) m = half == (uint32_t)v ? (uint32_t)(M[v / 2] >> (32 * (v & 1))) : m;
                        if ((m >> (rx & 31)) & 1) break;
                        x = L.qprev[x];
                    }
                    for (uint64_t dm = __builtin_amdgcn_ballot_w64(x >= (int)qlo); dm; dm &= dm - 1) {
                        const uint32_t l = (uint32_t)__builtin_ctzll(dm);
                        if (qlo + 64 * r + l < bk.qc + bk.len && lane_read((uint32_t)x, l) >= bk.qc) cnt--;
                    }
                }
            }
            run_step(a, L, sbuf, bk, rs, er, lane, mine, cnt, lane_read(c.j, bb), lane_read(c.lo, bb),
                     lane_read(c.kx, bb));
        }
    }
}

// A window's shared count changes when a minimizer of it gets its first kept
// hit in the target window or loses its last one.  With repeated hashes a
// window holding another marked minimizer of the same hash does not change:
// nearest marked ones before (a) and after (b).
struct Marks {
    uint32_t live, multi;  // lane l, bit r: minimizer qlo + 64 r + l has one kept hit, or several
};
static_assert(QCAP <= 64 * 32, "mark bits of a lane");
__device__ __forceinline__ bool mark_counts(const TileLds &L, const Marks &m, const Block &bk,
                                            uint32_t q, bool dup) {
    bool in = q - bk.qc < bk.len;
    if (dup) {
        const int qlo = (int)bk.qlo, qhi = (int)bk.qhi;
        auto live = [&](int r) {
            return (lane_read(m.live, (uint32_t)(r - qlo) & 63u) >> ((uint32_t)(r - qlo) >> 6)) & 1u;
        };
        int a = (int)uni((uint32_t)(int)L.qprev[q]);
        while (a >= qlo && !live(a)) a = (int)uni((uint32_t)(int)L.qprev[a]);
        int b = (int)uni((uint32_t)(int)L.u.post.qnext[q]);
        while (b >= 0 && b < qhi && !live(b)) b = (int)uni((uint32_t)(int)L.u.post.qnext[b]);
        if (a >= qlo) in = in && (uint32_t)a < bk.qc;
        if (b >= 0 && b < qhi) in = in && (uint32_t)b >= bk.qc + bk.len;
    }
    return in;
}

// The same as eval_masks for any number of minimizers.
__device__ __forceinline__ void eval_events(const SearchArgs &a, TileLds &L, SeedBuf &sbuf,
                                            const Block &bk, RunState &rs, EndedRuns &er,
                                           uint32_t ob, uint32_t oe,
                                            uint32_t lane, bool dup, uint32_t &n_evals,
                                            uint32_t &n_scan) {
    const PostLds &F = L.u.post;
    const uint32_t qlo = bk.qlo, nq = bk.qhi - bk.qlo;
    Marks mk{0, 0};
    uint32_t cnt = 0;
    uint32_t f = ob, fc = NONE32, fq = 0;  // next hit to enter; its chunk
    uint64_t frel = 0;
    uint32_t carry_q = EI_Q;  // minimizer of the hit before the chunk
    for (uint32_t e0 = ob & ~63u; e0 < oe; e0 += 64) {
        n_scan++;
        const uint32_t ex = e0 + lane;
        const bool valid = ex >= ob && ex < oe;
        const uint32_t info = valid ? F.einfo[ex] : 0u;
        const uint32_t qx = info & EI_Q;
        // hits whose minimizer lies in one of the block's windows
        const bool rel = valid && qx - qlo < nq;
        uint64_t mm = __ballot(rel);
        uint32_t pq = (uint32_t)__builtin_amdgcn_update_dpp((int)carry_q, (int)qx, DPP_WAVE_SHR1, 0xf,
                                                            0xf, false);
        carry_q = lane_read(qx, 63);
        if (!mm) continue;
        const uint32_t pq1 = (info & EI_SAMEP) ? pq + 1 : 0u;
        Cand c{0, 0, 0};
        uint32_t pend = 0;
        if (rel && (info & EI_CAND)) {
            c = candidate(a, L, ex);
            pend = F.rng_end[ex];
        }
        while (mm) {
            const uint32_t bb = (uint32_t)__ffsll((long long)mm) - 1;
            mm &= mm - 1;
            const uint32_t e = e0 + bb;
            const uint32_t ie = lane_read(info, bb);
            const uint32_t q = ie & EI_Q;
            const bool mine = (ie & EI_CAND) && q - bk.qc < bk.len && bk.qc >= lane_read(pq1, bb);
            const uint64_t mb = __ballot(mine);
            if (mb) {
                n_evals += (uint32_t)__popcll(mb);
                const uint32_t re = lane_read(pend, bb);
                if (f < e) f = e;  // hits passed before they entered
                while (f < re) {
                    if ((f & ~63u) != fc) {
                        fc = f & ~63u;
                        const uint32_t fx = fc + lane;
                        fq = fx < oe ? (F.einfo[fx] & EI_Q) : 0u;
                        frel = __ballot(fx < oe && fq - qlo < nq);
                    }
                    const uint32_t end = min(re, fc + 64);
                    uint64_t m2 = frel & (~0ull << (f & 63));
                    if (end < fc + 64) m2 &= (1ull << (end & 63)) - 1;
                    while (m2) {
                        const uint32_t b2 = (uint32_t)__ffsll((long long)m2) - 1;
                        m2 &= m2 - 1;
                        const uint32_t eq = lane_read(fq, b2);
                        const uint32_t ln = (eq - qlo) & 63u, bit = 1u << ((eq - qlo) >> 6);
                        const uint32_t cur = lane_read(mk.live, ln), mul = lane_read(mk.multi, ln);
                        if (cur & bit) {
                            mk.multi = lane == ln ? mul | bit : mk.multi;
                        } else {
                            cnt += mark_counts(L, mk, bk, eq, dup) ? 1u : 0u;
                            mk.live = lane == ln ? cur | bit : mk.live;
                        }
                    }
                    f = end;
                }
                run_step(a, L, sbuf, bk, rs, er, lane, mine, cnt, lane_read(c.j, bb), lane_read(c.lo, bb),
                         lane_read(c.kx, bb));
            }
            if (e < f) {  // hit e leaves
                const uint32_t ln = (q - qlo) & 63u, bit = 1u << ((q - qlo) >> 6);
                const uint32_t cur = lane_read(mk.live, ln), mul = lane_read(mk.multi, ln);
                uint32_t others = 0;
                if (mul & bit) {  // others of its minimizer among the entered
                    for (uint32_t g = e + 1; g < f; g += 64) {
                        const uint32_t gx = g + lane;
                        others += (uint32_t)__popcll(__ballot(gx < f && (F.einfo[gx] & EI_Q) == q));
                    }
                    if (others < 2) mk.multi = lane == ln ? mul & ~bit : mk.multi;
                }
                if (!others) {
                    mk.live = lane == ln ? cur & ~bit : mk.live;
                    cnt -= mark_counts(L, mk, bk, q, dup) ? 1u : 0u;
                }
            }
        }
    }
}

// Tile t of the queue and its span, into the next_* fields (by one wave, t the
// same in all lanes).  Consecutive tiles mostly stay in the span kept in LDS;
// otherwise the lanes probe 64 spans per round for the last one that starts
// at or before t.
__device__ __forceinline__ void next_tile(const SearchArgs &a, TileLds &L, uint32_t t, uint32_t lane) {
    if (t < L.ntiles && (t < L.span.tile0 || t >= L.span_end)) {
        uint32_t lo = 0, hi = a.nspans;
        while (hi - lo > 1) {
            const uint32_t step = (hi - lo + 63) / 64, p = lo + lane * step;
            const bool le = p < hi && a.spans[p].tile0 <= t;  // a prefix of the lanes
            const uint32_t c = max((uint32_t)__popcll(__ballot(le)), 1u);
            const uint32_t nhi = min(hi, lo + c * step);
            lo += (c - 1) * step;
            hi = nhi;
        }
        const uint32_t end = lo + 1 < a.nspans ? a.spans[lo + 1].tile0 : L.ntiles;
        const SpanDesc sd = a.spans[lo];
        if (lane == 0) {
            L.span = sd;
            L.span_end = end;
            L.span_tb = (uint32_t)a.ix.off[sd.qseq];
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) {
        L.next_tile = t;
        if (t < L.ntiles) {
            L.next_c0 = L.span.m_lo + (t - L.span.tile0) * a.core;
            L.next_c1 = min(L.next_c0 + a.core, L.span.m_hi);
            L.next_ge = L.span.ge;
            L.next_qid = L.span.qid;
            L.next_qtb = L.span_tb;
        }
    }
}

__global__ void __launch_bounds__(TB) __attribute__((amdgpu_waves_per_eu(SDF_TILE_WAVES_PER_EU)))
k_tile_search(SearchArgs) {
    __shared__ TileLds L;
    const uint32_t n = kernel_args().n, k = kernel_args().ix.k;
    const uint32_t wave = uni(wave_id());
    const bool prof = kernel_args().phase != nullptr && threadIdx.x == 0;
    if (threadIdx.x < PH_N) L.ph[threadIdx.x] = 0;
    if (threadIdx.x < CNT_N) L.cnt[threadIdx.x] = 0;
    uint64_t ph_t = prof ? wall_clock64() : 0;
    if (wave == NWAVES - 1) {
        const uint32_t lane = threadIdx.x & 63;
        if (lane == 0) {
            L.ntiles = *kernel_args().total_tiles;
            L.span.tile0 = 0;
            L.span_end = 0;  // no span kept yet
        }
        __builtin_amdgcn_wave_barrier();
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(kernel_args().work, 1u);
        next_tile(kernel_args(), L, uni(t), lane);
    }
    constexpr int QR = (QCAP + TB) / TB;  // minimizers per thread, the sentinel included

    for (;;) {
        __syncthreads();  // next_* written, everything of the previous tile read
        if (L.next_tile >= L.ntiles) break;
        // A tile core may be processed in several pieces when its windows
        // reach more minimizers than fit on chip.
        uint32_t c_begin = L.next_c0;
        const uint32_t piece_end = L.next_c1;
        const uint64_t ge = L.next_ge;
        const uint32_t qid = L.next_qid, qtb = L.next_qtb;
        // the next tile's number, asked for here and used by the last wave in the
        // window phase, where it has the least to do
        uint32_t ticket = NONE32;
        if (threadIdx.x == TB - 64) ticket = atomicAdd(kernel_args().work, 1u);
        __syncthreads();
        if (threadIdx.x == 0) {
            L.qid = qid;
            L.qtb = qtb;
        }
        bool first_piece = true;
        while (c_begin < piece_end) {
            const uint32_t tid = opaque(threadIdx.x), lane = tid & 63;
            const SearchArgs &a = kernel_args();
            const IndexView &ix = a.ix;
            // ---- query minimizers of the tile: all loads at once, the
            // directory entries of the eligible ones behind their hashes ----
            uint32_t C = piece_end - c_begin;
            uint32_t qn = min(C + a.halo, (uint32_t)QCAP + 1);  // loaded, at least core + 1
            uint32_t hash[QR];
            uint32_t mext = 0;
            if (tid == 0) {
                L.ndup = 0;
                L.dup = 0;
                L.nwin = 0;
                L.err = 0;
                L.skip = 0;
                L.c0 = c_begin;
            }
            if (tid < C) mext = ix.mext[c_begin + tid];
            uint16_t *dups = reinterpret_cast<uint16_t *>(L.coll);
            static_assert(sizeof(uint16_t) * QCAP <= sizeof(uint64_t) * CB, "dups in coll");
            for (;;) {
                __syncthreads();  // ndup and dup cleared
#pragma unroll
                for (int r = 0; r < QR; r++) {
                    const uint32_t q = tid + (uint32_t)r * TB;
                    const uint64_t m = (uint64_t)c_begin + q;
                    hash[r] = 0;
                    if (q >= qn) continue;
                    if (m >= ix.nm) {
                        L.qpos[q] = 0xFFFFFFFFu;
                        if (q < QCAP) {
                            L.qfl[q] = 0;
                            L.qprev[q] = -1;
                        }
                        continue;
                    }
                    L.qpos[q] = ix.mpos[m];
                    if (q == QCAP) continue;
                    hash[r] = ix.mhash[m];
                    const uint32_t fl = ix.mflags[m] & 3u, pg = ix.mprev[m];
                    L.qfl[q] = (uint8_t)fl;
                    const bool rep = pg != NONE32 && pg >= c_begin;
                    L.qprev[q] = rep ? (int16_t)(pg - c_begin) : (int16_t)-1;
                    if (rep) {  // the hash repeats inside the tile (usually few)
                        if (fl & QF_ELIG) L.dup = 1;
                        dups[atomicAdd(&L.ndup, 1u)] = (uint16_t)q;
                    }
                }
                __syncthreads();
                const uint64_t lim = (uint64_t)L.qpos[C - 1] + n - k;
                if (qn > QCAP || (uint64_t)L.qpos[qn - 1] > lim) break;
                // the windows reach past what was loaded: all that the tile holds
                __syncthreads();
                qn = QCAP + 1;
                if (tid == 0) {
                    L.ndup = 0;
                    L.dup = 0;
                }
            }
            // directory entries behind the hashes (in flight until the lists are made)
            uint32_t d0[QR], d1[QR], d2[QR];
#pragma unroll
            for (int r = 0; r < QR; r++) {
                const uint32_t q = tid + (uint32_t)r * TB;
                d0[r] = d1[r] = d2[r] = 0;
                if (ix.dir_shift == 0 && q < min(qn, (uint32_t)QCAP) && (L.qfl[q] & QF_ELIG)) {
                    const uint64_t h = (uint64_t)hash[r] * 2;
                    d0[r] = ix.dir[h];
                    d1[r] = ix.dir[h + 1];
                    d2[r] = ix.dir[h + 2];
                }
            }
            if ((uint64_t)L.qpos[min(qn, (uint32_t)QCAP + 1) - 1] <= (uint64_t)L.qpos[C - 1] + n - k) {
                // more minimizers than a tile holds: fewer window starts
                if (tid == 0) {
                    uint32_t c = C;
                    while (c > 1 && (uint64_t)L.qpos[QCAP] <= (uint64_t)L.qpos[c - 1] + n - k) c /= 2;
                    if ((uint64_t)L.qpos[QCAP] <= (uint64_t)L.qpos[c - 1] + n - k) {
                        L.skip = 1;  // one window alone reaches too many
                        list_dense(a, L, c_begin);
                        if (L.err) atomicOr(a.err, L.err);
                    }
                    L.C = c;
                }
                __syncthreads();
                C = L.C;
                if (L.skip) {
                    c_begin += C;
                    __syncthreads();
                    continue;
                }
            }
            const uint32_t c0 = c_begin;
            PHASE(PH_SETUP);

            // ---- windows of the core: eligible, inside the span, gap-free;
            // their minimizers, sketch sizes and thresholds ----
            {
                const uint32_t ndup = L.ndup;
                const uint32_t qc = tid;
                uint32_t T = 0xFFFFu;
                bool win = false;
                if (qc < C) {
                    const uint32_t i = L.qpos[qc];
                    const uint64_t wl = (uint64_t)i + n - k;  // last minimizer inside [i, i + n)
                    uint32_t lo = qc, hi = min(qn, (uint32_t)QCAP);
                    while (lo < hi) {
                        uint32_t m = (lo + hi) >> 1;
                        if ((uint64_t)L.qpos[m] <= wl) lo = m + 1; else hi = m;
                    }
                    win = (L.qfl[qc] & QF_ELIG) && (uint64_t)i + n <= ge && mext >= n;
                    uint32_t s = 0;
                    if (win) {
                        // s_i: distinct hashes among all minimizers of the window =
                        // all of them minus those repeating a hash already inside
                        s = lo - qc;
                        if (ndup <= 256) {
                            for (uint32_t d = 0; d < ndup; d++) {
                                const uint32_t q = dups[d];
                                if (q >= qc && q < lo && L.qprev[q] >= (int)qc) s--;
                            }
                        } else {
                            s = 0;
                            for (uint32_t q = qc; q < lo; q++) s += (L.qprev[q] < (int)qc) ? 1u : 0u;
                        }
                        T = a.T[s];
                    }
                    L.win_qend[qc] = (uint16_t)lo;
                    L.win_s[qc] = (uint16_t)s;
                }
                // minima over 32 window starts and over the wave
                uint32_t t = T;
#pragma unroll
                for (int d = 1; d < 32; d <<= 1) t = min(t, (uint32_t)__shfl_xor((int)t, d, 64));
                if (qc < CMAX && (lane & 31) == 0) L.Tblk[qc >> 5] = (uint16_t)t;
                t = min(t, (uint32_t)__shfl_xor((int)t, 32, 64));
                const uint32_t nw = (uint32_t)__popcll(__ballot(win));
                if (lane == 0) {
                    L.wmin[wave] = t;
                    if (nw) atomicAdd(&L.nwin, nw);
                }
                if (wave == NWAVES - 1 && first_piece) next_tile(a, L, uni(ticket), lane);
                first_piece = false;
                for (uint32_t t2 = tid; t2 < NCHUNK; t2 += TB) L.marks[t2] = 0;
                for (uint32_t t2 = tid; t2 < TBYTES / 16; t2 += TB)
                    L.u.vec[t2] = uint4{0, 0, 0, 0};
            }
            __syncthreads();
            PHASE(PH_QUERY);
            const uint32_t Q = L.win_qend[C - 1];
            if (L.nwin == 0) {
                c_begin += C;
                __syncthreads();
                continue;
            }
            if (tid == 0) {
                L.cnt[CNT_WINDOWS] += L.nwin;
                if (L.dup) L.cnt[CNT_DUP_TILES] += 1;
            }
            uint32_t Tmin = 0xFFFFu;
#pragma unroll
            for (int w = 0; w < NWAVES; w++) Tmin = min(Tmin, L.wmin[w]);
            Tmin = uni(Tmin);
            const bool dup = uni(L.dup) != 0;

            // Lists of the partition, in the order of their minimizers' threads:
            // records, the marks that let a hit find its list, and the counters
            // of the minimizers' own positions taken out (an occurrence is
            // never paired with itself).  Returns the hits; more than HCAP:
            // only their number (saturated) is right.
            auto make_lists = [&](const uint32_t (&lo0)[QR], const uint32_t (&n0)[QR],
                                  const uint32_t (&lo1)[QR], const uint32_t (&n1)[QR]) -> uint32_t {
                uint32_t hits = 0, cnt = 0;
#pragma unroll
                for (int r = 0; r < QR; r++) {
                    const uint32_t len = min(n0[r], 1u << 19) + min(n1[r], 1u << 19);
                    hits += len;  // at most 2^20 each: no overflow over QCAP lists
                    cnt += len ? 1u : 0u;
                }
                const uint32_t hx = wave_sum_scan(hits), cx = wave_sum_scan(cnt);
                if (lane == 63) L.wtmp[wave] = ((uint64_t)cx << 32) | hx;
                __syncthreads();
                uint32_t hb = hx - hits, cb = cx - cnt, H = 0;
#pragma unroll
                for (int w = 0; w < NWAVES; w++) {
                    const uint64_t t = L.wtmp[w];
                    if (w < wave) {
                        hb += (uint32_t)t;
                        cb += (uint32_t)(t >> 32);
                    }
                    H += (uint32_t)t;
                }
                H = uni(H);
                if (H > HCAP) return H;
#pragma unroll
                for (int r = 0; r < QR; r++) {
                    const uint32_t len = n0[r] + n1[r];
                    if (!len) continue;
                    const uint32_t q = tid + (uint32_t)r * TB;
                    L.rec[cb] = uint2{lo0[r] - hb, q | ((L.qfl[q] & QF_STRAND) << 11) |
                                                       ((hb + n0[r]) << 12)};
                    L.rec1[cb] = lo1[r] - (hb + n0[r]);
                    if (hb) atomicOr(&L.marks[(hb - 1) >> 6], 1ull << ((hb - 1) & 63));
                    for (uint32_t c = (hb + 63) >> 6; c * 64 < hb + len; c++) L.pre[c] = (uint16_t)cb;
                    hb += len;
                    cb++;
                }
                return H;
            };
            static_assert((uint64_t)QCAP << 20 <= 1ull << 31, "sums of clamped list lengths");

            // ---- full-range lists and partition count ----
            uint32_t lo0[QR], n0[QR], lo1[QR], n1[QR];
#pragma unroll
            for (int r = 0; r < QR; r++) {
                const uint32_t q = tid + (uint32_t)r * TB;
                lo0[r] = n0[r] = lo1[r] = n1[r] = 0;
                if (q >= Q) continue;
                // the smallest threshold of the windows that hold q, bounded by
                // the minima of the 32-entry blocks covering those windows
                // (lossless: never above the true minimum)
                uint32_t lo = 0, hi = C;  // first core entry whose window reaches past q
                while (lo < hi) {
                    uint32_t m = (lo + hi) >> 1;
                    if (L.win_qend[m] <= q) lo = m + 1; else hi = m;
                }
                const uint32_t last = q < C ? q : C - 1;
                uint32_t t = 0xFFFFu;
                if (lo <= last)
                    for (uint32_t b = lo >> 5; b <= (last >> 5); b++) t = min(t, (uint32_t)L.Tblk[b]);
                L.qT[q] = (uint16_t)t;
                const uint32_t fl = L.qfl[q];
                if ((fl & QF_ELIG) && t != 0xFFFFu) {
                    if (ix.dir_shift) lookup(ix, hash[r], d0[r], d1[r], d2[r]);
                    lo0[r] = d0[r];
                    n0[r] = d1[r] - d0[r];
                    lo1[r] = d1[r];
                    n1[r] = d2[r] - d1[r];
                    L.qfl[q] = (uint8_t)(fl | QF_LISTED);
                }
            }
            const uint32_t Hfull = make_lists(lo0, n0, lo1, n1);
            uint32_t P = (Hfull + a.hpart - 1) / a.hpart;
            if (P < 1) P = 1;
            bool lists_full = Hfull <= HCAP;  // the lists hold every hit of every window
            bool clean = true;                // table and marks as the window phase left them
            bool modes_set = false;           // some minimizer has a mode
            bool multi = P > 1;               // run state crosses partitions
            if (tid == 0) L.sp = 0;
            if (multi)
                for (uint32_t t = tid; t < 2 * C; t += TB) L.run_c[t] = 0;
            PHASE(PH_LISTS);
            // Target partitions in increasing order; a partition with too many
            // hits or kept hits is split in halves on a small stack (LIFO,
            // left half first, so candidates still arrive in target order).
            // A partition already down to 4n bases is split over its window
            // starts instead: each window keeps its own run state, so any
            // grouping of windows sees its candidates in target order.
            for (uint32_t pt = 0; pt < P; pt++) {
            if (tid == 0) {
                L.sp = 1;
                L.stackA[0] = (uint32_t)((ix.total * (uint64_t)pt) / P);
                L.stackB[0] = (uint32_t)((ix.total * (uint64_t)(pt + 1)) / P);
                L.stackW[0] = C << 16;
            }
            for (;;) {
                const uint32_t tid = opaque(threadIdx.x), lane = tid & 63;
                const SearchArgs &a = kernel_args();
                const IndexView &ix = a.ix;
                __syncthreads();
                if (L.sp == 0) break;
                const uint32_t A = uni(L.stackA[L.sp - 1]), B = uni(L.stackB[L.sp - 1]);
                const uint32_t WA = uni(L.stackW[L.sp - 1] & 0xFFFFu), WB = uni(L.stackW[L.sp - 1] >> 16);
                __syncthreads();
                if (tid == 0) {
                    L.sp--;
                    L.ncoll = 0;
                    L.nraw = 0;
                    L.csum = 0;
                    L.nself = 0;
                }
                const bool full = (A == 0 && (uint64_t)B >= ix.total);
                const bool allw = (WA == 0 && WB == C);
                const bool single = WB - WA == 1;
                const bool single_dup = dup && single;
                const uint32_t QE = L.win_qend[WB - 1];  // minimizers [WA, QE) of the windows
                const uint64_t lo_pos = (A > n) ? (uint64_t)A - n : 0;
                const uint64_t hi_pos = (uint64_t)B + 2ull * n;  // exclusive
                uint32_t H = Hfull;
                bool pieces = false;  // a list's strands are not adjacent
                if (!(full && allw && lists_full && !single_dup)) {
                    // ---- lists restricted to [A - n, B + 2n) and the windows' minimizers ----
                    if (!clean) {
                        for (uint32_t t = tid; t < NCHUNK; t += TB) L.marks[t] = 0;
                        for (uint32_t t = tid; t < TBYTES / 16; t += TB)
                            L.u.vec[t] = uint4{0, 0, 0, 0};
                    } else if (lists_full) {
                        for (uint32_t t = tid; t < NCHUNK; t += TB) L.marks[t] = 0;
                    }
                    if (single_dup) {
                        for (uint32_t q = tid; q < Q; q += TB) {
                            uint32_t m = L.qfl[q] & ~(uint32_t)(QF_SKIP | QF_UNION);
                            if (q >= WA && q < QE && (m & QF_ELIG))
                                for (int r = L.qprev[q]; r >= (int)WA; r = L.qprev[r])
                                    if ((L.qfl[r] & QF_ELIG) && ((L.qfl[r] ^ m) & QF_STRAND) == 0) {
                                        m |= QF_SKIP;
                                        break;
                                    }
                            L.qfl[q] = (uint8_t)m;
                        }
                        __syncthreads();
                        // the earliest member in the window stands for the skipped
                        // (several may write it: the same value)
                        for (uint32_t q = tid; q < Q; q += TB) {
                            if (!(L.qfl[q] & QF_SKIP)) continue;
                            int first = -1;
                            for (int r = L.qprev[q]; r >= (int)WA; r = L.qprev[r])
                                if ((L.qfl[r] & QF_ELIG) && ((L.qfl[r] ^ L.qfl[q]) & QF_STRAND) == 0)
                                    first = r;
                            if (first >= 0) L.qfl[first] = (uint8_t)(L.qfl[first] | QF_UNION);
                        }
                        modes_set = true;
                    } else if (modes_set) {
                        for (uint32_t q = tid; q < Q; q += TB)
                            L.qfl[q] = (uint8_t)(L.qfl[q] & ~(QF_SKIP | QF_UNION));
                        modes_set = false;
                    }
                    __syncthreads();
#pragma unroll
                    for (int r = 0; r < QR; r++) {
                        const uint32_t q = tid + (uint32_t)r * TB;
                        lo0[r] = n0[r] = lo1[r] = n1[r] = 0;
                        if (q >= Q) continue;
                        uint32_t fl = L.qfl[q] & ~(uint32_t)QF_LISTED;
                        if ((fl & QF_ELIG) && L.qT[q] != 0xFFFFu && q >= WA && q < QE &&
                            !(fl & QF_SKIP)) {
                            uint32_t x0, x1, x2;
                            lookup(ix, ix.mhash[c0 + q], x0, x1, x2);
                            uint32_t b0 = x1, b1 = x2;
                            lo0[r] = x0;
                            lo1[r] = x1;
                            if (!full) {
                                lower_pos2(ix, x0, x1, lo_pos, hi_pos, lo0[r], b0);
                                lower_pos2(ix, x1, x2, lo_pos, hi_pos, lo1[r], b1);
                            }
                            n0[r] = b0 - lo0[r];
                            n1[r] = b1 - lo1[r];
                            const uint64_t p = L.qpos[q];
                            if (p >= lo_pos && p < hi_pos) fl |= QF_LISTED;
                        }
                        L.qfl[q] = (uint8_t)fl;
                    }
                    H = make_lists(lo0, n0, lo1, n1);
                    lists_full = full && allw && !single_dup && H <= HCAP;
                    pieces = !full;
                    clean = true;
                }
                PHASE(PH_PLISTS);
                if (H == 0) continue;
                if (H > HCAP) {
                    __syncthreads();
                    if (tid == 0) split_partition(a, L, A, B, WA, WB, n);
                    if (!multi)
                        for (uint32_t t = tid; t < 2 * C; t += TB) L.run_c[t] = 0;
                    multi = true;
                    __syncthreads();
                    if (L.err) break;
                    continue;
                }
                __syncthreads();  // lists made, scalars cleared
                clean = false;
                if (tid == 0) {
                    L.cnt[CNT_HITS] += H;
                    L.cnt[CNT_PARTS] += 1;
                }
                const uint32_t SB = a.bin_shift;
                const uint32_t nch = (H + 63) / 64;
                // counter bits: 2^lb.  Four while the hits would crowd byte
                // counters (more than 0.42 a slot: at thresholds around 6 a
                // slot then gets hot by chance too often), 16 for a single
                // window, where what is kept has to be exactly what its own
                // threshold keeps (a window that cannot be split is listed as
                // dense when too many are kept), or past the smaller ones' range.
                uint32_t lb = (H * 19 > TBYTES * 8 && Tmin <= 15) ? 2u : 3u;
                if (Tmin > 255 || single) lb = 4;
                uint32_t st[SG][HU] = {};  // (set here, so that nothing lives on from the last partition)
                uint32_t om[SG] = {};
                bool fresh = true;
                for (;;) {
                    if (lb == 4) break;
                    // ---- gather: bin counts, hits into registers ----
                    const uint32_t tid = opaque(threadIdx.x), lane = tid & 63;
                    const uint32_t *const epos = kernel_args().ix.epos;
                    const uint32_t hl = TLOG + 2 - lb;  // log2 of half the slots
                    const uint32_t lw = 5 - lb;         // log2 of the slots per word
                    const uint32_t fm = (1u << lw) - 1;
                    auto count = [&](uint32_t p, uint32_t o) {
                        const uint32_t slot = slot_of(p, o, SB, hl);
                        atomicAdd(&L.u.table[slot >> lw], 1u << ((slot & fm) << lb));
                    };
#pragma unroll
                    for (int g = 0; g < SG; g++) {
                        const uint32_t c = (uint32_t)(g * NWAVES + wave) * HU;
                        if (c < nch) {
                            if (fresh) om[g] = gather_hits(L, epos, H, nch, pieces, c, lane, st[g]);
#pragma unroll
                            for (int u = 0; u < HU; u++)
                                if ((c + (uint32_t)u) * 64 + lane < H)
                                    count(st[g][u], (om[g] >> u) & 1u);
                        }
                    }
                    for (uint32_t c = (uint32_t)(SG * NWAVES + wave) * HU; c < nch; c += NWAVES * HU) {
                        uint32_t pv[HU];
                        const uint32_t ob = gather_hits(L, epos, H, nch, pieces, c, lane, pv);
#pragma unroll
                        for (int u = 0; u < HU; u++)
                            if ((c + (uint32_t)u) * 64 + lane < H) count(pv[u], (ob >> u) & 1u);
                    }
                    // the minimizers' own positions, each once in their lists
                    uint32_t self = 0;
                    for (uint32_t q = tid; q < Q; q += TB)
                        if (L.qfl[q] & QF_LISTED) {
                            const uint32_t slot = slot_of(L.qpos[q], 0, SB, hl);
                            atomicSub(&L.u.table[slot >> lw], 1u << ((slot & fm) << lb));
                            self++;
                        }
                    self = wave_sum_scan(self);
                    if (lane == 63 && self) atomicAdd(&L.nself, self);
                    __syncthreads();
                    PHASE(PH_PASS1);
                    // ---- counters into hot flags ----
                    uint4 hv[TBYTES / 16 / TB];
                    uint32_t sum = 0;
#pragma unroll
                    for (uint32_t v = 0; v < TBYTES / 16 / TB; v++) {
                        const uint32_t x = tid + v * TB;
                        const uint4 w = L.u.vec[x];
                        const uint32_t hb = (x * 4) & (TWORDS / 2), hm = TWORDS / 2 - 1;
                        const uint32_t pw = L.u.table[hb | ((x * 4 - 1) & hm)];
                        const uint32_t nw = L.u.table[hb | ((x * 4 + 4) & hm)];
                        if (lb == 2) {
                            hv[v].x = hot_nibbles(pw, w.x, w.y, Tmin, sum);
                            hv[v].y = hot_nibbles(w.x, w.y, w.z, Tmin, sum);
                            hv[v].z = hot_nibbles(w.y, w.z, w.w, Tmin, sum);
                            hv[v].w = hot_nibbles(w.z, w.w, nw, Tmin, sum);
                        } else {
                            hv[v].x = hot_bytes(pw, w.x, w.y, Tmin, sum);
                            hv[v].y = hot_bytes(w.x, w.y, w.z, Tmin, sum);
                            hv[v].z = hot_bytes(w.y, w.z, w.w, Tmin, sum);
                            hv[v].w = hot_bytes(w.z, w.w, nw, Tmin, sum);
                        }
                    }
                    sum = wave_sum_scan(sum);
                    if (lane == 63) atomicAdd(&L.csum, sum);
                    __syncthreads();
                    const bool exact = L.csum == H - L.nself;
                    if (exact) {
#pragma unroll
                        for (uint32_t v = 0; v < TBYTES / 16 / TB; v++) L.u.vec[tid + v * TB] = hv[v];
                        __syncthreads();
                        break;
                    }
                    // a counter overflowed: once more with wider ones
                    for (uint32_t t = tid; t < TBYTES / 16; t += TB) L.u.vec[t] = uint4{0, 0, 0, 0};
                    __syncthreads();
                    if (tid == 0) {
                        L.csum = 0;
                        L.nself = 0;
                    }
                    __syncthreads();
                    fresh = false;
                    lb++;
                }
                if (lb < 4) {
                    // ---- keep the hits of hot slots: position, orientation, hit number ----
                    const uint32_t tid = opaque(threadIdx.x), lane = tid & 63;
                    const uint32_t *const epos = kernel_args().ix.epos;
                    const uint32_t hl = TLOG + 2 - lb;
                    auto keep = [&](const uint32_t (&pv)[HU], uint32_t ob, uint32_t c) {
                        uint32_t kp = 0;
#pragma unroll
                        for (int u = 0; u < HU; u++) {
                            const uint32_t slot = slot_of(pv[u], (ob >> u) & 1u, SB, hl);
                            const uint32_t by = reinterpret_cast<const uint8_t *>(L.u.table)[slot >> (3 - lb)];
                            const uint32_t hot = (by >> ((slot << lb) & 7u)) & 1u;
                            kp |= ((c + (uint32_t)u) * 64 + lane < H ? hot : 0u) << u;
                        }
                        // one LDS atomic per wave and round for the kept hits' slots
                        const uint32_t nk = (uint32_t)__popc(kp);
                        if (!__ballot(nk != 0)) return;
                        const uint32_t ex = wave_sum_scan(nk) - nk;
                        uint32_t base = 0;
                        if (lane == 63) base = atomicAdd(&L.nraw, ex + nk);
                        base = lane_read(base, 63) + ex;
#pragma unroll
                        for (int u = 0; u < HU; u++) {
                            if (!((kp >> u) & 1u)) continue;
                            if (base < CB)
                                L.coll[base] = ((uint64_t)pv[u] << 17) | (((ob >> u) & 1u) << 16) |
                                               ((c + (uint32_t)u) * 64 + lane);
                            base++;
                        }
                    };
#pragma unroll
                    for (int g = 0; g < SG; g++) {
                        const uint32_t c = (uint32_t)(g * NWAVES + wave) * HU;
                        if (c < nch) keep(st[g], om[g], c);
                    }
                    for (uint32_t c = (uint32_t)(SG * NWAVES + wave) * HU; c < nch; c += NWAVES * HU) {
                        uint32_t pv[HU];
                        const uint32_t ob = gather_hits(L, epos, H, nch, pieces, c, lane, pv);
                        keep(pv, ob, c);
                    }
                    __syncthreads();
                    // ---- their minimizers; self-hits leave ----
                    const uint32_t nraw = L.nraw;
                    if (nraw <= CB) {
                        uint64_t key[CB / TB];
#pragma unroll
                        for (int r = 0; r < CB / TB; r++) {
                            const uint32_t x = tid + (uint32_t)r * TB;
                            key[r] = SENT64;
                            if (x >= nraw) continue;
                            const uint64_t v = L.coll[x];
                            const uint32_t p = (uint32_t)(v >> 17), o = (uint32_t)(v >> 16) & 1u;
                            const uint32_t q = L.rec[list_of(L, (uint32_t)v & 0xFFFFu)].y & 2047u;
                            if (p != L.qpos[q]) key[r] = ckey(o, p, q);
                        }
                        __syncthreads();
#pragma unroll
                        for (int r = 0; r < CB / TB; r++) {
                            const uint64_t m = __ballot(key[r] != SENT64);
                            if (!m) continue;
                            uint32_t base = 0;
                            if (lane == 0) base = atomicAdd(&L.ncoll, (uint32_t)__popcll(m));
                            base = lanes_below(m, uni(base));
                            if (key[r] != SENT64) L.coll[base] = key[r];
                        }
                    } else if (tid == 0) {
                        L.ncoll = NONE32;
                    }
                } else {
                    // ---- 16-bit counters, in two passes over the lists: counts
                    // without self-hits, then each hit against its minimizer's
                    // own threshold ----
                    constexpr uint32_t hl = TLOG - 2;
                    const uint32_t *const epos = kernel_args().ix.epos;
                    const uint16_t *t16 = reinterpret_cast<const uint16_t *>(L.u.table);
                    for (int pass = 0; pass < 2; pass++) {
                        for (uint32_t c = wave; c < nch; c += NWAVES) {
                            const uint32_t e = c * 64 + lane;
                            bool kp = false;
                            uint32_t p = 0, q = 0, o = 0;
                            if (e < H) {
                                const uint32_t l = list_of(L, e);
                                const uint2 r = L.rec[l];
                                const uint32_t b = e >= (r.y >> 12) ? 1u : 0u;
                                q = r.y & 2047u;
                                p = epos[(pieces && b ? L.rec1[l] : r.x) + e];
                                o = b ^ ((r.y >> 11) & 1u);
                                kp = p != L.qpos[q] || (L.qfl[q] & QF_UNION);
                            }
                            const uint32_t slot = slot_of(p, o, SB, hl);
                            if (pass == 0) {
                                if (kp) atomicAdd(&L.u.table[slot >> 1], 1u << ((slot & 1) * 16));
                                continue;
                            }
                            if (kp) {
                                const uint32_t hm = (1u << hl) - 1, hb = o << hl, Tq = L.qT[q];
                                const uint32_t m2 = t16[hb | ((slot - 2) & hm)];
                                const uint32_t m1 = t16[hb | ((slot - 1) & hm)];
                                const uint32_t z0 = t16[slot];
                                const uint32_t p1 = t16[hb | ((slot + 1) & hm)];
                                kp = m2 + m1 >= Tq || m1 + z0 >= Tq || z0 + p1 >= Tq;
                            }
                            const uint64_t m = __ballot(kp);
                            if (!m) continue;
                            uint32_t base = 0;
                            if (lane == 0) base = atomicAdd(&L.ncoll, (uint32_t)__popcll(m));
                            base = lanes_below(m, uni(base));
                            if (kp && base < CB) L.coll[base] = ckey(o, p, q);
                        }
                        __syncthreads();
                    }
                }
                __syncthreads();
                PHASE(PH_PASS2);
                const uint32_t ncoll = uni(L.ncoll);
                if (ncoll == 0) continue;
                if (ncoll > min(a.kept_cap, (uint32_t)CB)) {
                    if (tid == 0) split_partition(a, L, A, B, WA, WB, n);
                    if (!multi)
                        for (uint32_t t = tid; t < 2 * C; t += TB) L.run_c[t] = 0;
                    multi = true;
                    __syncthreads();
                    if (L.err) break;
                    continue;
                }
                if (tid == 0) L.cnt[CNT_KEPT] += ncoll;
                // ---- sort kept hits by (o, p', q) ----
                static_assert(CB % 64 == 0, "runs of 64 kept hits");
                block_sort_runs(L.coll, ncoll);
                PHASE(PH_SORT);
                // ---- exact hot starts: >= Tmin hits in [x, x + n - k] ----
                PostLds &F = L.u.post;
                for (uint32_t e = tid; e < ncoll; e += TB) {
                    const uint64_t key = L.coll[e];
                    uint32_t hv = 0;
                    const bool first = (e == 0) || ck_op(L.coll[e - 1]) != ck_op(key);
                    if (first && e + Tmin - 1 < ncoll) {
                        const uint64_t k2 = L.coll[e + Tmin - 1];
                        if (ck_o(k2) == ck_o(key) && (uint64_t)ck_p(k2) <= (uint64_t)ck_p(key) + n - k)
                            hv = e + 1;
                    }
                    F.hot[e] = hv;
                }
                __syncthreads();
                block_maxscan_u32(F.hot, (int)ncoll, L.wtmp);
                // ---- relevant: within [x, x + 2n - k) of the last hot x ----
                for (uint32_t e = tid; e < ncoll; e += TB) {
                    const uint64_t key = L.coll[e];
                    const uint32_t lh = F.hot[e];
                    uint32_t f = 0;
                    if (lh && ck_o(L.coll[lh - 1]) == ck_o(key)) {
                        const uint64_t x = ck_p(L.coll[lh - 1]);
                        const uint64_t d = (uint64_t)ck_p(key) - x;
                        if (d < 2ull * n - k) f |= 4;   // relevant
                        if (d < n) f |= EF_CAND;
                    }
                    F.relf[e] = (uint8_t)f;
                    F.pref[e] = (f & 4) ? 1u : 0u;
                }
                __syncthreads();
                const uint32_t nrel = uni(block_scan_u32(F.pref, (int)ncoll, L.wtmp));
                // stable compaction in place: read everything first, then write
                uint64_t keep_k[CB / TB] = {};
                uint32_t keep_at[CB / TB];
                uint8_t keep_f[CB / TB] = {};
#pragma unroll
                for (int r = 0; r < CB / TB; r++) {
                    const uint32_t e = tid + r * TB;
                    keep_at[r] = NONE32;
                    if (e < ncoll && (F.relf[e] & 4)) {
                        keep_k[r] = L.coll[e];
                        keep_f[r] = F.relf[e] & EF_CAND;
                        keep_at[r] = F.pref[e];
                    }
                }
                __syncthreads();
                PHASE(PH_HOT);
                if (nrel == 0) continue;
#pragma unroll
                for (int r = 0; r < CB / TB; r++) {
                    if (keep_at[r] != NONE32) {
                        L.coll[keep_at[r]] = keep_k[r];
                        F.einfo[keep_at[r]] = keep_f[r] ? EI_CAND : 0u;
                    }
                }
                if (dup)  // the repeats' chains forwards
                    for (uint32_t q = tid; q < Q; q += TB) F.qnext[q] = -1;
                __syncthreads();
                if (dup)
                    for (uint32_t q = tid; q < Q; q += TB)
                        if (L.qprev[q] >= 0) F.qnext[L.qprev[q]] = (int16_t)q;
                if (tid == 0) {
                    // orientation 1 starts at the first entry with o = 1
                    uint32_t lo = 0, hi = nrel;
                    while (lo < hi) {
                        uint32_t m = (lo + hi) >> 1;
                        if (ck_o(L.coll[m]) == 0) lo = m + 1; else hi = m;
                    }
                    L.obeg[0] = 0;
                    L.oend[0] = lo;
                    L.obeg[1] = lo;
                    L.oend[1] = nrel;
                }
                __syncthreads();
                for (uint32_t e = tid; e < nrel; e += TB) {
                    const uint64_t key = L.coll[e];
                    const uint32_t o = ck_o(key), p = ck_p(key), q = ck_q(key);
                    // end of the counting range [p, p + n - k]
                    uint32_t lo = e, hi = L.oend[o];
                    const uint64_t lim = (uint64_t)p + n - k;
                    while (lo < hi) {
                        uint32_t m = (lo + hi) >> 1;
                        if ((uint64_t)ck_p(L.coll[m]) <= lim) lo = m + 1; else hi = m;
                    }
                    F.rng_end[e] = (uint16_t)lo;
                    uint32_t info = q;
                    if (e > L.obeg[o] && ck_p(L.coll[e - 1]) == p) info |= EI_SAMEP;
                    if ((F.einfo[e] & EI_CAND) && p >= A && p < B) {  // owned by this partition
                        uint32_t sq = 0;
                        if (window_ok(ix, p, n, &sq)) info |= EI_CAND;
                        F.etb[e] = (uint32_t)ix.off[sq];
                    }
                    F.einfo[e] = info;
                }
                __syncthreads();
                PHASE(PH_SEGINFO);

                // ---- exact counts, runs and seeds: one lane per window ----
                // A wave takes 64 consecutive windows and one orientation, and
                // walks the kept hits that are candidates j of its windows in
                // target order; a window's count is the number of its
                // minimizers with a kept hit in [j, j + n - k] (repeats of a
                // hash once).  A step of a candidate is a few compares, ballots
                // and popcounts and the run logic, without memory accesses
                // (eval_masks); blocks whose windows reach more than 256
                // minimizers follow the hits that enter and leave instead.
                SeedBuf sbuf{F.seeds + wave * SBUF * 6, 0};
                uint32_t n_evals = 0, n_scan = 0;
                // all windows of orientation 0, then of 1: a tile's hits are mostly
                // of one orientation, and every wave gets a share of them
                const uint32_t nblock = (WB - WA + 63) / 64, ntask = 2 * nblock;
                for (uint32_t task = wave; task < ntask; task += NWAVES) {
                    const SearchArgs &a = kernel_args();
                    const uint32_t o = task >= nblock ? 1u : 0u, b0 = WA + (task - o * nblock) * 64;
                    const uint32_t ob = uni(L.obeg[o]), oe = uni(L.oend[o]);
                    if (ob >= oe) continue;  // nothing ends a run but a candidate
                    const uint32_t qc = b0 + lane;
                    Block bk;
                    bk.qlo = b0;
                    bk.qhi = uni(L.win_qend[min(b0 + 63, WB - 1)]);
                    bk.si = qc < WB ? L.win_s[qc] : 0u;
                    const bool win = bk.si != 0;
                    bk.Ti = opaque(win ? a.T[bk.si] : 0u);  // (waited for here, not in the steps)
                    bk.qc = qc;
                    bk.len = win ? L.win_qend[qc] - qc : 0u;
                    bk.i = win ? L.qpos[qc] : 0u;
                    bk.o = o;
                    bk.near = a.n - a.max_overlap - 1;
                    bk.runs_out = a.runs_out != 0;
                    RunState rs{0, 0, 0};
                    if (win && multi) {
                        rs.prev_j = L.run_prev[2 * qc + o];
                        rs.best_j = L.run_best[2 * qc + o];
                        rs.best_c = L.run_c[2 * qc + o];
                    }
                    EndedRuns er{0, 0, 0};
                    const uint32_t nq = bk.qhi - bk.qlo;
                    if (nq <= 192 && !dup)
                        eval_masks<3, false>(a, L, sbuf, bk, rs, er, ob, oe, lane, n_evals, n_scan);
                    // (a fourth form costs the 1,024-thread layout, for dense indexes, more
                    // than it gives: 3.1 Gbp 170.3 against 169.8 ms)
                    else if (TB == 512 && nq <= 192)
                        eval_masks<3, true>(a, L, sbuf, bk, rs, er, ob, oe, lane, n_evals, n_scan);
                    else if (nq <= 256 && !dup)
                        eval_masks<4, false>(a, L, sbuf, bk, rs, er, ob, oe, lane, n_evals, n_scan);
                    else if (nq <= 256)
                        eval_masks<4, true>(a, L, sbuf, bk, rs, er, ob, oe, lane, n_evals, n_scan);
                    else
                        eval_events(a, L, sbuf, bk, rs, er, ob, oe, lane, dup, n_evals, n_scan);
                    if (multi) {
                        if (win) {
                            L.run_prev[2 * qc + o] = rs.prev_j;
                            L.run_best[2 * qc + o] = rs.best_j;
                            L.run_c[2 * qc + o] = (uint16_t)rs.best_c;
                        }
                    } else {  // the only partition: the open runs end
                        const uint64_t em = __ballot(rs.best_c != 0);
                        if (em & er.m) push_ended(a, L, sbuf, bk, er, lane);
                        er.m |= em;
                        er.j = rs.best_c ? rs.best_j : er.j;
                        er.v = rs.best_c ? (bk.runs_out ? rs.prev_j : rs.best_c) : er.v;
                    }
                    if (er.m) push_ended(a, L, sbuf, bk, er, lane);
                }
                if (lane == 0) {
                    atomicAdd(&L.cnt[CNT_EVALS], (unsigned long long)n_evals);
                    atomicAdd(&L.cnt[CNT_SCAN], (unsigned long long)n_scan);
                }
                seeds_flush_block(a, L, sbuf, lane, wave);
                __syncthreads();
                PHASE(PH_EVAL);
            }  // stack of one partition
            __syncthreads();
            if (L.err) break;
            }  // partitions
            if (L.err) {
                if (tid == 0) atomicOr(a.err, L.err);
            } else if (multi) {
                // close the runs still open after the last partition: one
                // (window, orientation) per lane
                SeedBuf sbuf{L.u.post.seeds + wave * SBUF * 6, 0};
                for (uint32_t b0 = wave * 64; b0 < 2 * C; b0 += TB) {
                    const uint32_t x = b0 + lane, qc = x >> 1;
                    const bool mine = x < 2 * C && L.win_s[qc] && L.run_c[x];
                    seeds_push_lanes(a, sbuf, lane, mine, L.qid, mine ? L.qpos[qc] : 0,
                                     mine ? L.run_best[x] : 0, x & 1,
                                     mine ? (a.runs_out ? L.run_prev[x] : L.run_c[x]) : 0,
                                     mine ? L.win_s[qc] : 0);
                }
                seeds_flush_block(a, L, sbuf, lane, wave);
            }
            c_begin += C;
            __syncthreads();
            PHASE(PH_FLUSH);
        }
        // (every piece left out: no window phase ran)
        if (wave == NWAVES - 1 && first_piece)
            next_tile(kernel_args(), L, uni(ticket), threadIdx.x & 63);
    }
    __syncthreads();
    const SearchArgs &a = kernel_args();
    if (threadIdx.x < CNT_N && threadIdx.x != CNT_SEEDS && L.cnt[threadIdx.x])
        atomicAdd(&a.counters[threadIdx.x], L.cnt[threadIdx.x]);
    if (prof)
        for (int t = 0; t < PH_N; t++) atomicAdd(&a.phase[t], (unsigned long long)L.ph[t]);
}

void launch_tile_search(const SearchArgs &a, uint32_t grid, hipStream_t st) {
    k_tile_search<<<grid, TB, 0, st>>>(a);
    SDF_HIP(hipGetLastError());
}

uint32_t tile_core_max() { return CMAX; }
TileLimits tile_limits() { return TileLimits{CMAX, QCAP, HCAP, CB, 2 * TBYTES}; }

}  // namespace tile1024 / tile512

#if SDF_TILE_THREADS == 1024  // the span set-up is compiled once
// Per span: minimizer range of its window starts and its tile count.
__global__ void k_span_setup(const IndexView ix, SpanDesc *spans, uint32_t nspans, uint32_t n,
                             uint32_t core, uint32_t *ntiles) {
    uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nspans) return;
    SpanDesc &d = spans[s];
    uint32_t mlo = 0, mhi = 0;
    if (d.ge >= d.gb + n) {
        uint64_t lo = 0, hi = ix.nm;
        while (lo < hi) {
            uint64_t m = (lo + hi) >> 1;
            if ((uint64_t)ix.mpos[m] < d.gb) lo = m + 1; else hi = m;
        }
        mlo = (uint32_t)lo;
        hi = ix.nm;
        const uint64_t lim = d.ge - n;
        while (lo < hi) {
            uint64_t m = (lo + hi) >> 1;
            if ((uint64_t)ix.mpos[m] <= lim) lo = m + 1; else hi = m;
        }
        mhi = (uint32_t)lo;
    }
    d.m_lo = mlo;
    d.m_hi = mhi;
    ntiles[s] = (mhi - mlo + core - 1) / core;
}

__global__ void k_span_tiles(SpanDesc *spans, uint32_t nspans, const uint32_t *tile0) {
    uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < nspans) spans[s].tile0 = tile0[s];
}

void launch_span_setup(const IndexView &ix, SpanDesc *spans, uint32_t nspans, uint32_t n,
                       uint32_t core, uint32_t *ntiles, uint32_t *tile0, hipStream_t st) {
    k_span_setup<<<(nspans + 255) / 256, 256, 0, st>>>(ix, spans, nspans, n, core, ntiles);
    SDF_HIP(hipGetLastError());
    scan_u32(ntiles, tile0, nspans, st);
    k_span_tiles<<<(nspans + 255) / 256, 256, 0, st>>>(spans, nspans, tile0);
    SDF_HIP(hipGetLastError());
}

#endif

}  // namespace sdf
