// q-gram similarity of region pairs (Section 3.2, second paragraph).
//
// Q(G_i, G_j) counts the q-mers the two substrings share, with multiplicity:
// the sum over q-mers x of min(occurrences in G_i, occurrences in G_j).  A
// q-mer holding an N is skipped; in orientation 1 the q-mers of G_j are those
// of its reverse complement.  One workgroup per region builds both sides'
// histograms of 4^q bins in LDS from the index's 2-bit packed bases and gap
// bits, then sums the minima.  A lane takes a whole packed word, so the q-mers
// starting in its 16 bases come from two words and their gap bits in registers
// (0.375 B read per base and side) and cost a shift, a mask and one LDS atomic
// each, which is what bounds it; bins are the packed digits as they lie, and
// the reverse complement is taken once per bin in the final sum.  Measured on
// 9,157 regions with 443 Mbp of sides: one q-mer per lane, with its words read
// and its digits reversed each time, 1.71 ms a call; this 0.27 ms.
#include <algorithm>

#include "extend.h"

namespace sdf {

namespace {

constexpr int QT = 256;
constexpr uint32_t QMAX = 6;

// Reverse the order of q 2-bit digits.
__device__ __forceinline__ uint32_t digits_reversed(uint32_t v, uint32_t q) {
    uint32_t r = 0;
    for (uint32_t u = 0; u < q; u++) {
        r = (r << 2) | (v & 3);
        v >>= 2;
    }
    return r;
}

__global__ void __launch_bounds__(QT) k_qgram(IndexView ix, const sdf_region *reg, uint64_t n,
                                              uint32_t q, unsigned long long *out) {
    extern __shared__ uint32_t hist[];  // query side, then target side
    __shared__ unsigned long long part[QT / 64];
    const uint64_t id = blockIdx.x;
    if (id >= n) return;
    const sdf_region R = reg[id];
    const uint32_t nb = 1u << (2 * q);
    const uint32_t mask = nb - 1;
    for (uint32_t i = threadIdx.x; i < 2 * nb; i += QT) hist[i] = 0;
    __syncthreads();
    const uint32_t gmask = (1u << q) - 1;
    for (int side = 0; side < 2; side++) {
        const uint64_t base = ix.off[side ? R.t_seq : R.q_seq];
        const uint64_t a = base + (side ? R.t_begin : R.q_begin);
        const uint64_t b = base + (side ? R.t_end : R.q_end);
        if (b < a + q) continue;
        const uint64_t last = b - q;  // the last q-mer's start
        uint32_t *const h = hist + side * nb;
        for (uint64_t w = (a >> 4) + threadIdx.x; w <= (last >> 4); w += QT) {
            // the starts [s0, s1] of the word's bases 0 .. 15; the next word (and
            // its gap bits) only when one of them reaches into it, so no read
            // passes the last base of the index
            const uint32_t s0 = w * 16 < a ? (uint32_t)(a - w * 16) : 0u;
            const uint32_t s1 = (uint32_t)min(last - w * 16, (uint64_t)15);
            const bool two = s1 + q > 16;
            const uint32_t lo = ix.packed[w], hi = two ? ix.packed[w + 1] : 0u;
            uint32_t g = ix.gaps[w >> 1] >> (16 * (w & 1));  // gap bits of bases 0 .. 31
            if (w & 1) {
                g &= 0xFFFFu;
                if (two) g |= ix.gaps[(w >> 1) + 1] << 16;
            }
            if (s0 == 0 && s1 == 15 && g == 0) {
#pragma unroll
                for (uint32_t u = 0; u < 16; u++) {
                    const uint32_t v = (uint32_t)((((uint64_t)hi << 32) | lo) >> (2 * u));
                    atomicAdd(&h[v & mask], 1u);
                }
            } else {
                for (uint32_t u = s0; u <= s1; u++)
                    if (((g >> u) & gmask) == 0) {
                        const uint32_t v = (uint32_t)((((uint64_t)hi << 32) | lo) >> (2 * u));
                        atomicAdd(&h[v & mask], 1u);
                    }
            }
        }
    }
    __syncthreads();
    unsigned long long s = 0;
    // (the first base of a q-mer in the lowest digit: the reverse complement of
    // q-mer v is ~v with its digits in reverse)
    for (uint32_t i = threadIdx.x; i < nb; i += QT)
        s += min(hist[i], hist[nb + (R.strand ? ~digits_reversed(i, q) & mask : i)]);
    for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int wv = 0; wv < QT / 64; wv++) t += part[wv];
        out[id] = t;
    }
}

}  // namespace

uint32_t qgram_max_q() { return QMAX; }

void launch_qgram(const IndexView &ix, const sdf_region *reg, uint64_t n, uint32_t q,
                  unsigned long long *out, hipStream_t st) {
    if (n == 0) return;
    for (uint64_t done = 0; done < n;) {  // grids of at most 2^31 - 1 workgroups
        const uint64_t m = std::min<uint64_t>(n - done, 0x7FFFFFFFull);
        k_qgram<<<(unsigned)m, QT, 8u << (2 * q), st>>>(ix, reg + done, m, q, out + done);
        SDF_HIP(hipGetLastError());
        done += m;
    }
}

}  // namespace sdf
