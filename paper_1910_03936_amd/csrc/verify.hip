// Verification of the pairs a filter passes: the banded edit distance of each
// (read, reference segment) pair, min(distance, E + 1), restricted to the
// 2E+1 diagonals of the filter's map (Ukkonen's band).  This is the step the
// filter hands its accepted pairs to (Ch. 1, seed-and-extend), in the form of
// Sec. 8.7's prefix edit distance: the work grows with the number of edits
// found so far, and stops as soon as E is exceeded.
//
// One lane per pair, by diagonal transition (Ukkonen 1985; Landau and Vishkin
// 1989): F_k[d] is the furthest reference column c such that ref[0..c) and
// read[0..c+d) align with at most k edits inside the band.  From F_{k-1} on
// diagonals d-1, d and d+1 one edit more reaches column
//   x = max(F_{k-1}[d] + 1  (substitution),
//           F_{k-1}[d+1] + 1 (a reference base left out),
//           F_{k-1}[d-1]     (a read base left out)),
// and the diagonal's run of matches from x (a pipe of the map, Eq. 8.2) then
// comes for free.  The distance is the first k with F_k[0] = m.  Runs are
// found 32 bases at a time from the planar two-bit words: an XOR per code
// plane, an OR, and a count of trailing zeros.
//
// Every lane walks its own rounds and diagonals: a step is 32 bases of one run,
// after which the lane goes on with the run, the next diagonal or the next
// round.  F and the pair's words are in LDS columns of the lane's own, where
// any lane can be at any diagonal (in registers they force the lanes of a wave
// through the same diagonal together, as long as the longest run among them:
// a third of the lanes did work then).  A lane whose pair is decided takes the
// next one of the wave's list.
//
// Bound: the latency of a step's two LDS trips and its instruction issue,
// about 40 steps of 60 vector instructions a pair.  Measured, 250 bp unless
// said, against a lane per pair with F in registers: 4M pairs at E = 10 (333k
// survivors of SneakySnake) 130 -> 72 us, 1k pairs 44 -> 18, 500k E = 25 472 ->
// 122, 300k 500 bp E = 31 850 -> 187, 500k related pairs E = 15 773 -> 115, 4M
// 100 bp E = 3 19.0 -> 15.6.
//
// A selection (optional, e.g. the accept bits of a filter) names the pairs
// to verify; the others get E + 1.
#include <algorithm>

#include "paf_flow.h"

namespace paf {

namespace {

constexpr int kUnreached = -(1 << 14);

// A wave owns K tiles of 64 consecutive pairs and lists the ones selected (bit
// p of `sel`).
// Up to 32, or 64 where that avoids a second turn of long chains (max_E 20 and
// up): 4M pairs at E = 25 627 us in one turn, 877 in two; at E = 10 10M pairs
// 0.17 ms in three turns, 0.21 in two of longer chunks.
constexpr uint32_t kVerifyTiles = 32;
// Idle lanes that are worth the trip to memory for their next pairs' words (8
// and 16 measured the same, 32 7% slower).
constexpr int kRefill = 16;
// Waves per SIMD that a launch aims at: one / two / three / four take 81 / 71 / 72 / 72 us
// for 4M pairs at E = 10 and 20 / 18.6 / 15.6 / 14.9 us for 4M of 100 bp at E = 3,
// and three / four 147 / 131 us for 4M of 100 bp at E = 5, all selected (138 with a
// lane per pair in step); fewer where the LDS holds fewer.  Three until a wave has
// seven tiles (722k pairs of 100 bp at E = 6 12.6 us, 14.2 with four) and above
// max_E 8 (1.9M of 150 bp at E = 10 53 and 56).
uint32_t verify_waves(uint32_t n_tiles, int emax, int num_cus) {
    return n_tiles >= 7u * 16u * (uint32_t)num_cus && emax <= 8 ? 4u : 3u;
}

// Rows of F: diagonals -emax - 1 .. emax + 1.
__host__ __device__ constexpr uint32_t reach_rows(uint32_t emax) { return 2 * emax + 3; }

// Rows of words: two past the last one may be read.
__host__ __device__ constexpr uint32_t word_rows(uint32_t wmax) { return wmax + 2; }

// LDS of a wave, in the 1280-byte units it is allocated in.
constexpr size_t verify_lds_bytes(uint32_t wmax, uint32_t emax, uint32_t tiles) {
    const size_t b = (size_t)64 * (2 * word_rows(wmax) * 8 + reach_rows(emax) * 2 + tiles * 2);
    return (b + 1279) / 1280 * 1280;
}

// 32 bases of a lane's sequence from base position p on (planes lo, hi); past
// the pair's end they are any.
__device__ __forceinline__ void bases32(const uint64_t* col, uint32_t p, uint32_t& lo, uint32_t& hi) {
    const uint64_t* w = col + ((p & ~31u) << 1);
    lo = funnel((uint32_t)w[64], (uint32_t)w[0], p);
    hi = funnel((uint32_t)(w[64] >> 32), (uint32_t)(w[0] >> 32), p);
}

__global__ void __launch_bounds__(64) verify_kernel(FilterParams P, const uint32_t* sel, uint16_t* dist, uint32_t K,
                                                    uint32_t emax) {
    extern __shared__ uint64_t lds[];
    const int lane = threadIdx.x;
    const uint32_t words = word_rows(P.wmax) * 64;
    uint64_t* const rd = lds + lane;
    uint64_t* const rf = rd + words;
    int16_t* const F = reinterpret_cast<int16_t*>(lds + 2 * words) + (emax + 1) * 64 + lane;   // F[64 d]: diagonal d
    uint16_t* const list = reinterpret_cast<uint16_t*>(lds + 2 * words) + reach_rows(emax) * 64;
    const uint64_t slot0 = (uint64_t)blockIdx.x * K * 64;
    const uint32_t n_here = (uint32_t)min<uint64_t>((uint64_t)K * 64, P.n_pairs - slot0);
    uint32_t n_sel = 0;
    const uint32_t bits0 = chunk_bits(sel, slot0, min(n_here, 2048u), lane);
    const uint32_t bits1 = n_here > 2048u ? chunk_bits(sel, slot0 + 2048u, n_here - 2048u, lane) : 0u;
    constexpr uint32_t AHEAD = 4;   // tiles whose lengths and thresholds are loaded together
    for (uint32_t g0 = 0; g0 < n_here; g0 += 64 * AHEAD) {
        uint32_t ms[AHEAD], Es[AHEAD];
#pragma unroll
        for (uint32_t j = 0; j < AHEAD; ++j) {
            const uint64_t p = slot0 + min(g0 + 64 * j + (uint32_t)lane, n_here - 1u);
            ms[j] = P.len ? P.len[p] : P.uniform_len;
            Es[j] = P.E ? P.E[p] : P.uniform_E;
        }
#pragma unroll
        for (uint32_t j = 0; j < AHEAD; ++j) {
            const uint32_t g = g0 + 64 * j;
            if (g >= n_here) break;
            const uint32_t i = g + (uint32_t)lane;
            bool take = chunk_bit(g < 2048u ? bits0 : bits1, (g >> 6) & 31u, lane) && i < n_here;
            if (i < n_here) {
                if (ms[j] < 1 || ms[j] > P.max_len || Es[j] > P.max_E) {
                    atomicOr(P.err, 1u);
                    take = false;
                    dist[slot0 + i] = 0;
                } else if (!take) {
                    dist[slot0 + i] = (uint16_t)(Es[j] + 1u);
                }
            }
            const uint64_t bal = __ballot(take);
            if (take) list[n_sel + rank_in(bal)] = (uint16_t)i;
            n_sel += (uint32_t)__builtin_popcountll(bal);
        }
    }
    wave_lds_sync();

    // The lane's pair, its round k (over diagonals -reach .. reach, reach =
    // min(k, cap, E - k)), the diagonal d being walked at column c, which ends
    // at column `end`, and F_{k-1}[d].  An idle lane has m = 0 and stays at
    // column 0 of diagonal 0.
    uint64_t id = 0;
    int m = 0, E = 0, cap = 0, k = 0, d = 0, c = 0, end = 0, here = 0;
    uint32_t next = 0;
    uint64_t idle = ~0ull;
    for (;;) {
        if (next < n_sel) {
            const uint32_t at = next + rank_in(idle);
            if (m == 0 && at < n_sel) {
                id = slot0 + list[at];
                m = (int)(P.len ? P.len[id] : P.uniform_len);
                E = (int)(P.E ? P.E[id] : P.uniform_E);
                const uint64_t off = P.word_offset ? P.word_offset[id] : id * (uint64_t)P.stride_words;
                const uint64_t* gr = P.reads + off;
                const uint64_t* gf = P.refs + off;
                const int W = (m + 31) >> 5;
                int w = 0;
                for (; w + 4 <= W; w += 4) {
                    uint64_t a[4], b[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        a[j] = gr[w + j];
                        b[j] = gf[w + j];
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        rd[(w + j) * 64] = a[j];
                        rf[(w + j) * 64] = b[j];
                    }
                }
                for (; w < W; ++w) {
                    rd[w * 64] = gr[w];
                    rf[w * 64] = gf[w];
                }
                for (int j = -E - 1; j <= E + 1; ++j) F[j * 64] = (int16_t)kUnreached;
                cap = min(E, m);
                k = d = c = 0;
                end = m;
                here = kUnreached;
            }
            next = min(n_sel, next + (uint32_t)__builtin_popcountll(idle));
        } else if (idle == ~0ull) {
            break;
        }
        const int most = next < n_sel ? kRefill : 64;
        do {
            uint32_t alo, ahi, blo, bhi;
            bases32(rf, (uint32_t)c, alo, ahi);
            bases32(rd, (uint32_t)(c + d), blo, bhi);
            const uint32_t mism = or_xor(ahi, alo ^ blo, bhi);
            const int run = (int)min((uint32_t)(__builtin_ffs((int)mism) - 1), 32u);
            c = min(c + run, end);
            if (m != 0 && (mism != 0u || c >= end)) {
                F[d * 64] = (int16_t)c;
                const bool whole = d == 0 && c >= m;
                const int found = whole ? k : E + 1;
                // Diagonals beyond the pair's threshold or length stay unreachable.
                // A path on diagonal d after k edits needs |d| more to end on
                // diagonal 0, so round k only extends the diagonals with
                // k + |d| <= E: the others cannot lie on an alignment within E
                // edits (and the rounds after k only read diagonals that round k
                // kept).
                const int reach0 = min(k, min(cap, E - k));
                const bool wrap = d == reach0;
                k += wrap ? 1 : 0;
                const int reach = min(k, min(cap, E - k));
                const bool over = whole || k > E;
                d = over ? 0 : wrap ? -reach : d + 1;
                const int16_t* const f = F + d * 64;
                const int before = wrap ? f[-64] : here, after = f[64];
                here = f[0];
                end = min(m, m - d);
                c = min(max(max(here, after) + 1, before), end);
                if (over) {
                    dist[id] = (uint16_t)found;
                    m = c = end = 0;
                }
            }
            idle = __ballot(m == 0);
        } while (__builtin_popcountll(idle) < most);
    }
}

// 32 bases of one staged sequence from base position p on (planes lo, hi).
__device__ __forceinline__ void staged32(const uint64_t* rows, int lane, uint32_t p, uint32_t W, uint32_t& lo,
                                        uint32_t& hi) {
    const uint32_t k = p >> 5, sh = p & 31u;
    const uint64_t w0 = rows[k * kLdsRow + lane];
    const uint64_t w1 = k + 1 < W ? rows[(k + 1) * kLdsRow + lane] : 0ull;
    lo = funnel((uint32_t)w1, (uint32_t)w0, sh);
    hi = funnel((uint32_t)(w1 >> 32), (uint32_t)(w0 >> 32), sh);
}

// Furthest column reached on diagonal d from column x (x <= end): the run of
// matches ref[c] == read[c + d] for c = x, x+1, ... stops at the first
// mismatch or at end = min(m, m - d).
__device__ __forceinline__ int slide(const uint64_t* rdL, const uint64_t* rfL, int lane, int x, int d,
                                     int end, uint32_t W) {
    int c = x;
    while (c < end) {
        uint32_t alo, ahi, blo, bhi;
        staged32(rfL, lane, (uint32_t)c, W, alo, ahi);
        staged32(rdL, lane, (uint32_t)(c + d), W, blo, bhi);
        const uint32_t mism = (alo ^ blo) | (ahi ^ bhi);
        if (mism != 0u) {
            c += (int)__builtin_ctz(mism);
            break;
        }
        c += 32;
    }
    return min(c, end);
}

template <int EMAX>
__device__ uint32_t band_distance(const uint64_t* rdL, const uint64_t* rfL, int lane, bool act, int m, int E,
                                  uint32_t W) {
    constexpr int D = 2 * EMAX + 1;
    int F[D];
#pragma unroll
    for (int i = 0; i < D; ++i) F[i] = kUnreached;
    uint32_t dist = (uint32_t)E + 1u;
    if (act) {
        F[EMAX] = slide(rdL, rfL, lane, 0, 0, m, W);
        if (F[EMAX] >= m) dist = 0;
        if (F[EMAX] >= m || E == 0) act = false;
    }
    // Diagonals beyond the pair's threshold or length stay unreachable.  A
    // path on diagonal d after k edits needs |d| more to end on diagonal 0,
    // so round k only extends the diagonals with k + |d| <= E: the others
    // cannot lie on an alignment within E edits (and the rounds after k
    // only read diagonals that round k kept).
    const int lim = min(E, m);
    for (int k = 1; wave_any(act); ++k) {
        if (act) {
            int left = kUnreached;   // F_{k-1}[d-1]
            const int reach = min(k, min(lim, E - k));
#pragma unroll
            for (int i = 0; i < D; ++i) {
                const int d = i - EMAX;
                const int old = F[i];
                const int ad = d < 0 ? -d : d;
                if (ad <= reach) {
                    int x = old + 1;
                    if (i + 1 < D) x = max(x, F[i + 1] + 1);
                    x = max(x, left);
                    const int end = d > 0 ? m - d : m;
                    x = min(x, end);
                    F[i] = slide(rdL, rfL, lane, x, d, end, W);
                }
                left = old;
            }
            if (F[EMAX] >= m) {
                dist = (uint32_t)k;
                act = false;
            } else if (k >= E) {
                act = false;
            }
        }
    }
    return dist;
}

// Every pair of a batch, a tile of 64 per wave, its words staged in the wave's
// LDS rows, the lanes walking rounds and diagonals together.  Most pairs then
// need all E + 1 rounds, so that hardly a lane waits for another, and a step
// takes half the instructions.
template <int EMAX>
__global__ void __launch_bounds__(256) verify_step_kernel(FilterParams P, uint16_t* dist) {
    extern __shared__ uint64_t lds[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    uint64_t* rdL = lds + (size_t)wave * 2 * P.wmax * kLdsRow;
    uint64_t* rfL = rdL + (size_t)P.wmax * kLdsRow;
    const uint64_t slot0 = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + wave) * 64;
    if (slot0 >= P.n_pairs) return;
    PairSlot s;
    s.in_batch = slot0 + lane < P.n_pairs;
    s.slot = s.id = s.in_batch ? slot0 + lane : 0;
    s.m = s.in_batch ? (P.len ? P.len[s.id] : P.uniform_len) : 0u;
    s.E = s.in_batch ? (P.E ? P.E[s.id] : P.uniform_E) : 0u;
    s.valid = s.in_batch && s.m >= 1 && s.m <= P.max_len && s.E <= P.max_E;
    if (s.in_batch && !s.valid) {
        atomicOr(P.err, 1u);
        dist[s.id] = 0;
    }
    if (!s.valid) s.m = s.E = 0;
    s.W = (s.m + 31) >> 5;
    const uint64_t off = !s.valid ? 0
                         : P.word_offset ? P.word_offset[s.id]
                                         : s.id * (uint64_t)P.stride_words;
    stage_tile<true>(P, 0, lane, s, off, rdL, rfL);
    const uint32_t dd = band_distance<EMAX>(rdL, rfL, lane, s.valid, (int)s.m, (int)s.E, s.W);
    if (s.valid) dist[s.id] = (uint16_t)dd;
}

const void* verify_step_kernel_for(int emax) {
    switch (emax) {
#define PAF_CASE(X) \
    case X: return reinterpret_cast<const void*>(&verify_step_kernel<X>);
        PAF_CASE(0) PAF_CASE(1) PAF_CASE(2) PAF_CASE(3) PAF_CASE(4) PAF_CASE(5) PAF_CASE(6)
        PAF_CASE(7) PAF_CASE(8) PAF_CASE(10) PAF_CASE(12) PAF_CASE(15) PAF_CASE(20) PAF_CASE(25)
        PAF_CASE(31)
#undef PAF_CASE
        default: return nullptr;
    }
}

hipError_t launch_steps(const FilterParams& p, int emax, uint16_t* dist, hipStream_t s) {
    const void* k = verify_step_kernel_for(emax);
    if (!k) return hipErrorInvalidValue;
    const uint32_t waves = 4;
    const size_t lds = (size_t)waves * 2 * p.wmax * kLdsRow * sizeof(uint64_t);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    FilterParams arg = p;
    void* args[] = {&arg, &dist};
    return hipLaunchKernel(k, dim3((p.n_tiles + waves - 1) / waves), dim3(64 * waves), args, lds, s);
}

}  // namespace

hipError_t launch_verify(const FilterParams& p, int emax, const uint32_t* sel, uint16_t* dist, int num_cus,
                         hipStream_t s) {
    // Every pair of 10M at E = 5 / 10 / 25: 0.45 / 0.97 / 4.94 ms in step, 0.66 /
    // 1.77 / 9.05 lane by lane.
    if (sel == nullptr) return launch_steps(p, emax, dist, s);
    // All waves run at once where the tiles allow it, else in full turns: a
    // turn of few waves costs as much as a full one (4M pairs at E = 10: 96 us
    // with 2500 waves, of which the LDS holds 2304 at once; 72 with 2233).
    uint32_t K = 1;
    for (;;) {
        const uint64_t fit = 160 * 1024 / verify_lds_bytes(p.wmax, (uint32_t)emax, K);
        const uint64_t want = (uint64_t)num_cus * std::min<uint64_t>(4 * verify_waves(p.n_tiles, emax, num_cus), fit);
        const uint64_t most = want * (emax >= 20 && p.n_tiles <= want * 2 * kVerifyTiles ? 2 * kVerifyTiles : kVerifyTiles);
        const uint64_t turns = std::max<uint64_t>(1, (p.n_tiles + most - 1) / most);
        const uint32_t need = (uint32_t)((p.n_tiles + want * turns - 1) / (want * turns));
        if (need <= K) break;
        K = need;
    }
    const uint64_t chunks = (p.n_tiles + K - 1) / K;
    const size_t lds = verify_lds_bytes(p.wmax, (uint32_t)emax, K);
    verify_kernel<<<dim3((uint32_t)chunks), dim3(64), lds, s>>>(p, sel, dist, K, (uint32_t)emax);
    return hipGetLastError();
}

}  // namespace paf
