// MAGNET decision stage (Ch. 7) on the neighbourhood map of Ch. 6 (vacant
// cells blocked).  Extraction: the longest run of free cells over all 2E+1
// diagonals among the columns still in the search space (ties: the smallest
// start column, then the first diagonal in order -E..E).  Encapsulation: the
// run's columns and one column on each side leave the search space of every
// diagonal.  The search repeats, longest run first, until E + 1 runs are
// found or no free cell is left (the hardware form of Sec. 7.4: one problem
// of fixed size, excluded columns set to ones).  count = min(m - covered,
// E + 1), accept = count <= E.
//
// SneakySnake decides most pairs first: MAGNET's runs leave a column between
// them, so when they cover m - E columns or more, the columns they leave out
// are at most E obstacles of a path through the maze; SneakySnake, which finds
// the fewest obstacles, then accepts the pair.  A pair it rejects is rejected
// here too, with the same count E + 1 (and with E = 0 it decides every pair).
// So the call runs SneakySnake into the caller's outputs and the kernel below
// on the pairs whose accept bit is set: 8% of the 250 bp workload at E = 10,
// where a test of each diagonal for a run of m / (E + 1) free cells (Sec. 7.2's
// first test) took longer than SneakySnake does and left 33%.
//
// The longest runs do not need the diagonals apart: with reach(s) the end of
// the longest run that starts at column s on any diagonal, the search only
// sees the intervals [s, reach(s)) that lie in no other one.  Every run inside
// the columns still searched is part of such an interval clipped to them, a
// clipped interval is a run, and the best run of all (the smallest start among
// the longest) is one of them.  They come in order of both ends, so they are
// found by probing forward from a start s for the obstacle R (as SneakySnake
// does) and back from R for the smallest start of a run through R, the next
// interval's; a column no run passes is skipped.  A survivor of SneakySnake has
// few: every interval but its path's own holds one of at most E obstacles.
// An extraction takes the longest interval and clips the others (never from
// both sides at once, which would need a longer one).
//
// A wave owns a chunk of tiles, lists its selected pairs in LDS and takes them
// 64 at a time, one lane per pair: first the intervals, window by window, every
// lane's window at its own column, into LDS; then the extractions.  A pair with
// more intervals than a lane's part of the LDS holds, or with two runs that
// overlap by more than kBack columns at a long run's end (repeats), is done
// by the wave together, a lane per diagonal, by extracting from the diagonals'
// runs themselves.
//
// Bound: the serial chain of a group (about 25 windows of its longest pair, each
// a trip to memory and 2E + 1 diagonals of shifts and compares, then E + 1
// passes over its intervals), 60 us at E = 10, with two waves per SIMD to
// hide it.  Measured, SneakySnake included, 250 bp unless said, against a test
// kernel, a sort and an extraction over all diagonals' runs with a pair's words
// in registers: 1k pairs E = 10 186 -> 69 us, 1M E = 10 467 -> 174, 4M E = 7
// 885 -> 328, 500k E = 25 926 -> 693, 300k 400 bp E = 31 1355 -> 968, 500k
// related pairs of 100 to 250 bp 979 -> 501.
#include <algorithm>

#include "paf_flow.h"

namespace paf {

namespace {

// Longest run of ones inside one word x != ~0 and its lowest start.
__device__ __forceinline__ void word_longest(uint32_t x, uint32_t& L, uint32_t& s) {
    const uint32_t a1 = x;
    const uint32_t a2 = a1 & (a1 >> 1);
    const uint32_t a4 = a2 & (a2 >> 2);
    const uint32_t a8 = a4 & (a4 >> 4);
    const uint32_t a16 = a8 & (a8 >> 8);
    uint32_t cur = ~0u, len = 0;
    uint32_t c;
    c = cur & (a16 >> len); if (c) { cur = c; len += 16; }
    c = cur & (a8 >> len);  if (c) { cur = c; len += 8; }
    c = cur & (a4 >> len);  if (c) { cur = c; len += 4; }
    c = cur & (a2 >> len);  if (c) { cur = c; len += 2; }
    c = cur & (a1 >> len);  if (c) { cur = c; len += 1; }
    L = len;
    s = len ? (uint32_t)__builtin_ctz(cur) : 0u;
}

// Bits of word k for the columns at or above t (a clamp and one shift of
// a 64-bit constant, whose low half is zero once t passes the word).
__device__ __forceinline__ uint32_t cols_from(int k, uint32_t t) {
    const int x = min(max((int)t - 32 * k, 0), 32);
    return (uint32_t)(0xFFFFFFFFull << x);
}

// Bits of columns [a, b) that fall in word k.
__device__ __forceinline__ uint32_t cols_mask(int k, uint32_t a, uint32_t b) {
    return cols_from(k, a) & ~cols_from(k, b);
}

// Most tiles a wave owns: 4M pairs at E = 7 352 us with 16, 328 with 32; 300k at
// E = 31 1061 and 1086 (the longer list takes LDS a further wave would use).
__host__ __device__ constexpr uint32_t magnet_tiles(int emax) { return emax <= 15 ? 32u : 16u; }
constexpr uint32_t kBack = 24;          // columns searched back from a long run's end

// Most intervals found in one window (lanes that have more wait for the next
// one, the others do not wait for them).  At E = 25 three against two: 733 and
// 748 us for 500k pairs; at E = 10 two: 176 against 180 us for 1M.
constexpr uint32_t magnet_per_window(int emax) { return emax <= 15 ? 2u : 3u; }

// Waves per SIMD a launch aims at: 1 / 2 / 3 / 4 took 247 / 180 / 210 / 278 us
// for 1M pairs at E = 10, whose 8% of survivors then fill fewer lanes of each
// group, and 1748 / 1345 / 1239 / 1116 us for 500k related pairs at E = 25,
// which nearly all survive.
constexpr uint64_t kWavesPerSimd = 2;

// Intervals a lane holds (related pairs have about 2 E; 112 was the most seen
// for unrelated ones).  The LDS they take bounds the waves of a CU: 128 took
// 976 us where 80 takes 742 (500k pairs, E = 25).
__host__ __device__ constexpr uint32_t magnet_intervals(int emax) { return emax <= 10 ? 40u : (emax <= 15 ? 56u : (emax <= 25 ? 80u : 96u)); }

// Interval [s, s + len): longer ones and then smaller starts are larger.
__device__ __forceinline__ uint32_t ival(uint32_t s, uint32_t len) { return (len << 10) | (1023u - s); }
__device__ __forceinline__ uint32_t ival_len(uint32_t v) { return v >> 10; }
__device__ __forceinline__ uint32_t ival_start(uint32_t v) { return 1023u - (v & 1023u); }

// One pair by the whole wave: lane i searches diagonal i - E.  gone: the
// columns that left the search (one word per lane 0..15).
__device__ __noinline__ uint32_t magnet_pair_by_wave(const uint64_t* rd, const uint64_t* rf, uint32_t m, uint32_t E, int lane) {
    const int W = (int)((m + 31u) >> 5), d = lane - (int)E;
    const uint32_t sh = (uint32_t)d & 31u;
    uint32_t gone = vacant_word(lane, (int)m), covered = 0, it = 0;
    for (;;) {
        uint32_t best = 0, carry = 0;
        for (int k = 0; k < W; ++k) {
            const uint32_t out = (uint32_t)__shfl((int)gone, k);
            const WindowWords q = window_words_direct(rd, rf, k, W, (int)m);
            const bool pos = d >= 0;
            const uint32_t lo = funnel(pos ? q.nlo : q.clo, pos ? q.clo : q.plo, sh);
            const uint32_t hi = funnel(pos ? q.nhi : q.chi, pos ? q.chi : q.phi, sh);
            const uint32_t v = funnel(pos ? q.vn : q.vc, pos ? q.vc : q.vp, sh);
            const uint32_t x = lane <= 2 * (int)E ? ~((lo ^ q.flo) | (hi ^ q.fhi) | v | out) : 0u;
            const uint32_t t = x == ~0u ? 32u : (uint32_t)__builtin_ctz(~x);
            best = max(best, ival(32u * k - carry, carry + t));
            if (x != ~0u) {
                uint32_t L, s;
                word_longest(x, L, s);
                best = max(best, ival(32u * k + s, L));
            }
            carry = x == ~0u ? carry + 32u : (uint32_t)__builtin_clz(~x);
        }
        best = max(best, ival(32u * W - carry, carry));
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) best = max(best, (uint32_t)__shfl_xor((int)best, o));
        const uint32_t L = ival_len(best), s = ival_start(best);
        if (L == 0u) break;
        ++it;
        covered += L;
        gone |= cols_mask(lane, s > 0u ? s - 1u : 0u, min(s + L + 1u, m));
        if (it > E) break;
    }
    return min(m - covered, E + 1u);
}

template <int EMAX>
__global__ void __launch_bounds__(64) magnet_kernel(FilterParams P, uint32_t K) {
    constexpr int D = 2 * EMAX + 1;
    constexpr uint32_t CAP = magnet_intervals(EMAX);
    using DT = typename DeadMask<EMAX>::T;
    __shared__ uint32_t iv[CAP * 64];
    __shared__ uint32_t acc[magnet_tiles(EMAX) * 2];
    __shared__ uint16_t list[magnet_tiles(EMAX) * 64];
    const int lane = threadIdx.x;
    const uint64_t slot0 = (uint64_t)blockIdx.x * K * 64;
    const uint32_t n_here = (uint32_t)min<uint64_t>((uint64_t)K * 64, P.n_pairs - slot0);
    uint32_t end = 0;
    const uint32_t bits = chunk_bits(P.acc[0], slot0, n_here, lane);
    for (uint32_t g = 0; g < n_here; g += 64) {
        const uint32_t i = g + (uint32_t)lane;
        const bool take = chunk_bit(bits, g >> 6, lane) && i < n_here;
        const uint64_t bal = __ballot(take);
        if (take) list[end + rank_in(bal)] = (uint16_t)i;
        end += (uint32_t)__builtin_popcountll(bal);
    }
    for (uint32_t j = (uint32_t)lane; j < 2 * K; j += 64) acc[j] = 0u;
    wave_lds_sync();

    for (uint32_t g = 0; g < end; g += 64) {
        const bool mine = g + (uint32_t)lane < end;
        const uint32_t at = mine ? list[g + lane] : 0u;
        const uint64_t id = slot0 + at;
        const uint32_t m = mine ? (P.len ? P.len[id] : P.uniform_len) : 1u;
        const uint32_t E = mine ? (P.E ? P.E[id] : P.uniform_E) : 0u;
        const uint64_t off = !mine ? 0ull : P.word_offset ? P.word_offset[id] : id * (uint64_t)P.stride_words;
        const int W = (int)((m + 31u) >> 5);

        // The intervals.  s: start of the one being found; c: column of the
        // window; back: its end R, when the window was set to search back
        // from R (~0: none).  Inside a long run c lies past s, and `dead` marks
        // the diagonals whose runs from s ended before the window.
        uint32_t n = 0, s = 0, c = 0, back = ~0u;
        DT dead = 0;
        bool busy = mine, together = false;
        while (wave_any(busy)) {
            FlowWords q = flow_load<false>(P.reads + off, P.refs + off, c, W);
            flow_vacancy(q, c, m - c);
            uint32_t M[D];
            flow_map<EMAX, true>(q, E, dead, M);
            bool go = busy, inside = c > s && back == ~0u, run_on = false;
            // Back from the obstacle bit t of a window: the lowest start bit
            // of a run through it (t's own next bit when no run passes).
            auto search_back = [&](uint32_t t) -> uint32_t {
                const uint32_t upto = t | (t - 1u);
                uint32_t z0 = ~0u, z1 = ~0u;
#pragma unroll
                for (int d = 0; d < D; d += 2) {
                    z0 = min(z0, ~M[d] & upto);
                    if (d + 1 < D) z1 = min(z1, ~M[d + 1] & upto);
                }
                return min(z0, z1);
            };
            if (wave_any(go && back != ~0u)) {
                const bool it = go && back != ~0u;
                const uint32_t z = search_back(it ? 1u << (back - c) : 1u);
                if (it) {
                    // (0: a run through R fills the window too)
                    if (z == 0u) {
                        together = true;
                        busy = go = false;
                    } else {
                        s = c + 32u - (uint32_t)__builtin_clz(z);
                        if (s >= m) busy = go = false;
                    }
                    back = ~0u;
                }
            }
#pragma unroll 1
            for (uint32_t p = 0; p < magnet_per_window(EMAX) && wave_any(go); ++p) {
                const uint32_t b = inside ? 1u : 1u << (s - c);
                uint32_t r0 = 0, r1 = 0;
#pragma unroll
                for (int d = 0; d < D; d += 2) {
                    r0 = or_andn(r0, M[d], M[d] + b);
                    if (d + 1 < D) r1 = or_andn(r1, M[d + 1], M[d + 1] + b);
                }
                const uint32_t t = (r0 | r1) + b;   // the obstacle's bit, 0: none in the window
                const uint32_t z = search_back(t ? t : 1u);
                if (go) {
                    const uint32_t R = t ? c + (uint32_t)__builtin_ctz(t) : c + 32u;
                    const bool last = R >= m;
                    if (t != 0u || last) {
                        const uint32_t len = min(R, m) - s;
                        if (len > 0u) {
                            if (n < CAP) iv[n * 64 + lane] = ival(s, len);
                            else together = true;
                            ++n;
                        }
                    }
                    if (last || together) {
                        busy = go = false;
                    } else if (t == 0u) {
                        // On to the window's end and beyond: from s again, or
                        // past the window when s is its first column.
                        run_on = inside || s == c;
                        if (!run_on) c = s;
                        go = false;
                    } else if (inside && z <= 1u) {
                        // The next run starts before this window (whose first
                        // column shows only this run's diagonals).
                        back = R;
                        c = max(s + 1u, R > kBack ? R - kBack : 0u);
                        go = false;
                    } else {
                        s = c + 32u - (uint32_t)__builtin_clz(z);
                        inside = false;
                        if (s >= m) {
                            busy = go = false;
                        } else if (s >= c + 32u) {
                            c = s;
                            go = false;
                        }
                    }
                }
            }
            if (go) c = s;   // more intervals in this window: next turn, from here
            DT nd = 0;
            if (wave_any(run_on)) {
                // The run from the window's first column goes on exactly on
                // the diagonals that are free throughout.
                uint32_t lo = 0, hi = 0;
#pragma unroll
                for (int d = D - 1; d >= 0; --d) {
                    uint32_t sum;
                    const uint32_t cy = __builtin_add_overflow(M[d], 1u, &sum) ? 1u : 0u;
                    if (d >= 32) hi = hi + hi + cy;
                    else lo = lo + lo + cy;
                }
                const DT alive = (DT)lo | (sizeof(DT) > 4 ? (DT)((uint64_t)hi << 32) : (DT)0);
                constexpr DT all = (D >= 8 * (int)sizeof(DT)) ? ~(DT)0 : (((DT)1 << D) - 1);
                if (run_on) {
                    nd = (DT)(~alive & all);
                    c += 32u;
                }
            }
            dead = nd;
            if (!busy) {
                s = c = 0;
                back = ~0u;
            }
        }

        // The extractions: the longest interval's columns and one on each side
        // leave the search, the others are clipped.
        bool open = mine && !together;
        uint32_t covered = 0, it = 0, lo = 0, hi = 0, n_max = open ? min(n, CAP) : 0u;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) n_max = max(n_max, (uint32_t)__shfl_xor((int)n_max, o));
        const uint32_t n_all = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_max);
        bool rejected = false;
        while (wave_any(open)) {
            uint32_t best = 0;
#pragma unroll 4
            for (uint32_t j = 0; j < n_all; ++j) {
                uint32_t v = open && j < n ? iv[j * 64 + lane] : 0u;
                const uint32_t a = ival_start(v), b = a + ival_len(v);
                if (a < hi && b > lo) {
                    v = a < lo ? ival(a, lo - a) : (b > hi ? ival(hi, b - hi) : 0u);
                    iv[j * 64 + lane] = v;
                }
                best = max(best, ival_len(v) ? v : 0u);
            }
            if (open) {
                const uint32_t L = ival_len(best), x = ival_start(best);
                if (L == 0u) {
                    open = false;
                } else {
                    ++it;
                    covered += L;
                    lo = x > 0u ? x - 1u : 0u;
                    hi = x + L + 1u;
                    // The E + 1 - it runs still to come are no longer than this one.
                    rejected = covered + (E + 1u - it) * L + E < m;
                    open = !rejected && it <= E;
                }
            }
        }
        if (mine && !together) {
            const uint32_t count = rejected ? E + 1u : min(m - covered, E + 1u);
            P.cnt[0][id] = (uint16_t)count;
            if (count <= E) atomicOr(&acc[at >> 5], 1u << (at & 31u));
        }
        for (uint64_t rest = __ballot(together); rest != 0ull; rest &= rest - 1) {
            const int src = __builtin_ctzll(rest);
            const uint32_t jm = (uint32_t)__shfl((int)m, src), jE = (uint32_t)__shfl((int)E, src);
            const uint64_t jo = ((uint64_t)(uint32_t)__shfl((int)(off >> 32), src) << 32) | (uint32_t)__shfl((int)(uint32_t)off, src);
            const uint32_t count = magnet_pair_by_wave(P.reads + jo, P.refs + jo, jm, jE, lane);
            if (lane == src) {
                P.cnt[0][id] = (uint16_t)count;
                if (count <= E) atomicOr(&acc[at >> 5], 1u << (at & 31u));
            }
        }
        wave_lds_sync();
    }
    wave_lds_sync();
    for (uint32_t j = (uint32_t)lane; 32u * j < n_here; j += 64) P.acc[0][(slot0 >> 5) + j] = acc[j];
}

const void* magnet_kernel_for(int emax) {
    switch (emax) {
#define PAF_CASE(X) \
    case X: return reinterpret_cast<const void*>(&magnet_kernel<X>);
        PAF_CASE(1) PAF_CASE(2) PAF_CASE(3) PAF_CASE(4) PAF_CASE(5) PAF_CASE(6)
        PAF_CASE(7) PAF_CASE(8) PAF_CASE(10) PAF_CASE(12) PAF_CASE(15) PAF_CASE(20) PAF_CASE(25)
        PAF_CASE(31)
#undef PAF_CASE
        default: return nullptr;
    }
}

}  // namespace

hipError_t launch_magnet(const FilterParams& p, int emax, int num_cus, hipStream_t s) {
    const void* k = magnet_kernel_for(emax);
    if (!k) return hipErrorInvalidValue;
    const uint64_t want = (uint64_t)num_cus * 4 * kWavesPerSimd;
    uint32_t K = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(magnet_tiles(emax), p.n_tiles / want));
    const uint64_t chunks = (p.n_tiles + K - 1) / K;
    FilterParams arg = p;
    void* args[] = {&arg, &K};
    return hipLaunchKernel(k, dim3((uint32_t)chunks), dim3(64), args, 0, s);
}

}  // namespace paf
