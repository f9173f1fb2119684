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
// here too, with the same count E + 1.  So the call runs SneakySnake into the caller's outputs and the kernel below
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
// by a group of lanes together, a lane per diagonal, by extracting from the
// diagonals' runs themselves.
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

// Up to this threshold the pairs that SneakySnake found free of obstacles are left
// out, which are then a large part of the accepted ones (10M related pairs of 250
// bp at E = 1, half of them equal: 1777 -> 1129 us), where a wave owns several tiles
// (the counts of one are a trip to memory more: 0.5 us of 10).
constexpr int kSkipFree = 3;

// Intervals a lane holds (related pairs have about 2 E; 112 was the most seen
// for unrelated ones).  The LDS they take bounds the waves of a CU: 128 took
// 976 us where 80 takes 742 (500k pairs, E = 25).
__host__ __device__ constexpr uint32_t magnet_intervals(int emax) { return emax <= 10 ? 40u : (emax <= 15 ? 56u : (emax <= 25 ? 80u : 96u)); }

// LDS of a wave, in the 1280-byte units it is allocated in.
constexpr uint64_t magnet_lds_bytes(int emax) {
    return (magnet_intervals(emax) * 256 + magnet_tiles(emax) * (8 + 128) + 1279) / 1280 * 1280;
}

// Interval [s, s + len): longer ones and then smaller starts are larger.
__device__ __forceinline__ uint32_t ival(uint32_t s, uint32_t len) { return (len << 10) | (1023u - s); }
__device__ __forceinline__ uint32_t ival_len(uint32_t v) { return v >> 10; }
__device__ __forceinline__ uint32_t ival_start(uint32_t v) { return 1023u - (v & 1023u); }

// Largest value of each group of G lanes (16, 32 or 64), in all of its lanes.
template <int G>
__device__ __forceinline__ uint32_t group_max(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, false));   // row_ror:1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false));
#pragma unroll
    for (int o = 16; o < G; o <<= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o));
    return v;
}

// 64 / G pairs at once, lane i of a group searching diagonal i - E of the
// group's pair (m = 0: none), whose words of free cells it keeps in its LDS
// column `x` (`pair`: the pair's read and reference words, in turn).  A pass
// over the words that any diagonal still has free cells in clears the columns
// that left the search and finds the longest run at a word's edges or over
// several; only when that is none of 31 cells or more are runs inside words
// looked for.  Returns the pair's count.
//
// Bound by instruction issue and, at one wave per SIMD, by its latency: 6 us a
// round at E = 5 (four pairs) and E = 25 (one).  100k homopolymers of 250 bp with
// two or three edits at E = 5 / 10 / 25, every pair of which comes here: 988 / 1181 /
// 1279 us with one pair a wave and its words loaded and compared again in every
// pass, 218 / 364 / 617 now (extraction over all diagonals with a lane per pair:
// 212 / 443 / 966; 400k in tandem repeats 524 / 1100 / 2190 to 666 / 1177 / 2246 here).
// The words of free cells in registers, unrolled over 16, took 335 / 644 / 882.
template <int G>
__device__ __forceinline__ uint32_t magnet_by_diagonals(const uint64_t* pair, uint32_t m, uint32_t E, int lane, uint32_t* x) {
    const int W = (int)((m + 31u) >> 5), i = lane & (G - 1), d = i - (int)E;
    const uint32_t sh = (uint32_t)d & 31u;
    const bool pos = d >= 0, on = i <= 2 * (int)E;
    const int words = __builtin_amdgcn_readfirstlane((int)group_max<64>((uint32_t)W));
    uint32_t live = 0;   // words with a free cell on some lane
    uint64_t prev = 0, cur = pair[0];
    for (int k = 0; k < words; ++k) {
        const uint64_t next = k + 1 < W ? pair[2 * (k + 1)] : 0ull, ref = pair[2 * k + 1];
        const uint32_t vp = vacant_word(k - 1, (int)m), vc = vacant_word(k, (int)m), vn = vacant_word(k + 1, (int)m);
        const uint64_t a = pos ? cur : prev, b = pos ? next : cur;
        const uint32_t lo = funnel((uint32_t)b, (uint32_t)a, sh), hi = funnel((uint32_t)(b >> 32), (uint32_t)(a >> 32), sh);
        const uint32_t v = funnel(pos ? vn : vc, pos ? vc : vp, sh);
        const uint32_t w = on ? ~((lo ^ (uint32_t)ref) | (hi ^ (uint32_t)(ref >> 32)) | v | vc) : 0u;
        x[64 * k] = w;
        live |= wave_any(w != 0u) ? 1u << k : 0u;
        prev = cur;
        cur = next;
    }
    // f(k, word k), the next live word on its way.
    auto each_live = [&](auto f) {
        uint32_t rest = live, k = rest ? (uint32_t)__builtin_ctz(rest) : 0u, ahead = x[64 * k];
        while (rest != 0u) {
            const uint32_t w = ahead, at = k;
            rest &= rest - 1u;
            k = rest ? (uint32_t)__builtin_ctz(rest) : at;
            ahead = x[64 * k];
            f(at, w);
        }
    };
    bool open = m != 0u, rejected = false;
    uint32_t covered = 0, it = 0, from = 0, upto = 0;   // columns [from, upto) leave the search
    while (wave_any(open)) {
        uint32_t best = 0, carry = 0, next = 0;
        each_live([&](uint32_t k, uint32_t old) {
            if (k != next) {
                best = max(best, ival(32u * next - carry, carry));
                carry = 0;
            }
            next = k + 1u;
            const uint32_t w = old & ~cols_mask((int)k, from, upto);
            x[64 * k] = w;
            if (!wave_any(w != 0u)) live ^= 1u << k;
            const uint32_t head = min((uint32_t)__builtin_ffs((int)~w) - 1u, 32u);
            best = max(best, ival(32u * k - carry, carry + head));
            carry = w == ~0u ? carry + 32u : (uint32_t)__builtin_clz(~w);
        });
        best = max(best, ival(32u * next - carry, carry));
        best = group_max<G>(best);
        if (wave_any(open && ival_len(best) < 31u)) {
            each_live([&](uint32_t k, uint32_t w) {
                uint32_t L, s;
                word_longest(w, L, s);   // (a full word: 31, less than the run it is part of)
                best = max(best, ival(32u * k + s, L));
            });
            best = group_max<G>(best);
        }
        const uint32_t L = ival_len(best), s = ival_start(best);
        if (L == 0u) {
            open = false;
        } else if (open) {
            ++it;
            covered += L;
            from = s > 0u ? s - 1u : 0u;
            upto = s + L + 1u;
            rejected = covered + (E + 1u - it) * L + E < m;
            open = !rejected && it <= E;
        }
        if constexpr (G == 64) {
            from = (uint32_t)__builtin_amdgcn_readfirstlane((int)from);
            upto = (uint32_t)__builtin_amdgcn_readfirstlane((int)upto);
        }
    }
    return rejected ? E + 1u : min(m - covered, E + 1u);
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
    for (uint32_t j = (uint32_t)lane; j < 2 * K; j += 64) acc[j] = 0u;
    wave_lds_sync();
    constexpr uint32_t AHEAD = 8;   // tiles whose counts are loaded together
    uint32_t counts[EMAX <= kSkipFree ? AHEAD : 1];
    for (uint32_t g = 0; g < n_here; g += 64) {
        const uint32_t i = g + (uint32_t)lane;
        bool take = chunk_bit(bits, g >> 6, lane) && i < n_here;
        if (EMAX <= kSkipFree && K > 1) {
            // A pair that SneakySnake crossed without an obstacle is one run.
            const uint32_t t = (g >> 6) % AHEAD;
            if (t == 0u) {
#pragma unroll
                for (uint32_t j = 0; j < AHEAD; ++j) counts[j] = P.cnt[0][slot0 + min(i + 64 * j, n_here - 1u)];
            }
            uint32_t c = 0;
#pragma unroll
            for (uint32_t j = 0; j < AHEAD; ++j) c = j == t ? counts[j] : c;
            const uint64_t free = __ballot(take && c == 0u);
            if (lane < 2) acc[2 * (g >> 6) + lane] = lane ? (uint32_t)(free >> 32) : (uint32_t)free;
            take = take && c != 0u;
        }
        const uint64_t bal = __ballot(take);
        if (take) list[end + rank_in(bal)] = (uint16_t)i;
        end += (uint32_t)__builtin_popcountll(bal);
    }
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
        // The pairs left, 64 / G at a time: lane i of a group loads words i of
        // its pair (a round ahead), which the group then reads from the LDS.
        constexpr int G = D <= 16 ? 16 : (D <= 32 ? 32 : 64);
        constexpr uint32_t WORDS = PAF_MAX_LEN / 32;
        static_assert(G >= WORDS && CAP >= WORDS + 4, "a lane per word; a pair's words and its diagonals' in the intervals' place");
        uint64_t* const staged = reinterpret_cast<uint64_t*>(iv + 64 * WORDS);   // [64][read, reference]
        uint64_t rest = __ballot(together), wr = 0, wf = 0;
        uint32_t jm = 0, jE = 0, jat = 0;
        auto fetch = [&]() {
            int src = -1;   // lane whose pair this one's group takes
#pragma unroll
            for (int j = 0; j < 64 / G; ++j) {
                if (rest != 0ull && lane / G == j) src = __builtin_ctzll(rest);
                rest &= rest - 1;
            }
            const int of = max(src, 0);
            const uint64_t jo = ((uint64_t)(uint32_t)__shfl((int)(off >> 32), of) << 32) | (uint32_t)__shfl((int)(uint32_t)off, of);
            jm = (uint32_t)__shfl((int)m, of);
            jE = (uint32_t)__shfl((int)E, of);
            jat = (uint32_t)__shfl((int)at, of);
            if (src < 0) jm = 0;
            const uint32_t word = (uint32_t)lane % G;
            wr = wf = 0;
            if (word < ((jm + 31u) >> 5)) {
                wr = P.reads[jo + word];
                wf = P.refs[jo + word];
            }
        };
        bool more = rest != 0ull;
        if (more) fetch();
        while (more) {
            wave_lds_sync();
            staged[2 * lane] = wr;
            staged[2 * lane + 1] = wf;
            wave_lds_sync();
            const uint32_t gm = jm, gE = jE, gat = jat;
            more = rest != 0ull;
            if (more) fetch();
            const uint32_t count = magnet_by_diagonals<G>(staged + 2 * (lane / G * G), gm, gE, lane, iv + lane);
            if (gm != 0u && lane % G == 0) {
                P.cnt[0][slot0 + gat] = (uint16_t)count;
                if (count <= gE) atomicOr(&acc[gat >> 5], 1u << (gat & 31u));
            }
        }
        wave_lds_sync();
    }
    wave_lds_sync();
    for (uint32_t j = (uint32_t)lane; 32u * j < n_here; j += 64) P.acc[0][(slot0 >> 5) + j] = acc[j];
}

// max_E 0: the one run that counts is the main diagonal's, all of it, so a pair
// is accepted when its words are equal.  Bound by HBM: rows are read as they lie,
// a word a lane, and a lane whose word differs marks its pair (a lane per pair
// reads rows apart, whose lines leave the L1 between its loads: 10M pairs of 250
// bp 307 us, 216 this way).  A wave takes 512 words of a batch of one length, or a
// tile whose rows are of wmax words.
constexpr uint32_t kExactTiles = 8;
__host__ __device__ __forceinline__ uint32_t exact_tiles(bool general, uint32_t stride) {
    return general || stride >= kExactTiles ? 1u : kExactTiles / stride;
}
template <bool GENERAL>
__global__ void __launch_bounds__(256) magnet_exact_kernel(FilterParams P) {
    constexpr int B = 8;   // words on their way
    __shared__ uint32_t marks[4][kExactTiles * 64];
    const int lane = threadIdx.x & 63;
    uint32_t* const differs = marks[threadIdx.x >> 6];
    const uint32_t T = exact_tiles(GENERAL, P.stride_words);
    const uint64_t tile = ((uint64_t)blockIdx.x * 4u + (threadIdx.x >> 6)) * T;
    if (tile >= P.n_tiles) return;
    const uint32_t n_here = (uint32_t)min<uint64_t>(64u * T, P.n_pairs - tile * 64);
    for (uint32_t i = 0; i < T; ++i) differs[64 * i + lane] = 0u;
    // The bits that count of a pair's last word.
    auto kept = [](uint32_t m) -> uint64_t {
        const uint64_t x = (1ull << (m & 31u)) - 1ull;
        return x ? x << 32 | x : ~0ull;
    };
    uint64_t off = 0;
    PairSlot ps = {};
    if constexpr (GENERAL) ps = load_slot<true>(P, tile, lane, off);
    const uint32_t S = GENERAL ? P.wmax : P.stride_words, rows = GENERAL ? 64u : n_here;
    const uint64_t base = tile * 64 * (uint64_t)S;
    uint32_t pr = (uint32_t)lane / S, k = (uint32_t)lane - pr * S;
    const uint32_t dp = 64u / S, dk = 64u - dp * S;
    wave_lds_sync();
    while (wave_any(pr < rows)) {
        uint64_t x[B], y[B], keep[B];
        uint32_t at[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            uint32_t m = P.uniform_len;
            uint64_t a = base + (uint64_t)pr * S + k;
            if constexpr (GENERAL) {
                const int of = (int)min(pr, 63u);
                m = (uint32_t)__shfl((int)ps.m, of);   // (0: no pair there, or one out of range)
                a = ((uint64_t)(uint32_t)__shfl((int)(off >> 32), of) << 32 | (uint32_t)__shfl((int)(uint32_t)off, of)) + k;
            }
            const uint32_t W = (m + 31u) >> 5;
            const bool ok = pr < rows && k < W;
            x[b] = P.reads[ok ? a : 0ull];
            y[b] = P.refs[ok ? a : 0ull];
            keep[b] = !ok ? 0ull : k + 1u == W ? kept(m) : ~0ull;
            at[b] = pr;
            pr += dp;
            k += dk;
            if (k >= S) { k -= S; pr += 1; }
        }
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (((x[b] ^ y[b]) & keep[b]) != 0ull) differs[at[b]] = 1u;
    }
    wave_lds_sync();
    for (uint32_t i = 0; 64u * i < n_here; ++i) {
        const uint32_t j = 64u * i + (uint32_t)lane;
        const bool valid = GENERAL ? ps.valid : j < n_here, diff = differs[j] != 0u;
        const uint64_t bal = __ballot(valid && !diff);
        if (j < n_here) P.cnt[0][tile * 64 + j] = valid && diff ? 1 : 0;
        if (lane < 2 && 64u * i + 32u * lane < n_here)
            P.acc[0][2 * (tile + i) + lane] = lane ? (uint32_t)(bal >> 32) : (uint32_t)bal;
    }
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

hipError_t launch_magnet_exact(const FilterParams& p, hipStream_t s) {
    const bool general = p.len || p.E || p.word_offset;
    const uint32_t T = exact_tiles(general, p.stride_words);
    const dim3 grid((uint32_t)(((uint64_t)p.n_tiles + 4 * T - 1) / (4 * T)));
    if (general) magnet_exact_kernel<true><<<grid, dim3(256), 0, s>>>(p);
    else magnet_exact_kernel<false><<<grid, dim3(256), 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_magnet(const FilterParams& p, int emax, int num_cus, hipStream_t s) {
    const void* k = magnet_kernel_for(emax);
    if (!k) return hipErrorInvalidValue;
    const uint64_t want = (uint64_t)num_cus * 4 * kWavesPerSimd;
    uint32_t K = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(magnet_tiles(emax), p.n_tiles / want));
    if (emax >= 12 && K > 1) {
        // The LDS holds eight to six of these waves on a CU: where the last turn
        // would run few, longer chunks take one turn less (400k homopolymers of
        // 250 bp at E = 25 2821 -> 2263 us; of the usual mix 1.5M pairs at E = 25
        // 1816 -> 1443 and 500k at E = 15 291 -> 207).  Not where it would run half (500k
        // at E = 25 652 -> 689), nor chunks of one tile (140k related pairs 559 -> 627).
        const uint64_t most = (uint64_t)num_cus * std::min<uint64_t>(4 * kWavesPerSimd, 160 * 1024 / magnet_lds_bytes(emax));
        const uint64_t chunks = (p.n_tiles + K - 1) / K, turns = chunks / most;
        if (turns >= 1 && (chunks - turns * most) * 5 < 2 * most)
            K = (uint32_t)std::min<uint64_t>(magnet_tiles(emax), (p.n_tiles + turns * most - 1) / (turns * most));
    }
    const uint64_t chunks = (p.n_tiles + K - 1) / K;
    FilterParams arg = p;
    void* args[] = {&arg, &K};
    return hipLaunchKernel(k, dim3((uint32_t)chunks), dim3(64), args, 0, s);
}

}  // namespace paf
