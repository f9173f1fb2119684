// SneakySnake of small batches and of most with per-pair lengths (Ch. 8, Sec.
// 8.4; which ones: snake_engine): one lane per pair, every lane's 32-column
// window starting at its own snake's column.
//
// A wave owns every `waves`-th tile of the batch (so that the whole grid walks
// the batch front to back) and its lanes take the pairs in order: a lane whose
// pair is decided takes the next one, so no lane waits for the slowest pair of
// its tile or for the other lanes' windows.  Each turn builds the match words
// of one window and probes it a fixed number of times; a snake that crossed
// fewer columns than the window holds gets its next window from where it
// stands, which costs less than letting the wave probe on for its slowest lane.
//
// Against the compacting engine (10M pairs of 250 bp, E = 10): 11% fewer VALU
// instructions and 21% more of their lanes active, but every window's words
// are loaded from the L2 (about four L1 misses a pair; the compacting engine,
// whose first two windows come from one load, has about two), and the misses
// bound it: eight waves per CU run no slower than sixteen.  So it is the
// faster one where a batch is too small to fill the chip with the compacting
// engine's chunks, whose waves walk four to six tiles one after another (250
// bp, E = 10: 100k pairs 46 -> 18 us, 1M pairs 85 -> 71 us, but 2M pairs 121 ->
// 125 us and 10M pairs 470 -> 584 us; E = 0 at 1M 28 -> 25, E = 31 at 1M pairs of
// 400 bp 463 -> 356 us), and where lengths and thresholds differ from lane to
// lane, so that a group of 64 pairs is as slow as its longest (uneven mix: 20k
// pairs 66 -> 18, 200k 79 -> 36, 2M 182 -> 147, 5M 375 -> 330 us).
#include <algorithm>

#include "paf_flow.h"

namespace paf {

namespace {

constexpr uint32_t kRing = 1024;   // counts a wave holds in LDS until their tile is complete
constexpr uint32_t kMeta = 128;    // GENERAL: pairs whose offset, length and threshold are staged ahead

// Probes from bit 0 of the window (b = 1; 0: an idle lane): each finds the
// deepest pipe from its start bit b, whose run plus b is the obstacle's bit
// (0 when the pipe runs through the window's end), and the next one starts
// one column after it.  A lane whose window is used up probes nothing more
// (b = 0).  Returns the obstacles crossed; b: the next start.
template <int D>
__device__ __forceinline__ uint32_t flow_probe(const uint32_t* M, uint32_t probes, uint32_t& b) {
    uint32_t obst = 0;
#pragma unroll 1
    for (uint32_t p = 0; p < probes; ++p) {
        uint32_t r0 = 0, r1 = 0;
#pragma unroll
        for (int d = 0; d < D; d += 2) {
            r0 = or_andn(r0, M[d], M[d] + b);
            if (d + 1 < D) r1 = or_andn(r1, M[d + 1], M[d + 1] + b);
        }
        const uint32_t t = (r0 | r1) + b;
        obst |= t;
        b = t + t;
    }
    return obst;
}

template <bool GENERAL>
struct FlowLds {
    uint64_t off[GENERAL ? kMeta : 1];
    uint32_t mE[GENERAL ? kMeta : 1];      // length, threshold << 16, in range << 31
    uint16_t cnt[kRing];                   // count, bit 15: accepted
};

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

constexpr int kFlowWaves = 4;   // waves per block
// SAMPLED: the launch runs only if the batch's lengths differ (a kernel of its own:
// with the question in the general one its loop ran 2 to 5% slower).
template <int EMAX, bool GENERAL, bool SAMPLED = false>
__global__ void __launch_bounds__(64 * kFlowWaves) __attribute__((amdgpu_waves_per_eu(EMAX <= 5 ? 8 : 4)))
flow_kernel(FilterParams P) {
    constexpr int D = 2 * EMAX + 1;
    using DT = typename DeadMask<EMAX>::T;
    __shared__ FlowLds<GENERAL> lds[kFlowWaves];
    const int lane = threadIdx.x & 63;
    if constexpr (SAMPLED)
        if (!lengths_differ(P, lane)) return;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    FlowLds<GENERAL>& L = lds[wave];
    // The wave's share: tiles first, first + waves, first + 2 waves, ...
    const uint32_t first = blockIdx.x * kFlowWaves + (uint32_t)wave;
    if (first >= P.waves) return;
    const uint32_t n_mine = (P.n_tiles - first + P.waves - 1) / P.waves;
    const uint64_t past = (uint64_t)P.n_tiles * 64u - P.n_pairs;
    const uint32_t n_here = n_mine * 64u - (first + (n_mine - 1u) * P.waves == P.n_tiles - 1u ? (uint32_t)past : 0u);
    auto slot_of = [&](uint32_t i) { return ((uint64_t)(i >> 6) * P.waves + first) * 64u + (i & 63u); };

    // Pairs [0, issued) of the share were taken by a lane, [0, flushed) are
    // written; GENERAL: offset, length and threshold of pairs [0, known) are
    // in LDS and those of the next 64 on their way.
    uint32_t issued = 0, flushed = 0, known = 0;
    uint64_t p_off = 0;
    uint32_t p_mE = 0;
    auto fetch_meta = [&]() {
        const uint32_t i = known + (uint32_t)lane;
        if (i < n_here) {
            const uint64_t id = slot_of(i);
            const uint32_t m = P.len ? P.len[id] : P.uniform_len;
            const uint32_t E = P.E ? P.E[id] : P.uniform_E;
            p_off = P.word_offset ? P.word_offset[id] : id * (uint64_t)P.stride_words;
            p_mE = m | (E << 16);
        }
    };
    auto keep_meta = [&]() {
        if (known + (uint32_t)lane < n_here) {
            const uint32_t m = p_mE & 0xFFFFu;
            const bool ok = m >= 1u && m <= P.max_len && (p_mE >> 16) <= P.max_E;
            if (!ok) atomicOr(P.err, 1u);
            L.off[(known + lane) & (kMeta - 1)] = ok ? p_off : 0ull;
            L.mE[(known + lane) & (kMeta - 1)] = ok ? p_mE | 0x80000000u : 1u;
        }
        known += 64;
    };

    auto flush = [&](uint32_t upto) {
        // Counts and accept bits of the tiles that end at or below `upto`
        // (and of the share's last, partial tile).
        wave_lds_sync();
        while (flushed < upto && (flushed + 64 <= upto || upto == n_here)) {
            const uint32_t i = flushed + (uint32_t)lane;
            const uint32_t v = i < n_here ? L.cnt[i & (kRing - 1)] : 0u;
            const uint64_t bal = __ballot((v & 0x8000u) != 0u);
            const uint64_t slot = slot_of(flushed);
            if (i < n_here) P.cnt[0][slot + lane] = (uint16_t)(v & 0x7FFFu);
            if (lane < 2 && flushed + 32u * lane < n_here)
                P.acc[0][slot / 32 + lane] = lane ? (uint32_t)(bal >> 32) : (uint32_t)bal;
            flushed += 64;
        }
        wave_lds_sync();
    };

    // The lane's pair: index in the share, offset, length, threshold; the
    // snake's column and edits, and the diagonals whose pipes ended before
    // the window when it is inside one.
    uint32_t idx = 0, m = GENERAL ? 1u : P.uniform_len, E = P.uniform_E;
    uint64_t off = 0;
    uint32_t c = 0, e = 0;
    bool busy = false, cont = false;
    DT dead = 0;

    if constexpr (GENERAL) fetch_meta();
    for (;;) {
        const uint64_t idle = __ballot(!busy);
        if (idle != 0ull) {
            if (issued >= n_here) {
                if (idle == ~0ull) break;
            } else {
                const uint32_t n_idle = (uint32_t)__builtin_popcountll(idle);
                if (issued - flushed + n_idle > kRing) flush(wave_min(busy ? idx : issued));
                const uint32_t take = min(min(n_idle, n_here - issued), kRing - min(kRing, issued - flushed));
                if constexpr (GENERAL) {
                    if (issued + take > known) {
                        keep_meta();
                        fetch_meta();
                        wave_lds_sync();
                    }
                }
                const uint32_t rank = rank_in(idle);
                if (!busy && rank < take) {
                    idx = issued + rank;
                    busy = true;
                    if constexpr (GENERAL) {
                        off = L.off[idx & (kMeta - 1)];
                        const uint32_t v = L.mE[idx & (kMeta - 1)];
                        m = v & 0xFFFFu;
                        E = (v >> 16) & 0xFFu;
                        if ((v & 0x80000000u) == 0u) {
                            L.cnt[idx & (kRing - 1)] = 0;
                            busy = false;
                        }
                    } else {
                        off = slot_of(idx) * P.stride_words;
                    }
                    e = 0;
                }
                issued += take;
            }
        }
        const uint32_t rem = m - c;
        FlowWords q = flow_load<!GENERAL>(P.reads + off, P.refs + off, c, (int)((m + 31u) >> 5));
        flow_vacancy(q, c, rem);
        uint32_t M[D];
        flow_map<EMAX, GENERAL>(q, E, dead, M);
        uint32_t b = busy ? 1u : 0u;
        const uint32_t obst = flow_probe<D>(M, P.probes, b);
        e += popc(obst & ~q.vc);
        cont = b == 0u && (int32_t)obst >= 0;
        // The last probe's start, for the diagonals of a pipe running on: its
        // run reaches bit 31 exactly when M + bs carries out of it.
        const uint32_t bs = 1u << ((obst ? 32u - (uint32_t)__builtin_clz(obst) : 0u) & 31u);
        c += b != 0u ? (uint32_t)__builtin_ctz(b) : 32u;
        if (busy && (c >= m || e > E)) {
            L.cnt[idx & (kRing - 1)] = (uint16_t)(e > E ? E + 1u : (e | 0x8000u));
            busy = false;
        }
        if (!busy) {
            c = 0;
            cont = false;
        }
        dead = 0;
        if (wave_any(cont)) {
            uint32_t lo = 0, hi = 0;
#pragma unroll
            for (int d = D - 1; d >= 0; --d) {
                uint32_t sum;
                const uint32_t cy = __builtin_add_overflow(M[d], bs, &sum) ? 1u : 0u;
                if (d >= 32) hi = hi + hi + cy;
                else lo = lo + lo + cy;
            }
            const DT alive = (DT)lo | (sizeof(DT) > 4 ? (DT)((uint64_t)hi << 32) : (DT)0);
            constexpr DT all = (D >= 8 * (int)sizeof(DT)) ? ~(DT)0 : (((DT)1 << D) - 1);
            dead = cont ? (DT)(~alive & all) : (DT)0;
        }
    }
    flush(n_here);
}

template <bool GENERAL, bool SAMPLED = false>
const void* flow_kernel_for(int emax) {
    switch (emax) {
#define PAF_CASE(X) \
    case X: return reinterpret_cast<const void*>(&flow_kernel<X, GENERAL, SAMPLED && (X < 20)>);
        PAF_CASE(0) PAF_CASE(1) PAF_CASE(2) PAF_CASE(3) PAF_CASE(4) PAF_CASE(5) PAF_CASE(6)
        PAF_CASE(7) PAF_CASE(8) PAF_CASE(10) PAF_CASE(12) PAF_CASE(15) PAF_CASE(20) PAF_CASE(25)
        PAF_CASE(31)
#undef PAF_CASE
        default: return nullptr;
    }
}

}  // namespace

// Rows of more words than this take a wave's share of the L1 with them: 64 lanes
// read two rows each, and four waves per SIMD evict one another's.
constexpr uint32_t kNarrowWords = 6;

// The largest batches that run here, from both engines' times (us, this one and
// the compacting one, 70% unrelated pairs and in brackets none).
//   Uniform: 16384 tiles, so that nothing is slower than the compacting engine in
// its own chunks: 1M pairs, 250 bp, E = 0 25 / 28 (51 / 82), E = 10 72 / 85 (137 /
// 151); 100 bp, E = 5 22 / 26 (38 / 39).  13312 where wide rows meet E = 4 to 6 (250
// bp, E = 5, 850k 31 / 36 (72 / 71), 1M 36 / 38 (93 / 76)) and where the threshold
// belongs to a lower class, whose general kernel is the slower one here (250 bp,
// E = 20 as 25, 1M 209 / 197).  (Chunks fitted to the batch as in api.hip take 68
// (105) at 1M and E = 10 and 39 (55) at 500k, less than this engine's 72 (137)
// and 43 (69), but 65 (103) at 700k, more than its 52 (91).)
//   Offsets or thresholds per pair, one length: to where lanes that are alike
// stop gaining.  250 bp: E = 3 4M 134 / 134, 8M 264 / 249; E = 5 500k 29 / 30, 1M 44 /
// 42; E = 10 2M 129 / 137, 4M 248 / 236; E = 25 4M 795 / 861; 150 bp, E = 7 8M 243 / 262.
//   Lengths per pair: mixes gain at every size (5M of the uneven mix, thresholds
// of 2% / 5% 155 / 191 and 330 / 375), lengths that are alike lose in large batches
// (all 250 bp, 10M at E = 10 588 / 526, 8M at E = 5 336 / 273), so above 32768
// tiles a launch of each engine asks 64 of the pairs which of them it is for:
// 4 us on 100 and more.
SnakeEngine snake_engine(const FilterParams& p, int emax) {
    const bool wide = p.wmax > kNarrowWords, per_pair = p.len || p.E || p.word_offset;
    uint32_t most;   // tiles
    if (!per_pair) most = (wide && emax >= 4 && emax <= 6) || (int)p.uniform_E <= emax_below(emax) ? 13312u : 16384u;
    else if (emax >= 20 || (!wide && (emax >= 7 || emax <= 3))) most = ~0u;
    else if (emax <= 3) most = 65536u;
    else if (emax <= 6 && wide && !p.len) most = 8192u;
    else most = 32768u;
    return p.n_tiles <= most ? SnakeEngine::Flow : p.len ? SnakeEngine::Sampled : SnakeEngine::Compacting;
}

hipError_t launch_flow(FilterParams p, int emax, int num_cus, hipStream_t stream) {
    // The uniform kernels mask only the diagonals between their threshold
    // class and the one below, and load two words at a time.
    const bool general = p.len || p.E || p.word_offset || words_for(p.uniform_len) < 2 ||
                         (int)p.uniform_E <= emax_below(emax);
    const void* k = p.pick == kPickMixed ? flow_kernel_for<true, true>(emax)
                    : general            ? flow_kernel_for<true>(emax)
                                         : flow_kernel_for<false>(emax);
    if (!k) return hipErrorInvalidValue;
    // Two waves per SIMD, and up to `most` once every wave keeps four tiles.
    // (250 bp, E = 5, 1M pairs: 36 us with two, 68 with four; 100 bp 48 and 38 when
    // all are related; 2M of the uneven mix with thresholds of 2% 67 with two or
    // three, 81 with four, of 5% 158, 148 and 147.)
    const uint64_t simds = (uint64_t)num_cus * 4;
    const bool per_pair = p.len || p.E || p.word_offset;
    uint64_t most = 4;
    if (!per_pair) most = p.wmax <= kNarrowWords && p.n_tiles >= 14 * simds ? 4 : 2;
    else if (p.wmax > kNarrowWords && emax <= 6) most = emax <= 3 ? 2 : 3;
    const uint64_t waves = std::max(2 * simds, std::min<uint64_t>(most * simds, p.n_tiles / 4));
    p.waves = (uint32_t)std::min<uint64_t>(waves, p.n_tiles);
    // The probes of a window: E + 1 obstacles in as few windows of at most
    // seven as hold them (a window of random bases holds seven to eight);
    // four where thresholds differ (uneven mix, 2M pairs: 147 us, 150 with six).
    const uint32_t windows = (uint32_t)(emax + 7) / 7;
    p.probes = general ? 4u : ((uint32_t)emax + windows) / windows;
    void* args[] = {&p};
    return hipLaunchKernel(k, dim3((p.waves + kFlowWaves - 1) / kFlowWaves), dim3(64 * kFlowWaves), args, 0, stream);
}

}  // namespace paf
