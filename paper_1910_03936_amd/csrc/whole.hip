// Whole-map decision stages for gfx950: GateKeeper (Ch. 5) and Shouji
// (Ch. 6), which read every window of the map, plus SneakySnake on the same
// map when asked for.  One lane per pair, 64 pairs per wave staged in LDS
// (word-major); windows are walked in step.
#include "paf_tile.h"

namespace paf {

namespace {

// ---------------------------------------------------------------------------
// Whole-map engine.  The raw mismatch words of the current and the next window
// are kept; vacant and past-end cells are folded in (blocked for SneakySnake
// and Shouji, free for GateKeeper) only in the windows that hold any.
//
// Bound by VALU issue, where adds, shifts right and logic (v_bitop3 on
// registers included) take about 2.4 cycles a wave and funnel shifts, shifts
// left, field extracts and compares about 4.3: the diagonals are worked on with
// as few of the latter as the definitions allow.  2M pairs of 250 bp at E = 10:
// GateKeeper 148 -> 104 us (opening once a window instead of amending every
// diagonal), Shouji 400 -> 264 us (eight ranks instead of a ones count, and the
// store by table look-up instead of ten instructions a column), the two
// together 543 -> 282 us (one set of raw words instead of a map each, which
// had left two waves per SIMD).

// Three-input logic in one v_bitop3 each (truth table bit s0 * 4 + s1 * 2 + s2).
__device__ __forceinline__ uint32_t sel3(uint32_t m, uint32_t x, uint32_t y) {   // m ? x : y
    return __builtin_amdgcn_bitop3_b32(m, x, y, 0xCA);
}
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}
// One step of a bit-sliced less-than from the low bit up, (~n & o) | (~(n ^ o) & t).
__device__ __forceinline__ uint32_t lt_step(uint32_t n, uint32_t o, uint32_t t) {
    return __builtin_amdgcn_bitop3_b32(n, o, t, 0x8E);
}
__device__ __forceinline__ uint32_t or_and(uint32_t a, uint32_t b, uint32_t c) {   // (a | b) & c
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xA8);
}

// Shouji's best 4-column segment at each of the window's 32 start columns,
// bit-sliced.  A segment of bits b0..b3 (b0: its first column) with r ones in
// b1..b3 is ranked by 2 (r + b0) + b0: fewer ones first, and on a tie a
// segment that starts with a zero.  That key takes eight values, so its rank
// k (k2 k1 k0) is three functions of b0 and r; b0 and r's low bit are
// functions of k again, and b3 is the parity that is left.
struct ShoujiBest {
    uint32_t k0, k1, k2, b1, b2;
};

__device__ __forceinline__ void shouji_candidate(ShoujiBest& bs, uint32_t cur, uint32_t nxt, bool first) {
    const uint32_t B1 = funnel(nxt, cur, 1);
    const uint32_t B2 = funnel(nxt, cur, 2);
    const uint32_t B3 = funnel(nxt, cur, 3);
    const uint32_t r0 = xor3(B1, B2, B3), r1 = maj3(B1, B2, B3);
    const uint32_t k2 = maj3(cur, r1, r0);
    const uint32_t k1 = __builtin_amdgcn_bitop3_b32(cur, r1, r0, 0xD4);
    const uint32_t k0 = __builtin_amdgcn_bitop3_b32(cur, r1, r0, 0x8E);
    if (first) {
        bs = {k0, k1, k2, B1, B2};
        return;
    }
    // Equal ranks keep the earlier diagonal.
    const uint32_t rep = lt_step(k2, bs.k2, lt_step(k1, bs.k1, ~k0 & bs.k0));
    bs.k0 = sel3(rep, k0, bs.k0);
    bs.k1 = sel3(rep, k1, bs.k1);
    bs.k2 = sel3(rep, k2, bs.k2);
    bs.b1 = sel3(rep, B1, bs.b1);
    bs.b2 = sel3(rep, B2, bs.b2);
}

// Shouji's sequential store (Sec. 6.2.2): the best segment V of column j
// overwrites the vector's bits j..j+3 when it holds strictly more zeros.  Bit
// j + 3 is still 1 then, so the vector's bits j..j+2 are the whole state s,
// and the column is an automaton: V is taken when popc(V) <= popc(s); the
// column's final bit is V's (s's) lowest, and the next state is V >> 1 (s >> 1
// with a 1 on top).  Two columns go through one table look-up: entry (V pair,
// s) holds the next state times two in its low bits and 256 times the ones
// the two columns add to the count.  A V pair is a byte with bit t (2 p + t)
// of column t's segment bit p.
struct alignas(16) ShoujiTable {
    uint16_t e[256 * 8];
};
constexpr ShoujiTable make_shouji_table() {
    ShoujiTable T{};
    for (uint32_t v = 0; v < 256; ++v)
        for (uint32_t s0 = 0; s0 < 8; ++s0) {
            uint32_t s = s0, ones = 0;
            for (uint32_t t = 0; t < 2; ++t) {
                uint32_t V = 0, nv = 0;
                for (uint32_t p = 0; p < 4; ++p) V |= ((v >> (2 * p + t)) & 1u) << p;
                for (uint32_t p = 0; p < 4; ++p) nv += (V >> p) & 1u;
                const uint32_t ns = (s & 1u) + ((s >> 1) & 1u) + (s >> 2);
                const bool take = nv <= ns;
                ones += take ? V & 1u : s & 1u;
                s = take ? V >> 1 : (s >> 1) | 4u;
            }
            T.e[v * 8 + s0] = (uint16_t)(2u * s | ones << 8);
        }
    return T;
}
__device__ const ShoujiTable kShoujiTable = make_shouji_table();

// V pairs of columns 8 q .. 8 q + 7 (a byte per two columns) from the planes.
__device__ __forceinline__ uint32_t shouji_pairs(int q, uint32_t b0, uint32_t b1, uint32_t b2, uint32_t b3) {
    auto spread = [q](uint32_t b) {
        uint32_t x = (b << (24 - 8 * q)) & 0xFF000000u;
        x = or_and(x, x >> 12, 0xF000F000u);
        return or_and(x, x >> 6, 0xC0C0C0C0u);
    };
    return or3(spread(b0) >> 6, spread(b1) >> 4, spread(b2) >> 2) | spread(b3);
}

// The window's 32 columns through the table: the ones they add, `state` (times
// two) carried on.
__device__ __forceinline__ uint32_t shouji_store(const uint16_t* table, const ShoujiBest& bs, uint32_t past, uint32_t& state) {
    const uint32_t b0 = __builtin_amdgcn_bitop3_b32(bs.k2, bs.k1, bs.k0, 0xD4) | past;
    const uint32_t r0 = __builtin_amdgcn_bitop3_b32(bs.k2, bs.k1, bs.k0, 0xB2);
    const uint32_t b3 = xor3(r0, bs.b1, bs.b2) | past;
    const uint32_t b1 = bs.b1 | past, b2 = bs.b2 | past;
    const char* tab = reinterpret_cast<const char*>(table);
    uint32_t total = 0, r = state;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t w = shouji_pairs(q, b0, b1, b2, b3);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const uint32_t v = (t == 0 ? w << 4 : w >> (8 * t - 4)) & 0xFF0u;
            r = *reinterpret_cast<const uint16_t*>(tab + (v | (r & 0xEu)));
            total += r;   // the states add up to less than 256
        }
    }
    state = r & 0xEu;
    return total >> 8;
}

// Diagonals beyond the pair's threshold are all ones (the ones that can lie
// beyond it, see over_E).
template <int EMAX, bool GENERAL>
__host__ __device__ constexpr bool may_exceed(int ad) {
    return GENERAL ? ad > 0 : ad > emax_below(EMAX) + 1;
}
__device__ __forceinline__ uint32_t over_E(uint32_t E, int ad) { return (uint32_t)((int32_t)(E - (uint32_t)ad) >> 31); }

// Vacant and past-end cells of a window (none on the diagonals beyond the
// threshold, whose words are ones for every stage).
struct Vacancy {
    uint32_t vp, vc, vn;
};
__device__ __forceinline__ Vacancy vacancy_of(int k, int m) {
    return Vacancy{vacant_word(k - 1, m), vacant_word(k, m), vacant_word(k + 1, m)};
}
template <int d, bool MASK>
__device__ __forceinline__ uint32_t diag_blank(const Vacancy& v, uint32_t E) {
    uint32_t x = v.vc;
    if constexpr (d > 0) x |= funnel(v.vn, v.vc, d);
    if constexpr (d < 0) x |= funnel(v.vc, v.vp, 32 + d);
    if constexpr (MASK) x &= ~over_E(E, d < 0 ? -d : d);
    return x;
}

// A window's words as they are kept: raw where two stages share them, else
// with the vacant and past-end cells folded in for the stage that reads them
// (kFree: GateKeeper, kBlocked: Shouji), so that no window's are worked out
// twice: 2M uneven pairs 180 -> 140 us for GateKeeper, 364 -> 321 for Shouji.
// (blank_words is a pass of its own over the windows that have such cells: as
// two branches of one pass the words of both were live.)
constexpr int kRaw = 0, kFree = 1, kBlocked = 2;
template <int EMAX, bool GENERAL, bool BLOCK, int I = 0>
__device__ __forceinline__ void build_raw(const WindowWords& q, uint32_t E, uint32_t* R) {
    if constexpr (I < 2 * EMAX + 1) {
        constexpr int d = I - EMAX, ad = d < 0 ? -d : d;
        R[I] = diag_raw<d>(q);
        if constexpr (BLOCK && may_exceed<EMAX, GENERAL>(ad)) R[I] |= over_E(E, ad);
        build_raw<EMAX, GENERAL, BLOCK, I + 1>(q, E, R);
    }
}
template <int EMAX, int KEEP, int I = 0>
__device__ __forceinline__ void blank_words(const Vacancy& v, uint32_t* R) {
    if constexpr (I < 2 * EMAX + 1) {
        const uint32_t x = diag_blank<I - EMAX, false>(v, 0u);
        R[I] = KEEP == kFree ? R[I] & ~x : R[I] | x;
        blank_words<EMAX, KEEP, I + 1>(v, R);
    }
}
template <int EMAX, bool GENERAL, int I = 0>
__device__ __forceinline__ void block_over_E(uint32_t E, uint32_t* R) {
    if constexpr (I < 2 * EMAX + 1) {
        constexpr int d = I - EMAX, ad = d < 0 ? -d : d;
        if constexpr (may_exceed<EMAX, GENERAL>(ad)) R[I] |= over_E(E, ad);
        block_over_E<EMAX, GENERAL, I + 1>(E, R);
    }
}
template <int EMAX, bool GENERAL, int KEEP>
__device__ __forceinline__ void build_words(const WindowWords& q, const Vacancy& v, bool blanks, uint32_t E, uint32_t* R) {
    build_raw<EMAX, GENERAL, KEEP == kRaw>(q, E, R);
    if constexpr (KEEP == kRaw) return;
    if (blanks) blank_words<EMAX, KEEP>(v, R);
    // Many diagonals' masks are worked out again each window, not held (they
    // would take the registers of a wave per SIMD).
    if constexpr (GENERAL && EMAX > 15) asm volatile("" : "+v"(E));
    block_over_E<EMAX, GENERAL>(E, R);
}

// GateKeeper (Ch. 5, Sec. 5.2.2): the amendment turns streaks of one or two
// zeros into ones, which leaves the zeros that lie in a run of three or more
// (beyond the map's ends all cells count as zero).  The masks are AND-ed, so a
// result bit is zero when some diagonal keeps a zero there; since taking the
// cells that a run covers commutes with that, each diagonal only gives the
// starts of its runs of three, not (g | g1 | g2), and the runs grow back to
// their cells once a window, over all diagonals together: four instructions a
// diagonal instead of seven.  Shouji's candidates share the same words.
template <int EMAX, bool GENERAL, bool INNER, bool GKS, bool SHS, int I = 0>
__device__ __forceinline__ void whole_diagonals(const uint32_t* Rc, const uint32_t* Rn, const Vacancy& vc, const Vacancy& vn,
                                                uint32_t E, uint32_t& starts, ShoujiBest& bs) {
    if constexpr (I < 2 * EMAX + 1) {
        constexpr int d = I - EMAX, ad = d < 0 ? -d : d;
        constexpr bool MASK = may_exceed<EMAX, GENERAL>(ad);
        const uint32_t c = Rc[I], n = Rn[I];
        uint32_t bc = 0, bn = 0;
        if constexpr (!INNER) {
            bc = diag_blank<d, MASK>(vc, E);
            bn = diag_blank<d, MASK>(vn, E);
        }
        if constexpr (GKS) {
            const uint32_t gc = c & ~bc, gn = n & ~bn;
            starts &= or3(gc, funnel(gn, gc, 1), funnel(gn, gc, 2));
        }
        if constexpr (SHS && EMAX > 0) shouji_candidate(bs, c | bc, n | bn, I == 0);
        whole_diagonals<EMAX, GENERAL, INNER, GKS, SHS, I + 1>(Rc, Rn, vc, vn, E, starts, bs);
    }
}

// SneakySnake's map of a window: vacant and past-end cells blocked.
template <int EMAX, bool GENERAL, int I = 0>
__device__ __forceinline__ void blocked_words(const uint32_t* R, const Vacancy& v, uint32_t E, uint32_t* M) {
    if constexpr (I < 2 * EMAX + 1) {
        constexpr int d = I - EMAX, ad = d < 0 ? -d : d;
        M[I] = R[I] | diag_blank<d, may_exceed<EMAX, GENERAL>(ad)>(v, E);
        blocked_words<EMAX, GENERAL, I + 1>(R, v, E, M);
    }
}

// The starts of runs of three zeros in the two columns before the first: their
// runs reach column 0 (all of it free on some diagonal, or columns 0 and 1).
template <int EMAX, bool GENERAL, int KEEP, int I = 0>
__device__ __forceinline__ void left_starts(const uint32_t* R, const Vacancy& v, uint32_t E, uint32_t& one, uint32_t& two) {
    if constexpr (I < 2 * EMAX + 1) {
        constexpr int d = I - EMAX, ad = d < 0 ? -d : d;
        uint32_t g = R[I];
        if constexpr (KEEP == kRaw) g &= ~diag_blank<d, may_exceed<EMAX, GENERAL>(ad)>(v, E);
        one &= g;
        two &= g | (g >> 1);
        left_starts<EMAX, GENERAL, KEEP, I + 1>(R, v, E, one, two);
    }
}

// FS: the decision stages this instantiation runs (bits of PAF_*), or 0 for
// any mask given at run time.
template <int EMAX, bool GENERAL, int FS>
__device__ void whole_tile(const FilterParams& P, uint64_t tile, int lane, uint64_t* rdL, uint64_t* rfL,
                           const uint16_t* table) {
    constexpr int D = 2 * EMAX + 1;
    using DT = typename DeadMask<EMAX>::T;
    uint64_t off;
    const PairSlot ps = load_slot<GENERAL>(P, tile, lane, off);
    stage_tile<GENERAL>(P, tile, lane, ps, off, rdL, rfL);

    constexpr bool RT = FS == 0;
    // (Shouji's blocked words pay where some lane's pair ends in most windows, and
    // where registers are short: 2M uniform pairs at E = 10 264 us raw, 273
    // blocked; 500k at E = 25 149 and 133.)
    constexpr int KEEP = FS == PAF_GATEKEEPER ? kFree
                         : FS == PAF_SHOUJI && (GENERAL || EMAX > 15) ? kBlocked : kRaw;
    constexpr bool GKS = RT || (FS & PAF_GATEKEEPER), SHS = RT || (FS & PAF_SHOUJI), SSS = RT || (FS & PAF_SNEAKYSNAKE);
    const bool doSS = RT ? (P.filters & PAF_SNEAKYSNAKE) != 0 : SSS;
    const bool doGK = RT ? (P.filters & PAF_GATEKEEPER) != 0 : GKS;
    const bool doSH = RT ? (P.filters & PAF_SHOUJI) != 0 : SHS;
    const uint32_t m = ps.m, E = ps.E;

    Snake z{0u, 0u, ps.valid && doSS, false, 0u};
    bool cont = false;
    DT dead = 0;
    uint32_t gk_ham = 0, gk_cnt = 0, prev_starts = 0;
    uint32_t sh_cnt = 0, sh_state = 7u << 1;

    uint32_t Ra[D], Rb[D];
    {
        const WindowWords q = window_words(rdL, rfL, lane, 0, P.wmax, (int)m);
        build_words<EMAX, GENERAL, KEEP>(q, vacancy_of(0, (int)m), true, E, Ra);
        if (GKS && doGK) {
            uint32_t one = ~0u, two = ~0u;
            left_starts<EMAX, GENERAL, KEEP>(Ra, vacancy_of(0, (int)m), E, one, two);
            prev_starts = (~one & 1u) << 30 | (~two & 1u) << 31;
        }
    }
    // One window: its words in Rc, the next one's built into Rn.  Lanes past
    // their pair's last window run along (their words are staged as zeros) and
    // their results are not counted.
    auto window = [&](uint32_t w, const uint32_t (&Rc)[D], uint32_t (&Rn)[D]) {
        const bool have = ps.valid && w < ps.W;
        const WindowWords qn = window_words(rdL, rfL, lane, (int)w + 1, P.wmax, (int)m);
        if constexpr (KEEP == kRaw) build_raw<EMAX, GENERAL, true>(qn, E, Rn);
        const uint32_t past = have ? vacant_word((int)w, (int)m) : ~0u;   // columns >= m
        const Vacancy vc = vacancy_of((int)w, (int)m), vn = vacancy_of((int)w + 1, (int)m);
        // Cells of this window or the next one are vacant only near the ends.
        const bool inner_n = !wave_any(have && ((KEEP == kRaw && w == 0u) || 32u * (w + 2u) + (uint32_t)EMAX > m));
        const bool inner = KEEP != kRaw || inner_n;
        if constexpr (KEEP != kRaw) build_words<EMAX, GENERAL, KEEP>(qn, vn, !inner_n, E, Rn);
        if constexpr (SSS)
            if (doSS && have && z.act) {
                uint32_t M[D];
                blocked_words<EMAX, GENERAL>(Rc, vc, E, M);
                snake_window<EMAX, DT>(z, M, w, m, E, cont, dead);
            }
        uint32_t starts = ~0u;
        ShoujiBest bs;
        auto diagonals = [&](auto gk, auto sh) {
            constexpr bool G = decltype(gk)::value, S = decltype(sh)::value;
            if (inner) whole_diagonals<EMAX, GENERAL, true, G, S>(Rc, Rn, vc, vn, E, starts, bs);
            else if constexpr (KEEP == kRaw) whole_diagonals<EMAX, GENERAL, false, G, S>(Rc, Rn, vc, vn, E, starts, bs);
        };
        using yes = std::true_type;
        using no = std::false_type;
        if constexpr (!RT) {
            diagonals(std::integral_constant<bool, GKS>{}, std::integral_constant<bool, SHS>{});
        } else {
            if (doGK && doSH) diagonals(yes{}, yes{});
            else if (doGK) diagonals(yes{}, no{});
            else if (doSH) diagonals(no{}, yes{});
        }
        // The main diagonal's mismatches (never vacant inside the pair).
        const uint32_t ham = popc(Rc[EMAX] & ~past);
        if (GKS && doGK) {
            gk_ham += ham;   // GateKeeper's fast path
            const uint32_t runs = ~starts;
            const uint32_t kept = or3(runs, funnel(runs, prev_starts, 31), funnel(runs, prev_starts, 30));
            gk_cnt += popc(~(kept | past));
            prev_starts = runs;
        }
        if (SHS && doSH) {
            if constexpr (EMAX == 0) {
                // One diagonal (E = 0): the window starting at column j
                // replaces the vector's bits j..j+3, which hold the diagonal's
                // bits j..j+2 and a still unset 1 at j+3, exactly when bit j+3
                // of the diagonal is 0; the first window leaves the vector's
                // first four bits equal to the diagonal's either way.  So the
                // vector ends equal to the diagonal, and the count is its
                // Hamming distance.
                sh_cnt += ham;
            } else {
                // Start columns at or past the pair's end get segment 1111,
                // which never replaces anything.  The vector stays 1 in the
                // columns past the end, which are not counted.
                const uint32_t ones = shouji_store(table, bs, past, sh_state);
                sh_cnt += have ? ones - popc(past) : 0u;
            }
        }
    };
    // (two windows a turn, so that no window's words are copied on)
    for (uint32_t w = 0;; w += 2) {
        if (!wave_any(ps.valid && w < ps.W)) break;
        if constexpr (RT) {
            // (as a function it takes the words through scratch)
            [[clang::always_inline]] window(w, Ra, Rb);
            if (!wave_any(ps.valid && w + 1 < ps.W)) break;
            [[clang::always_inline]] window(w + 1, Rb, Ra);
        } else {
            window(w, Ra, Rb);
            if (!wave_any(ps.valid && w + 1 < ps.W)) break;
            window(w + 1, Rb, Ra);
        }
    }

    const bool gk_acc = gk_ham <= E || gk_cnt <= E;
    const uint32_t gk_out = gk_ham <= E ? gk_ham : gk_cnt;
    const bool sh_acc = sh_cnt <= E;
    bool accs[3] = {z.acc, gk_acc, sh_acc};
    uint32_t cnts[3] = {z.cnt, gk_out, sh_cnt};
#pragma unroll
    for (int f = 0; f < 3; ++f) {
        if (!(P.filters & (1u << f))) continue;
        if (GENERAL && P.perm) {
            if (ps.in_batch) P.cnt[f][ps.id] = (uint16_t)(ps.valid ? cnts[f] : 0u);
        } else {
            const uint64_t bal = __ballot(ps.valid && accs[f]);
            if (ps.in_batch) P.cnt[f][ps.slot] = (uint16_t)(ps.valid ? cnts[f] : 0u);
            if (lane == 0) {
                P.acc[f][2 * tile] = (uint32_t)bal;
                if (tile * 64 + 32 < P.n_pairs) P.acc[f][2 * tile + 1] = (uint32_t)(bal >> 32);
            }
        }
    }
}

template <int EMAX, bool GENERAL, int FS>
__global__ void __launch_bounds__(256) whole_kernel(FilterParams P) {
    extern __shared__ uint64_t lds[];
    constexpr bool TABLE = EMAX > 0 && (FS == 0 || (FS & PAF_SHOUJI) != 0);
    __shared__ typename std::conditional<TABLE, ShoujiTable, uint4>::type table;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if (TABLE && (FS != 0 || (P.filters & PAF_SHOUJI) != 0)) {
        for (uint32_t i = threadIdx.x; i < sizeof(ShoujiTable) / 16; i += blockDim.x)
            reinterpret_cast<uint4*>(&table)[i] = reinterpret_cast<const uint4*>(&kShoujiTable)[i];
        __syncthreads();
    }
    uint64_t* rdL = lds + (size_t)wave * 2 * P.wmax * kLdsRow;
    uint64_t* rfL = rdL + (size_t)P.wmax * kLdsRow;
    const uint16_t* tab = reinterpret_cast<const uint16_t*>(&table);
    // The masks read at run time in one place where pairs have lengths and
    // thresholds of their own: 100k at E = 15, SneakySnake and Shouji, 216 us in
    // two, 185 in one; 1M of 400 bp at E = 31, all three, 4945 and 2146.  (The
    // others are the faster form inlined twice: GateKeeper and Shouji on 1M pairs
    // at E = 10 149 us, 158 in one place.)
    for_each_tile<FS == 0 && GENERAL>(P, lane, wave,
                                      [&](uint64_t tile) { whole_tile<EMAX, GENERAL, FS>(P, tile, lane, rdL, rfL, tab); });
}

template <bool GENERAL, int FS>
const void* whole_for(int emax) {
    switch (emax) {
#define PAF_CASE(X) \
    case X: return reinterpret_cast<const void*>(&whole_kernel<X, GENERAL, FS>);
        PAF_CASE(0) PAF_CASE(1) PAF_CASE(2) PAF_CASE(3) PAF_CASE(4) PAF_CASE(5) PAF_CASE(6)
        PAF_CASE(7) PAF_CASE(8) PAF_CASE(10) PAF_CASE(12) PAF_CASE(15) PAF_CASE(20) PAF_CASE(25)
        PAF_CASE(31)
#undef PAF_CASE
        default: return nullptr;
    }
}

}  // namespace

// GateKeeper, Shouji, the two together and SneakySnake with GateKeeper get
// kernels of their own (the last: 1M pairs at E = 5 in a given order 133 us on the
// kernel below, 122 on its own); SneakySnake with Shouji and all three run on
// the kernel that reads the mask at run time.
const void* whole_kernel_ptr(bool general, int emax, uint32_t filters) {
    switch (filters) {
        case PAF_GATEKEEPER: return general ? whole_for<true, PAF_GATEKEEPER>(emax) : whole_for<false, PAF_GATEKEEPER>(emax);
        case PAF_SHOUJI: return general ? whole_for<true, PAF_SHOUJI>(emax) : whole_for<false, PAF_SHOUJI>(emax);
        case PAF_GATEKEEPER | PAF_SHOUJI:
            return general ? whole_for<true, PAF_GATEKEEPER | PAF_SHOUJI>(emax)
                           : whole_for<false, PAF_GATEKEEPER | PAF_SHOUJI>(emax);
        case PAF_SNEAKYSNAKE | PAF_GATEKEEPER:
            return general ? whole_for<true, PAF_SNEAKYSNAKE | PAF_GATEKEEPER>(emax)
                           : whole_for<false, PAF_SNEAKYSNAKE | PAF_GATEKEEPER>(emax);
        default: return general ? whole_for<true, 0>(emax) : whole_for<false, 0>(emax);
    }
}

}  // namespace paf
