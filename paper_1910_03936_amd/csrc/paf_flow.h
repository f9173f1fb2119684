// Device code shared by the engines whose lanes each work on a window at a
// column of their own (flow.hip, magnet.hip): the words of a window that starts
// at any column, its vacant cells, and the match words of all diagonals.
#pragma once

#include "paf_tile.h"

namespace paf {
namespace {

// The 32 columns from a lane's column c: read planes of positions c - 32 ..
// c + 63 (p, c, n), reference planes of columns c .. c + 31, and the vacant
// read positions (set by flow_vacancy).
struct FlowWords {
    uint32_t plo, phi, clo, chi, nlo, nhi, flo, fhi;
    uint32_t vp, vc, vn;
};

__device__ __forceinline__ uint32_t lo32(uint64_t x) { return (uint32_t)x; }
__device__ __forceinline__ uint32_t hi32(uint64_t x) { return (uint32_t)(x >> 32); }

// From the words around c: read words k - 1 .. k + 2 and reference words k,
// k + 1, k = c / 32.
__device__ __forceinline__ FlowWords flow_words(uint64_t wp, uint64_t wc, uint64_t wn, uint64_t wn2, uint64_t f0,
                                                uint64_t f1, uint32_t c) {
    FlowWords q;
    q.plo = funnel(lo32(wc), lo32(wp), c);
    q.phi = funnel(hi32(wc), hi32(wp), c);
    q.clo = funnel(lo32(wn), lo32(wc), c);
    q.chi = funnel(hi32(wn), hi32(wc), c);
    q.nlo = funnel(lo32(wn2), lo32(wn), c);
    q.nhi = funnel(hi32(wn2), hi32(wn), c);
    q.flo = funnel(lo32(f1), lo32(f0), c);
    q.fhi = funnel(hi32(f1), hi32(f0), c);
    return q;
}

typedef uint64_t u64x2 __attribute__((ext_vector_type(2), aligned(8)));

// The same with the words loaded.  A word outside the pair is replaced by one
// inside it: every cell it would feed is vacant or past the pair's end.
// WIDE: 16-byte loads (W >= 2).
template <bool WIDE>
__device__ __forceinline__ FlowWords flow_load(const uint64_t* rd, const uint64_t* rf, uint32_t c, int W) {
    const int k = (int)(c >> 5);
    uint64_t wp, wc, wn, wn2, f0, f1;
    if constexpr (WIDE) {
        const u64x2 x = *reinterpret_cast<const u64x2*>(rd + max(k - 1, 0));
        const u64x2 y = *reinterpret_cast<const u64x2*>(rd + min(k + 1, W - 2));
        const u64x2 f = *reinterpret_cast<const u64x2*>(rf + min(k, W - 2));
        wp = x[0];
        wc = k == 0 ? x[0] : x[1];
        wn = k + 1 > W - 2 ? y[1] : y[0];
        wn2 = y[1];
        f0 = k > W - 2 ? f[1] : f[0];
        f1 = f[1];
    } else {
        wp = rd[max(k - 1, 0)];
        wc = rd[k];
        wn = rd[min(k + 1, W - 1)];
        wn2 = rd[min(k + 2, W - 1)];
        f0 = rf[k];
        f1 = rf[min(k + 1, W - 1)];
    }
    return flow_words(wp, wc, wn, wn2, f0, f1, c);
}

__device__ __forceinline__ void flow_vacancy(FlowWords& q, uint32_t c, uint32_t rem) {
    q.vp = c >= 32u ? 0u : ~0u >> c;
    const uint64_t v = ~0ull << min(rem, 63u);
    q.vc = (uint32_t)v;
    q.vn = (uint32_t)(v >> 32);
}

// Match words of all diagonals (bit j of M[i]: column c + j of diagonal
// i - EMAX is free).  Vacant cells are blocked, and so are the diagonals
// beyond the lane's own threshold (MASK: the ones that can lie beyond it); a
// lane inside a pipe sees the diagonals whose pipes ended before the window
// blocked in its first column.
template <int EMAX, bool GENERAL, typename DT, int I = 0>
__device__ __forceinline__ void flow_map(const FlowWords& q, uint32_t E, DT dead, uint32_t* M) {
    if constexpr (I < 2 * EMAX + 1) {
        constexpr int d = I - EMAX;
        constexpr int ad = d < 0 ? -d : d;
        constexpr bool MASK = GENERAL ? ad > 0 : ad > emax_below(EMAX) + 1;
        uint32_t lo, hi;
        if constexpr (d > 0) {
            lo = funnel(q.nlo, q.clo, d);
            hi = funnel(q.nhi, q.chi, d);
        } else if constexpr (d == 0) {
            lo = q.clo;
            hi = q.chi;
        } else {
            lo = funnel(q.clo, q.plo, 32 + d);
            hi = funnel(q.chi, q.phi, 32 + d);
        }
        uint32_t v = 0, x = 0;
        if constexpr (d < 0) v = q.vp >> (32 - ad);
        if constexpr (d > 0) v = funnel(q.vn, q.vc, d);
        if constexpr (MASK) x = (uint32_t)((int32_t)(E - (uint32_t)ad) >> 31);
        const uint32_t y = (uint32_t)(dead >> I) & 1u;
        M[I] = nor_xor(hi, or_xor(lo, or3(v, x, y), q.flo), q.fhi);
        flow_map<EMAX, GENERAL, DT, I + 1>(q, E, dead, M);
    }
}

__device__ __forceinline__ uint32_t rank_in(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Words of a bit array for a wave's pairs slot0 .. slot0 + n - 1 (n <= 2048),
// two per tile of 64: lane j loads word j, and the bits of a tile are read from
// its lanes (a load per tile, each waited for, took 1 us apiece).
__device__ __forceinline__ uint32_t chunk_bits(const uint32_t* bits, uint64_t slot0, uint32_t n, int lane) {
    return 32u * (uint32_t)lane < n ? bits[(slot0 >> 5) + (uint32_t)lane] : 0u;
}
__device__ __forceinline__ bool chunk_bit(uint32_t words, uint32_t tile, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)words, (int)(2u * tile));
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)words, (int)(2u * tile + 1u));
    return (((lane < 32 ? lo : hi) >> (lane & 31)) & 1u) != 0u;
}

}  // namespace
}  // namespace paf
