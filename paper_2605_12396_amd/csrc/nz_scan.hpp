// nz_scan.hpp -- wave-wide decoupled look-back and canonical-code ranking, shared by the gfx950 kernels.
#pragma once
#include <type_traits>
#include "nz_common.hpp"

namespace nz {

constexpr uint64_t kDescA    = 1ull << 62;          // descriptor holds this item's own amount
constexpr uint64_t kDescP    = 2ull << 62;          // descriptor holds the inclusive prefix up to this item
constexpr uint64_t kDescMask = (1ull << 62) - 1;

// Decoupled look-back, executed by one full wave.  Items lo..idx-1 precede item idx; a virtual item lo-1
// carries the inclusive prefix base0.  Every item publishes kDescA|own as soon as it knows its amount and
// kDescP|inclusive once it knows its prefix; a waiter only ever waits on items that were started before
// it (dynamic tickets), so every wait ends.  Returns the exclusive prefix of item idx.
__device__ inline uint64_t lookback_exclusive(const uint64_t* desc, int64_t lo, int64_t idx, uint64_t base0) {
    const int lane = (int)lane_id();
    uint64_t acc = 0;
    int64_t pos = idx - 1;
    for (;;) {
        const int64_t j = pos - lane;
        uint64_t v;
        int pl;
        for (;;) {
            v = (j >= lo) ? ld_agent(desc + j) : (kDescP | base0);
            const uint64_t pm = __ballot((v >> 62) == 2);
            const uint64_t zm = __ballot((v >> 62) == 0);
            pl = pm ? (__ffsll((unsigned long long)pm) - 1) : 64;
            const uint64_t need = (pl >= 64) ? ~0ull : ((2ull << pl) - 1ull);
            if ((zm & need) == 0) break;
            __builtin_amdgcn_s_sleep(2);
        }
        // (own amounts have 32 bits, and 64 of them together: a frame is at most some 8 MB; the prefix that ends the look-back has more)
        const uint32_t own = wave_incl_scan_dpp(lane < pl ? (uint32_t)v : 0u);
        acc += (uint32_t)__builtin_amdgcn_readlane((int)own, 63);
        if (pl < 64) { acc += wave_read64(v, pl) & kDescMask; break; }
        pos -= 64;
    }
    return acc;
}

// Canonical-code bookkeeping for an alphabet of K <= 1024 symbols whose code lengths sit in s_len[0..K)
// (0 = unused).  NT threads (multiple of 64) cooperate; thread t has the symbols t, t + NT, ... below K.  On return (after
// the trailing barrier):
//   s_cnt[L]   number of symbols with length L (s_cnt[0] = 0), L = 0..31
//   s_first[L] first canonical code of length L:  first[L] = (first[L-1] + cnt[L-1]) << 1
//   s_idx0[L]  number of symbols with a shorter length (index of the first length-L symbol in (len,sym) order)
//   rank[i]    position of the thread's i-th symbol among the symbols of its own length, in increasing symbol order
// so code(s) = s_first[len] + rank and sorted position = s_idx0[len] + rank.
// Scratch: s_wcnt[16*32].
// What bounds it is latency, and a decoder builds a frame's tables in front of its first symbol.  The lanes of a wavefront that
// have the same length find each other with one ballot per bit of a length (5; one ballot per possible length took 2.2 us of a decoder's
// start and 1.9 us of the codebook kernel, this one a third of that), and the ranks stay in registers.
template <int NT>
__device__ __forceinline__ void canonical_tables(const uint8_t* s_len, uint32_t K, uint32_t* s_wcnt, uint32_t* s_cnt,
                                        uint32_t* s_first, uint32_t* s_idx0, uint32_t (&rank)[kMaxK / NT]) {
    const uint32_t tid = threadIdx.x, lane = lane_id();
    static_assert(kMaxLen < 32, "five bits of a length");
#pragma unroll
    for (uint32_t i = 0; i < kMaxK / NT; i++) {
        const uint32_t s = i * NT + tid, grp = s >> 6;                 // (a group of 64 symbols is one wavefront's)
        rank[i] = 0;
        if (grp * 64u >= K) continue;                                  // (uniform over the wavefront)
        const uint32_t L = (s < K) ? s_len[s] : 0u;
        uint32_t lo = 0xFFFFFFFFu, hi = 0xFFFFFFFFu;                   // lanes with my length
#pragma unroll
        for (uint32_t b = 0; b < 5; b++) {
            const uint64_t set = __ballot((L >> b) & 1u);
            const uint32_t flip = ((L >> b) & 1u) - 1u;                // all ones where my bit is clear
            lo &= (uint32_t)set ^ flip; hi &= (uint32_t)(set >> 32) ^ flip;
        }
        rank[i] = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
        if (lane < 32) s_wcnt[grp * 32 + lane] = 0;
        if (L && rank[i] == 0) s_wcnt[grp * 32 + L] = (uint32_t)(__builtin_popcount(lo) + __builtin_popcount(hi));
    }
    __syncthreads();
    // per length (lane = length, wave 0): exclusive prefix over the groups and the total count, then
    // idx0 = exclusive scan of the counts and first[L] = sum over l < L of cnt[l] << (L - l), taken as an
    // exclusive scan of the counts left-justified to 28 bits (the Kraft sum is at most 1, so it fits).
    if (tid < 64) {
        uint32_t run = 0;
        if (tid >= 1 && tid <= kMaxLen) {
            auto prefix = [&](auto groups) {
                constexpr uint32_t G = decltype(groups)::value;
                uint32_t c[G];
#pragma unroll
                for (uint32_t g = 0; g < G; g++) c[g] = (g * 64u < K) ? s_wcnt[g * 32 + tid] : 0u;
#pragma unroll
                for (uint32_t g = 0; g < G; g++) { s_wcnt[g * 32 + tid] = run; run += c[g]; }
            };
            if (K <= 256u) prefix(std::integral_constant<uint32_t, 4>{}); else prefix(std::integral_constant<uint32_t, 16>{});
        }
        const uint32_t lj = (tid >= 1 && tid <= kMaxLen) ? (run << (kMaxLen - tid)) : 0u;
        const uint32_t incl_i = wave_incl_scan_dpp(run);
        const uint32_t incl_f = wave_incl_scan_dpp(lj);
        if (tid < 32) {
            s_cnt[tid] = run;
            s_idx0[tid] = incl_i - run;
            s_first[tid] = (tid <= kMaxLen) ? ((incl_f - lj) >> (kMaxLen - tid)) : (incl_f << (tid - kMaxLen));
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kMaxK / NT; i++) {
        const uint32_t s = i * NT + tid;
        if (s < K) { const uint32_t L = s_len[s]; if (L) rank[i] += s_wcnt[(s >> 6) * 32 + L]; }
    }
}

}  // namespace nz
