// nz_width.hpp -- threads per workgroup of the adding passes: a rule on the message and its frames (plain C++, no device code).
#pragma once
#include <stdint.h>

namespace nz {

// Adding passes: 512 threads (two statistics halves, two workgroups per compute unit, four wavefronts per SIMD), or 256 (one
// half, three workgroups per compute unit).  256 threads spread a message over more compute units, and half as many
// wavefronts share a unit's shared memory for their counting, but they build a frame's decode tables with half the
// threads, and have half as many for a block that takes more of a workgroup than its wavefronts: a FIXEDLEN one, and element by
// element a RAW or FIXEDLEN one that starts off a multiple of four.  What a thread is left with there counts as much as the spread.
constexpr uint32_t kAddThreads = 512, kAddThreadsSmall = 256;
constexpr uint32_t kAddResident = 2, kAddResidentSmall = 3;          // workgroups of a compute unit, by their shared memory
constexpr uint32_t kComputeUnits = 256, kSpreadFrom = 8;

// Elements of a block which a frame of nf fills in part, or which is taken one by one, that a thread of a workgroup of `threads` is left with
// (aligned: the frame starts at a multiple of four).
inline uint32_t add_pass_rest(uint32_t nf, bool aligned, uint32_t threads) {
    const uint32_t block = threads * 256u;
    const uint32_t rest = aligned ? nf % block : (nf < block ? nf : block);
    return (rest + threads - 1u) / threads;
}

// Us per call, 512 / 256 threads, of nz_reduce_local (HUFFMAN, 4.9 bits a symbol; FIXEDLEN, 14):
//   a frame is one workgroup either way -- frames of 16384, 16 MB 94 / 95; 41 / 49; of 49152, 16 MB 104 / 104; 58 / 82.  256 threads where 512
//     need more rounds of workgroups on the chip, up to kComputeUnits blocks of 512: of 16384, 136 MB 456 / 368; 187 / 190; of 49152 226 /
//     184; 168 / 162; of 32768 310 / 266; 185 / 202.  Frames of exactly 65536 take 256: that was for the HUFFMAN ones, which are
//     the same by now, and FIXEDLEN loses: 4 MB 96 / 96; 52 / 77; 64 MB 128 / 128; 91 / 126, sum of two streams 163 / 163;
//   a frame's second workgroup has less than half a block -- frames of 65537, 16 MB 172 / 175; 97 / 152; 136 MB 419 / 448; 378 / 566
//     (of 98304 113 / 107; 88 / 100);
//   other frames: 4 MB 103 / 97; 83 / 78; 48 MB 126 / 120; 128 / 119; 64 MB 132 / 127; 131 / 123.  Below kSpreadFrom
//     blocks the line is a cautious one: 64 KB 78 / 78; 27 / 33, but 1.2 MB 109 / 108; 83 / 76, 3 MB 102 / 97; 90 / 83, 2 MB 102 / 94; 86 / 76.
//     Past one 256-thread workgroup per compute unit a ragged end decides (a difference of up to 32 elements a thread does not show): 72 MB
//     with one of 43136 155 / 165; 147 / 145; frames of 100003, 64 MB 216 / 212; 173 / 203.  HUFFMAN would rather have 512 there, whatever
//     the end: 80 MB, which takes 256, 146 / 160; 149 / 146.
// From 256 blocks of 512 threads on the chip is full: 256 MB 229 / 256; 223 / 306 (at 128 MB 149 / 150; 157 / 156).
inline uint32_t add_pass_threads(uint64_t n, uint32_t chunk) {
    const uint64_t big = kAddThreads * 256u, small = kAddThreadsSmall * 256u, blocks = (n + big - 1) / big;
    if (blocks < kSpreadFrom || blocks >= kComputeUnits) return kAddThreads;
    const uint64_t frames = (n + chunk - 1) / chunk;
    const uint32_t last = (uint32_t)(n - (frames - 1) * chunk);
    if (chunk <= small) {                                                // one workgroup per frame
        if (chunk == small) return kAddThreadsSmall;
        const uint64_t rounds_big = (frames + kAddResident * kComputeUnits - 1) / (kAddResident * kComputeUnits);
        const uint64_t rounds_small = (frames + kAddResidentSmall * kComputeUnits - 1) / (kAddResidentSmall * kComputeUnits);
        return rounds_small < rounds_big ? kAddThreadsSmall : kAddThreads;
    }
    if (chunk < small + small / 2) return kAddThreads;
    const uint64_t grid_small = (frames - 1) * ((chunk + small - 1) / small) + (last + small - 1) / small;
    if (grid_small <= kComputeUnits) return kAddThreadsSmall;
    uint32_t rest[2];
    for (uint32_t i = 0; i < 2; i++) {
        const uint32_t threads = i ? kAddThreadsSmall : kAddThreads;
        const uint32_t every = frames > 1 ? add_pass_rest(chunk, (chunk & 3u) == 0, threads) : 0u;
        const uint32_t end = add_pass_rest(last, (((frames - 1) * chunk) & 3u) == 0, threads);
        rest[i] = every > end ? every : end;
    }
    return rest[1] > rest[0] + 32u ? kAddThreads : kAddThreadsSmall;
}

}  // namespace nz
