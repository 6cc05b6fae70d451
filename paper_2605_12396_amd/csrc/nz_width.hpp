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
//   a frame is one workgroup either way -- frames of 16384, 16 MB 81 / 82; 35 / 44; of 49152, 16 MB 91 / 91; 53 / 77.  256 threads where 512
//     need more rounds of workgroups on the chip, up to kComputeUnits blocks of 512: of 16384, 136 MB 379 / 302; 180 / 184; of 49152 194 /
//     161; 163 / 157; of 32768 262 / 222; 179 / 196.  Frames of exactly 65536 take 256: that was for the HUFFMAN ones, which are
//     the same by now, and FIXEDLEN loses: 4 MB 83 / 83; 46 / 71; 64 MB 115 / 115; 86 / 120, sum of two streams 152 / 152;
//   a frame's second workgroup has less than half a block -- frames of 65537, 16 MB 162 / 163; 95 / 157; 136 MB 382 / 409; 379 / 576
//     (of 98304 99 / 94; 83 / 95);
//   other frames: 4 MB 87 / 83; 76 / 72; 48 MB 111 / 105; 122 / 113; 64 MB 118 / 113; 126 / 117.  Below kSpreadFrom
//     blocks the line is a cautious one: 64 KB 67 / 65; 23 / 29, but 1.2 MB 85 / 84; 76 / 70, 3 MB 87 / 83; 85 / 77, 2 MB 87 / 80; 79 / 72.
//     Past one 256-thread workgroup per compute unit a ragged end decides (a difference of up to 32 elements a thread does not show): 72 MB
//     with one of 43136 132 / 140; 141 / 138; frames of 100003, 64 MB 190 / 186; 172 / 208.  HUFFMAN would rather have 512 there, whatever
//     the end: 80 MB, which takes 256, 124 / 135; 143 / 140.
// From 256 blocks of 512 threads on the chip is full: 256 MB 218 / 240; 216 / 297 (at 128 MB 138 / 136; 151 / 150).
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
