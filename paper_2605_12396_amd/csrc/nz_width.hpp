// nz_width.hpp -- threads per workgroup of the adding passes: a rule on the message and its frames (plain C++, no device code).
#pragma once
#include <stdint.h>

namespace nz {

// Adding passes: 512 threads (two statistics halves, two workgroups per compute unit, four wavefronts per SIMD), or 256 (one
// half, three workgroups per compute unit).  256 threads spread a message over more compute units, and half as many
// wavefronts share a unit's shared memory for their counting, but they build a frame's decode tables with half the
// threads and have half as many for a block that is taken element by element: one that a frame fills only in part, or that
// starts off a multiple of four.  What a thread is left with there counts as much as the spread.
constexpr uint32_t kAddThreads = 512, kAddThreadsSmall = 256;
constexpr uint32_t kAddResident = 2, kAddResidentSmall = 3;          // workgroups of a compute unit, by their shared memory
constexpr uint32_t kComputeUnits = 256, kSpreadFrom = 8;

// Elements that a thread of a workgroup of `threads` takes one by one, at most, in a frame of nf (aligned: the frame starts at a
// multiple of four).
inline uint32_t add_pass_rest(uint32_t nf, bool aligned, uint32_t threads) {
    const uint32_t block = threads * 256u;
    const uint32_t rest = aligned ? nf % block : (nf < block ? nf : block);
    return (rest + threads - 1u) / threads;
}

// Us per call, 512 / 256 threads, of nz_reduce_local (gradients coded HUFFMAN; uniform values coded FIXEDLEN):
//   a frame is one workgroup either way -- frames of 16384, 16 MB 126 / 135; 46 / 54; of 49152, 16 MB 173 / 201; 82 / 108.  256
//     threads where 512 need more rounds of workgroups on the chip: frames of 16384, 130 MB 508 / 465; 167 / 178; of 49152, 130 MB
//     337 / 274; 165 / 164 (but of 32768, two rounds either way, 317 / 360; 140 / 176).  And in frames of exactly 65536, which 512
//     threads take element by element when HUFFMAN: 64 MB 212 / 180, two streams 300 / 246, while FIXEDLEN loses (137 / 168; 176 / 207);
//   a frame's second workgroup has less than half a block -- frames of 65537, 16 MB 251 / 289; 168 / 230; 130 MB 322 / 541; 258 / 514
//     (of 98304 231 / 187; 143 / 140);
//   other frames: 4 MB 171 / 158; 135 / 114; 48 MB 218 / 178; 174 / 163; 64 MB 185 / 182; 170 / 170.  Below kSpreadFrom
//     blocks the ragged end is most of a message: 64 KB 109 / 117; 35 / 40; 1.2 MB 178 / 189; 138 / 111 (whole blocks would gain there
//     too, 3 MB 170 / 158; 146 / 119, and 2 MB 227 / 198; 140 / 111: the line is a cautious one).
//     Past one 256-thread workgroup per compute unit there is little left to spread and the element-by-element part decides
//     (a difference of up to 32 elements a thread does not show): 72 MB with a ragged end of 43136 190 / 230; 179 / 176, of 77056 (80 MB)
//     230 / 187; frames of 100003, 64 MB 301 / 321; 224 / 256.
// From 256 blocks of 512 threads on the chip is full: 256 MB 241 / 300; 229 / 311.
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
