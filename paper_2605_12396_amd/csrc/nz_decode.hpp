// nz_decode.hpp -- gfx950 kernel of the receiver side, and the choice of its shape: validate stream and frame headers, rebuild the
// canonical decode table from the code lengths carried in the frame, decode one 256-symbol segment per
// thread from its recorded bit offset, then dequantize (decompress), or -- front end of the fused reduce --
// stage the codes of operand A (first pass) and add operand B to them while gathering the statistics of the
// sum (second pass).  One operand per pass keeps the per-workgroup shared memory small enough for four
// waves per SIMD in workgroups of 512 threads, three in workgroups of 256.
//
// Paper mapping: receiver side of Algorithm 2 (ParseHeader, ValidateHeader, DecodeOrMemcpy) and the
// decode + reduce part of the fused receive-decode-reduce-encode-send step (Sec. IV-D).
#pragma once
#include "nz_common.hpp"
#include "nz_scan.hpp"
#include "nz_width.hpp"
#include <type_traits>

namespace nz {

constexpr uint32_t kPrimaryBits = 11;         // first-level decode table: 2048 entries (their fields: below)
enum : uint32_t { KIND_RAW = 0, KIND_FIXED = 1, KIND_HUFF = 2, KIND_ZERO = 3 };

__device__ inline uint64_t pad4d(uint64_t v) { return (v + 3u) & ~(uint64_t)3u; }
__device__ inline uint64_t pad16d(uint64_t v) { return (v + 15u) & ~(uint64_t)15u; }

// Stream header checks (format violations first, then disagreement with the caller's n / step / options).
__device__ inline uint32_t check_stream(const uint8_t* s, uint64_t bytes, const DecodeArgs& A, uint64_t& total) {
    total = 0;
    if (bytes < kStreamHdr) return ST_CORRUPT;
    const uint32_t* h = reinterpret_cast<const uint32_t*>(s);
    if (h[0] != kMagicStream || h[1] != 1u) return ST_CORRUPT;
    const uint64_t n = (uint64_t)h[2] | ((uint64_t)h[3] << 32);
    const uint32_t chunk = h[4], nfr = h[5], stepb = h[6], seg = h[7], K = h[8], pred = h[9];
    total = (uint64_t)h[10] | ((uint64_t)h[11] << 32);
    if (n == 0 || chunk == 0 || chunk > kMaxChunk) return ST_CORRUPT;
    if (seg < 32u || seg > 1024u) return ST_CORRUPT;
    if (K < 2u || K > kMaxK || (K & (K - 1u))) return ST_CORRUPT;
    if (pred > 1u) return ST_CORRUPT;
    if ((n + chunk - 1) / chunk != (uint64_t)nfr) return ST_CORRUPT;
    if (total > bytes || total < kStreamHdr + pad16d(8ull * nfr)) return ST_CORRUPT;
    if (n != A.n || stepb != A.step_bits) return ST_MISMATCH;
    if (chunk != A.chunk || K != A.K || seg != kSeg || pred != A.pred) return ST_MISMATCH;
    return ST_OK;
}

// Shared memory of one operand's decoder.
constexpr uint32_t kSubBits = 6;               // second-level tables resolve codes of 12..17 bits
constexpr uint32_t kMaxSub = 51;               // at most this many second-level tables (the rest: canonical search)
// Table entries (32 bits), one field a byte, so that a field costs one instruction:
//   byte 0  bits to go on by (an escape's include the raw word's 32)
//   byte 2  bytes of the row that the entry's codes take: 2, 4 for two codes, 0 where the entry is no symbol
//   bytes 1 and 3  the quantization codes.  Alphabets of up to kPairAlphabet symbols: the first code and the second, each at most 127 in magnitude.
//           Larger ones (WIDE in what follows): low and high byte of the only code (at most 511 in magnitude).
//   byte 3 = 0x80 (no code has it): the entry is an escape, leads to a second-level table, or stands for codes that no table resolves
//           (deep_symbol; it uses no bits up).  Byte 1 is then the place of the table that the next bits are looked up in, in units of
//           256 bytes (0: the first level).
// First level: indexed by the next 11 stream bits, which may hold two codes.  Second level: by the six after them, for codes of 12..17 bits.
constexpr int32_t kStops = (int32_t)0x81000000;                        // (signed) entries below this one are no symbols
constexpr uint32_t kStopEntry = 0x80000000u, kOneCode = 2u << 16, kEscEntry = kStopEntry | kOneCode | 32u, kPlaceMask = 0xFF00u, kPlaceSub = 0x2000u;
constexpr uint32_t kMainEntries = 1u << kPrimaryBits;
static_assert(4 * kMainEntries == kPlaceSub && 4 << kSubBits == 0x100 && 4 * (kMainEntries + (kMaxSub << kSubBits)) <= kPlaceMask + 0x100, "places of tables");
// the entry of one symbol, `bits` bits after the ones before it
__device__ inline uint32_t symbol_entry(uint32_t sy, uint32_t bits) {
    if (sy == 0) return kEscEntry + bits;
    const uint32_t q = (uint32_t)unzigzag(sy - 1u);
    return kOneCode | bits | ((q & 0xFFu) << 8);                       // (byte 3: see open_frame)
}

template <uint32_t SUBS>                       // second-level tables
struct DecTables {
    int32_t tab[kMainEntries + (SUBS << kSubBits)];
    uint16_t sorted[kMaxK];                    // (alphabets that have entries of two codes: behind their symbols, the length of every symbol's code)
    uint32_t cnt[32], first[32], idx0[32];
    __align__(16) uint32_t lim[32];            // lim[l]: end of the codes of length <= l, left-justified to 28 bits
    int32_t base[32];                          // base[l] = idx0[l] - first[l]: sorted index = (code of length l) + base[l]
    __device__ inline uint8_t* lens() { return reinterpret_cast<uint8_t*>(sorted + kMaxK / 2); }
    __device__ inline const uint8_t* lens() const { return reinterpret_cast<const uint8_t*>(sorted + kMaxK / 2); }
};
static_assert(kPairAlphabet <= kMaxK / 2 && kPairAlphabet <= kMaxK, "the lengths lie behind the sorted symbols");

// Steps after which the windows of a frame are renewed.  0: once a phase.  A window lasts for some 250 bits: a phase of 32 symbols of less than six bits and
// what the loop takes until the next one is there; from there on eight steps, of two lookups each, or six where symbols of eight bits and more are escapes for a
// percent and more, which take 32 bits besides.
__device__ inline uint32_t renew_steps(uint64_t bits, uint32_t symbols, bool often) {
    return bits < 6ull * symbols ? 0u : bits < 8ull * symbols ? 8u : often ? 6u : 8u;
}

struct FrameView {
    uint32_t status;          // ST_OK or the reason the frame was rejected
    uint32_t kind;            // KIND_*
    uint32_t w;               // FIXEDLEN width
    const uint32_t* words;    // RAW: payload words; FIXEDLEN/HUFFMAN: bitstream words
    uint32_t nwords;
    uint32_t bits;            // HUFFMAN: of the whole frame
    uint32_t seglen, bit0;    // bits of this thread's segment, and in front of it
    uint32_t renew;           // HUFFMAN: steps after which a window is renewed (0: once a phase)
    bool starts;              // (predictor) escapes are so rare that they may be the starts of segments alone
    bool escapes, subs;       // HUFFMAN: some symbol is the escape; there are codes of more than 11 bits
    bool hot_esc;             // escapes are frequent in this frame (short escape code / codes wider than the alphabet)
};

// Build-time scratch shared by both operands.
struct BuildScratch {
    __align__(4) uint8_t len[kMaxK];
    uint32_t wcnt[16 * 32];
    uint32_t red[6][8];
    uint32_t wsum[8];
};

// Sums over the workgroup of six 32-bit values (the caller keeps every total below 2^32): wave totals over the DPP
// network (no shared-memory crossbar), one barrier pair for all of them.
template <int NT>
__device__ inline void block_sum32(uint32_t (&v)[6], uint32_t (*s_red)[8]) {
    static_assert(NT / 64 <= 8, "one slot per wavefront");
#pragma unroll
    for (int k = 0; k < 6; k++) v[k] = wave_incl_scan_dpp(v[k]);          // lane 63: the wave's total
    __syncthreads();
    if (lane_id() == 63) {
#pragma unroll
        for (int k = 0; k < 6; k++) s_red[k][threadIdx.x >> 6] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 6; k++) { v[k] = 0; for (int i = 0; i < NT / 64; i++) v[k] += s_red[k][i]; }
}

// Validate one frame and prepare its decoder (all threads of the workgroup call this together).
template <int NT, uint32_t SUBS, int WIDE>
__device__ inline void open_frame(const uint8_t* s, uint64_t total, uint64_t off, uint64_t bytes, uint32_t nf, uint32_t first_seg,
                                  const DecodeArgs& A, DecTables<SUBS>* T, BuildScratch* B, FrameView& V) {
    // off: the frame's entry of the offsets table, read by the caller at kernel start; bytes: size of the stream buffer
    // (total <= bytes was checked with the stream header), the bound of the early read of the code lengths below
    const uint32_t tid = threadIdx.x;
    V.status = ST_CORRUPT; V.kind = KIND_ZERO; V.w = 0; V.words = nullptr; V.nwords = 0; V.bits = 0; V.seglen = 0; V.bit0 = 0; V.renew = 0; V.escapes = false; V.starts = false; V.subs = false;
    V.hot_esc = false;
    // (total holds the stream header and the offsets table at least; written so that no offset, however large, wraps around)
    if ((off & 15u) || off < kStreamHdr + pad16d(8ull * A.n_frames) || off > total - kHdrBytes) return;
    const uint8_t* fr = s + off;
    const uint4 h0 = reinterpret_cast<const uint4*>(fr)[0], h1 = reinterpret_cast<const uint4*>(fr)[1];
    // the code-length table of a HUFFMAN frame starts right behind the header: its words are requested together with
    // the header (inside the stream buffer; used only once the header has shown that they belong to the table)
    const uint32_t lens_word = (off + kHdrBytes + 4ull * tid + 4ull <= bytes) ? reinterpret_cast<const uint32_t*>(fr + kHdrBytes)[tid] : 0u;
    const uint32_t x = kCheckXor ^ h0.x ^ h0.y ^ h0.z ^ h0.w ^ h1.x ^ h1.y ^ h1.z;
    if (h0.x != kMagicFrame || h1.w != x) return;
    const uint32_t codec = h0.y, raw_bytes = h0.z, payload = h0.w, p0 = h1.x, p1 = h1.y;
    if (codec > 2u || raw_bytes != 4u * nf) return;
    if ((uint64_t)payload > total - kHdrBytes - off) return;
    if (h1.z != A.step_bits) { V.status = ST_MISMATCH; return; }
    const uint8_t* pay = fr + kHdrBytes;
    if (codec == CODEC_RAW) {
        if (payload != 4u * nf || p0 || p1) return;
        V.status = ST_OK; V.kind = KIND_RAW; V.words = reinterpret_cast<const uint32_t*>(pay); V.nwords = nf;
        return;
    }
    if (codec == CODEC_FIXED) {
        if (p0 > 32u || (p1 & 0x7FFFFFFFu) || (p1 >> 31) != A.pred) return;   // (the stream's predictor is the caller's: checked before)
        const uint64_t need = 4ull * (((uint64_t)nf * p0 + 31u) / 32u);
        if (payload != need) return;
        V.status = ST_OK; V.kind = KIND_FIXED; V.w = p0; V.hot_esc = (p0 >= 32u) || ((1u << p0) > A.K);
        V.words = reinterpret_cast<const uint32_t*>(pay); V.nwords = payload / 4;
        return;
    }
    // HUFFMAN
    const uint32_t nsym = p0, seg = p1 & 0xFFFFu, K = (p1 >> 16) & 0x7FFFu;
    if ((p1 >> 31) != A.pred) return;
    if (seg != kSeg || K != A.K || nsym == 0 || nsym > K) return;
    const uint32_t nseg = (nf + kSeg - 1) / kSeg;
    const uint64_t tables = pad4d(nsym) + pad4d(2ull * nseg);
    if (payload < tables || (payload & 3u)) return;
    const uint16_t* segt = reinterpret_cast<const uint16_t*>(pay + pad4d(nsym));
    // code lengths (4 per thread): <= 28, padding zero, at least one used, Kraft sum <= 1
    static_assert(NT * 4 >= kMaxK, "one pass over the code lengths");
    uint32_t bad = 0;
    uint64_t kraft = 0;
    {
        const uint32_t lw = (4u * tid < (uint32_t)pad4d(nsym)) ? lens_word : 0u;
        uint32_t clean = 0;
#pragma unroll
        for (uint32_t j = 0; j < 4; j++) {
            const uint32_t L = (lw >> (8 * j)) & 0xFFu, t = 4u * tid + j;
            if (L > kMaxLen || (t >= nsym && L)) bad = 1;
            else if (L) { kraft += 1ull << (kMaxLen - L); clean |= L << (8 * j); }
        }
        if (4u * tid < kMaxK) reinterpret_cast<uint32_t*>(B->len)[tid] = clean;
    }
    // segment table (two entries per load): bits before this workgroup's first segment, and in the whole frame
    uint32_t pre = 0, all = 0, mine = 0;
    const uint32_t end_seg = first_seg + NT;
    const uint32_t seglen = first_seg + tid < nseg ? segt[first_seg + tid] : 0u;
    {
        const uint32_t* segt32 = reinterpret_cast<const uint32_t*>(segt);
        const uint32_t npairs = (nseg + 1u) / 2u;
        for (uint32_t p2 = tid; p2 < npairs; p2 += NT) {
            const uint32_t v = segt32[p2], g = 2u * p2, v0 = v & 0xFFFFu, v1 = v >> 16;
            all += v0; if (g < first_seg) pre += v0; else if (g < end_seg) mine += v0;
            if (g + 1u < nseg) { all += v1; if (g + 1u < first_seg) pre += v1; else if (g + 1u < end_seg) mine += v1; }
            else if (v1) bad = 1;                                      // padding entry of an odd table
        }
    }
    // workgroup sums: the Kraft sum in two halves (a thread adds at most 4 x 2^27: the low 16 bits and the rest each
    // sum to less than 2^32 over the workgroup), the bits of the whole frame, those before this workgroup and its own (a segment
    // has at most 65535 bits, a frame at most 4096 segments), and the number of threads that saw something illegal
    uint32_t sums[6] = { (uint32_t)(kraft & 0xFFFFu), (uint32_t)(kraft >> 16), all, pre, bad, mine };
    block_sum32<NT>(sums, B->red);
    kraft = (uint64_t)sums[0] + ((uint64_t)sums[1] << 16);
    const uint64_t pre_bits = sums[3], all_bits = sums[2], mine_bits = sums[5];
    if (sums[4] || kraft == 0 || kraft > (1ull << kMaxLen)) return;
    const uint64_t avail = 8ull * (payload - tables);
    if (all_bits > avail || 4ull * ((all_bits + 31u) / 32u) != payload - tables) return;
    if (all_bits < nf) return;            // every symbol costs at least one bit (so the bitstream is never empty here)
    // The lines of this workgroup's part of the bitstream are touched once, side by side, while the tables are built: the
    // windows are requested lane by lane later, a few symbols ahead, and would wait for memory each time.
    constexpr uint32_t kTouch = 4;                                      // (4 x NT lines of 128 bytes: 16 bits a symbol)
    uint32_t touched[kTouch];
    {
        const uint64_t first = (uint64_t)(pay + tables) + (pre_bits >> 3), last = (uint64_t)(pay + tables) + ((pre_bits + mine_bits) >> 3);
#pragma unroll
        for (uint32_t k = 0; k < kTouch; k++) {
            typedef const uint32_t __attribute__((address_space(1))) * wptr;
            const uint64_t at = (first & ~3ull) + 128ull * (tid + k * NT);
            touched[k] = at < last ? *reinterpret_cast<wptr>(at) : 0u;
        }
    }
    V.hot_esc = B->len[0] != 0 && B->len[0] <= 6u;                   // the escape symbol has a probability of a percent or more
    V.renew = renew_steps(all_bits, nf, V.hot_esc);
    // bits in front of this thread's segment: the workgroup's, and a scan whose wavefronts meet at the next barrier
    const uint32_t seg_incl = wave_incl_scan_dpp(seglen);
    if (lane_id() == 63) B->wsum[tid >> 6] = seg_incl;
    // canonical tables and the first-level lookup
    uint32_t* s_cnt = T->cnt; uint32_t* s_first = T->first; uint32_t* s_idx0 = T->idx0;
    uint32_t rank[kMaxK / NT];
    canonical_tables<NT>(B->len, K, B->wcnt, s_cnt, s_first, s_idx0, rank);
    {
        uint32_t before = (uint32_t)pre_bits + seg_incl - seglen;
#pragma unroll
        for (uint32_t w = 0; w + 1 < NT / 64; w++) before += w < (tid >> 6) ? B->wsum[w] : 0u;
        V.bit0 = before; V.seglen = seglen; V.bits = (uint32_t)all_bits;
    }
#pragma unroll
    for (uint32_t i = 0; i < kMaxK / NT; i++) {
        const uint32_t sy = i * NT + tid;
        const uint32_t L = sy < K ? B->len[sy] : 0u;
        if (L) T->sorted[s_idx0[L] + rank[i]] = (uint16_t)sy;
        if (!WIDE && sy < K) T->lens()[sy] = (uint8_t)L;
    }
    if (tid < 32) {
        T->lim[tid] = (tid >= 1 && tid <= kMaxLen) ? ((s_first[tid] + s_cnt[tid]) << (kMaxLen - tid)) : 0u;
        T->base[tid] = (int32_t)s_idx0[tid] - (int32_t)s_first[tid];
    }
    __syncthreads();
    // Canonical codes left-justified to a common width are ordered by length, so the length of the code that
    // starts an entry's bits is found by comparing against the end of every length's range (no table walk).
    {
        uint32_t lim[kPrimaryBits + 1];                                // end of the codes of length <= l, 11-bit scale
#pragma unroll
        for (uint32_t l = 1; l <= kPrimaryBits; l++) lim[l] = T->lim[l] >> (kMaxLen - kPrimaryBits);    // (a multiple of that)
        // second-level tables: the prefixes that no code of <= 11 bits starts with, in order (the shortest of the long codes first)
        uint32_t nsub = kMainEntries - lim[kPrimaryBits];
        nsub = nsub < SUBS ? nsub : SUBS;
        // a thread's entries in three sweeps (lengths and sorted positions, symbols, entries), so that the shared-memory
        // reads of all of them are in flight together
        constexpr uint32_t EPT = (1u << kPrimaryBits) / NT;
        uint32_t LL[EPT], pos[EPT], sym[EPT];
        bool has[EPT];
        // A thread's entries i = tid + k NT differ in their top bits only, so their prefixes v = reversed(i) share all but
        // the lowest log2(EPT) bits: the limits of the short lengths are multiples of EPT and compare alike for all of
        // them (counted once), only the last lengths are compared entry by entry.
        constexpr uint32_t kLowBits = (EPT == 8) ? 3u : ((EPT == 4) ? 2u : 0u);     // log2(EPT) for the workgroup sizes in use
        static_assert(EPT == 8 || EPT == 4, "entries per thread");
        const uint32_t vhigh = __brev(tid) >> (32 - kPrimaryBits);                  // prefix of entry k = 0 (low bits zero)
        uint32_t Lshared = 1;
#pragma unroll
        for (uint32_t l = 1; l + kLowBits <= kPrimaryBits; l++) Lshared += (vhigh >= lim[l]) ? 1u : 0u;   // lim[l] is a multiple of 2^(11-l)
#pragma unroll
        for (uint32_t k = 0; k < EPT; k++) {
            const uint32_t i = tid + k * NT;
            const uint32_t v = __brev(i) >> (32 - kPrimaryBits);       // stream order: first bit is the code's MSB
            uint32_t L = Lshared;
#pragma unroll
            for (uint32_t l = kPrimaryBits - kLowBits + 1; l < kPrimaryBits; l++) L += (v >= lim[l]) ? 1u : 0u;
            LL[k] = L; has[k] = v < lim[kPrimaryBits];
            pos[k] = has[k] ? (uint32_t)((int32_t)(v >> (kPrimaryBits - L)) + T->base[L]) : 0u;
        }
#pragma unroll
        for (uint32_t k = 0; k < EPT; k++) sym[k] = T->sorted[pos[k]];
        // (the high byte of a code, where the alphabet's codes have one)
        auto entry = [&](uint32_t sy, uint32_t bits) -> uint32_t {
            return symbol_entry(sy, bits) | (WIDE && sy ? ((uint32_t)unzigzag(sy - 1u) & 0xFF00u) << 16 : 0u);
        };
#pragma unroll
        for (uint32_t k = 0; k < EPT; k++) {
            const uint32_t i = tid + k * NT, L = LL[k], sy = sym[k];
            uint32_t e = kStopEntry;
            if (has[k]) e = entry(sy, L);
            else {
                const uint32_t id = (__brev(i) >> (32 - kPrimaryBits)) - lim[kPrimaryBits];
                if (id < nsub) e = kStopEntry | (4u * (kMainEntries + (id << kSubBits))) | kPrimaryBits;
            }
            T->tab[i] = (int32_t)e; LL[k] = e;
        }
        // second level, table by table
        constexpr uint32_t W2 = kPrimaryBits + kSubBits;
        uint32_t lim2[kSubBits + 1];                                   // end of the codes of length <= 11 + l, 17-bit scale
#pragma unroll
        for (uint32_t l = 1; l <= kSubBits; l++) lim2[l] = T->lim[kPrimaryBits + l] >> (kMaxLen - W2);
#pragma unroll 1
        for (uint32_t idx = tid; idx < (nsub << kSubBits); idx += NT) {
            const uint32_t v = ((lim[kPrimaryBits] + (idx >> kSubBits)) << kSubBits) | (__brev(idx & ((1u << kSubBits) - 1u)) >> (32 - kSubBits));
            uint32_t L = kPrimaryBits + 1;
#pragma unroll
            for (uint32_t l = 1; l < kSubBits; l++) L += (v >= lim2[l]) ? 1u : 0u;
            uint32_t e = kStopEntry | (4u * (kMainEntries + (idx & ~((1u << kSubBits) - 1u))));   // (stays in this table)
            if (v < lim2[kSubBits]) e = entry(T->sorted[s_idx0[L] + (v >> (W2 - L)) - s_first[L]], L - kPrimaryBits);
            T->tab[kMainEntries + idx] = (int32_t)e;
        }
        // Two codes that 11 bits hold together become one entry: what follows an entry's first code stands in the first level too, at the
        // bits that are left, where a code that they hold whole is found whatever comes after them.  (No code of five bits or less: no pair.  Frames of six bits a symbol
        // and more have next to none, and their loop stores one code a lookup: 4 MB at 6.6 bits 47.3 -> 46.5 us, a 128 MB field at 7.9 79 -> 77.)
        if (!WIDE && V.renew == 0 && lim[5] != 0) {
            __syncthreads();
            uint32_t second[EPT];
#pragma unroll
            for (uint32_t k = 0; k < EPT; k++) second[k] = (uint32_t)T->tab[(tid + k * NT) >> (LL[k] & 15u)];
            __syncthreads();
#pragma unroll
            for (uint32_t k = 0; k < EPT; k++) {
                const uint32_t bits = (LL[k] & 0xFFu) + (second[k] & 0xFFu);
                if ((int32_t)LL[k] >= 0 && (int32_t)second[k] >= 0 && bits <= kPrimaryBits)
                    T->tab[tid + k * NT] = (int32_t)((LL[k] & 0xFF00u) | (2u * kOneCode) | bits | ((second[k] & 0xFF00u) << 16));
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kTouch; k++) asm volatile("" :: "v"(touched[k]));
    V.status = ST_OK; V.kind = KIND_HUFF;
    V.escapes = B->len[0] != 0; V.starts = A.pred && B->len[0] >= 8u; V.subs = T->lim[kPrimaryBits] < (1u << kMaxLen);
    V.words = reinterpret_cast<const uint32_t*>(pay + tables); V.nwords = (uint32_t)((payload - tables) / 4);
}

// Per-thread sequential reader of one HUFFMAN segment.  Every lane owns a small window (W words) in LDS, filled from
// global memory with dword-aligned 16-byte loads that start one word in front of the one the lane is in.  The windows of a wavefront are
// renewed together, once a phase of 32 symbols or, where symbols have many bits, every few steps, from loads requested a few steps
// ahead, and by a lane on its own where it has come too far into its window.
// What bounds the loop is vector issue and the chain from one lookup to the next, which alone is left where the chip is not full (a trip to
// shared memory takes some 125 cycles, a branch 40, a dependent vector instruction 8: measured, one wavefront on a SIMD).  A step makes two lookups out of
// 32 bits, each of which finds one symbol or two, and reads three window words for the next step.  A lookup that finds an
// escape or a long code ends the step: the escape's entry has skipped the raw word, which is then the 32 bits in front of the new position,
// two of the words that are read anyway; a long code's next lookup goes to a second-level table.  So no lookup is ever made twice, and what is
// rare costs a mask.  How many symbols lanes find differs, so each has a place of its own in its row, and the loop goes on until all have 32:
// rows hold three more.
// Measured against four lookups of one symbol each out of 64 bits, some of which were made again behind an escape (us): decompression of 4 MB at ten
// bits a symbol 67 -> 47, of 4 MB of gradients 48 -> 39, of a 512 MB field of 7.8 bits 276 -> 231, of 256 MB of gradients 76 -> 74 (28.5 -> 19.8 vector
// instructions a symbol, 79 -> 56 % of the issue slots); sum of eight 128 MB messages of ten bits 795 -> 680, ring step on 44 MB 126 -> 119.
// Alphabets that have no entries of two codes (WIDE) are kernels of their own: in a loop that stored a second code for every lookup, with the 12 or 24 tables
// that the wider rows leave, and in which a long code waited for the next two steps, they lost (us, four lookups / that loop / these kernels): alphabet of 1024,
// decompression of 64 MB at 4.9 bits a symbol 44 / 48 / 44, at 8.2 104 / 113 / 101, of 256 MB 171 / 190 / 158, sum of two 128 MB messages at 8.2 bits
// 328 / 349 / 315, of gradients 236 / 260 / 228, ring step on them 178 / 189 / 164, sum of four 64 MB messages 539 / 598 / 530; of 512, 64 MB at 4.9 bits 40 / 46 / 42.
// Kept out: a loop for all kinds of frames with the kind asked for in every step (4 MB at 4.9 bits 36 -> 41), one 32-bit store for two codes
// (at odd halfwords the shared memory stalls, 32 cycles a symbol), the window words kept in registers from step to step (no faster).
// Positions count from two bits in front of the lane's next one: the byte offset of a table entry is then a mask away.
// Near the end of the bitstream words are fetched one by one with the index clamped to the last word, so any
// input stays in bounds (a valid stream never consumes a clamped word).  The words in front of the bitstream, which
// the first window starts with, are the end of the frame's tables (8 bytes at least).
constexpr uint32_t kMainMask = ((1u << kPrimaryBits) - 1u) << 2, kSubMask = ((1u << kSubBits) - 1u) << 2;
constexpr uint32_t kWinOver = 4;               // rows behind the window that two steps may read
constexpr uint32_t kTwoCodes = 0x09030801u;    // byte selectors, entry to row: bytes 1 and 3, each with its sign behind it
constexpr uint32_t kOneWideCode = 0x0C0C0301u; // bytes 1 and 3, and zeros

// The tile: 16-bit quantization codes, 32 per thread between two output phases, so that eight lanes write
// one thread's run of 32 consecutive elements together (a full 128-byte line of fp32 or int32 output); behind them those of the
// next phase that the steps have come to.
constexpr uint32_t ahead(int wide) { return wide ? 1u : 3u; }                        // symbols that a step may take beyond the phase
constexpr uint32_t tile_stride(int wide) { return kTile16R + (wide ? 2u : 6u); }     // halfwords per row: 17 or 19 words, an odd word stride
constexpr uint32_t row_spare(int wide) { return 2 * (tile_stride(wide) - 1u); }      // (bytes) a place of the row that nothing reads


// A window that is renewed once a phase is requested when no lane needs more symbols than this: early, so that its loads are on their
// way while the rest is decoded, but so that windows of w words last until the next one is installed, some 28 symbols more.  At most 14: parts of a frame
// have longer codes than others, and a lane that runs out of its window waits for a load of its own.  us with at most 10 / 14 / 20: decompression
// of 256 MB at 4.9 bits a symbol 96.5 / 95.8 / 94, of a field of 512 MB at 4.3 143 / 140 / 142, of 125 MB at 4.4 47 / 47 / 53.
__device__ inline int32_t ask_late(uint32_t w, uint32_t bits, uint32_t symbols) {
    const int32_t spare = (int32_t)((uint64_t)(32u * w - 139u) * symbols / bits) - 28;
    return spare < 6 ? 6 : spare > 14 ? 14 : spare;
}

template <int NT, uint32_t SUBS, uint32_t W, bool SHARED, int WIDE>
struct HuffReader {
    static constexpr uint32_t kSel = WIDE ? kOneWideCode : kTwoCodes;
    static constexpr uint32_t kLimit = 32 * (W - 2);       // two words from a position below this one lie inside the window
    static_assert((kLimit - 1 + 2 * (kPrimaryBits + kPrimaryBits + 32)) / 32 + 2 < W + kWinOver, "what two steps read past their window");
    uint64_t bits_addr;                  // byte address of bitstream word 0
    int32_t nwords;                      // words in the bitstream (at least 1)
    uint32_t* win;                       // this lane's window in LDS (word j at win[j * NT])
    const uint32_t* win0; uint32_t lane4;   // the first lane's, and how many bytes behind it this one is
    int32_t win_bit0;                    // bit index (relative to bitstream bit 0) of window word 1
    uint32_t p;                          // position from there on: two bits before the next stream bit
    int32_t start_bit;
    uint32_t c;                          // the 32 bits at p
    uint32_t c1;                         // (frames without escapes) the 32 bits behind those
    uint32_t limit;                      // positions below it have the words they need in the window
    uint32_t mask, base;                 // the table that the next lookup goes to
    uint32_t bad;
    bool seen;                           // (RARE) an escape
    const DecTables<SUBS>* T;
    __device__ inline void init(const FrameView& V, const DecTables<SUBS>* tables, uint32_t bitpos, const void* safe16,
                                uint32_t* windows) {
        T = tables; bad = 0; seen = false; win = windows + threadIdx.x; win0 = windows; lane4 = 4u * threadIdx.x; mask = kMainMask; base = 0; c = 0; c1 = 0; limit = V.escapes ? kLimit : kLimit - 21u;
        if (V.nwords == 0 || V.kind != KIND_HUFF) {                      // not a HUFFMAN frame: the reader is never used
            bits_addr = reinterpret_cast<uint64_t>(safe16); nwords = 1;
        } else {
            bits_addr = reinterpret_cast<uint64_t>(V.words); nwords = (int32_t)V.nwords;
        }
        start_bit = (int32_t)bitpos - 2;
        place(start_bit);
    }
    __device__ inline void place(int32_t cur) { win_bit0 = cur & ~31; p = (uint32_t)cur & 31u; }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
    typedef const u32x4_a4 __attribute__((address_space(1))) * gptr;     // plain global loads, not flat ones
    static constexpr uint32_t kLoads = (W + 3) / 4;
    // the window is stored word-major (word j of every lane side by side): conflict-free for equal j
    __device__ inline void put_window(const u32x4 (&x)[kLoads]) {
#pragma unroll
        for (uint32_t j = 0; j < W; j++) win[j * NT] = x[j / 4][j % 4];
    }
    // the word in front of the one that position `at` lies in, that one, and the next
    __device__ inline void read_words(uint32_t at, uint32_t& a, uint32_t& b, uint32_t& d) const {
        const uint32_t* w = word_at(at);
        a = w[0]; b = w[NT]; d = w[2 * NT];
    }
    // What a rare branch loads has arrived before the branch ends: left to the first use of its registers, the wait would
    // stand in the common path too, and there it would be for the windows requested ahead.
    __device__ static inline void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); asm volatile("" ::: "memory"); }   // vmcnt(0)
    __device__ inline void reload() {
        const int32_t cur = win_bit0 + (int32_t)p, wi = (cur >> 5) - 1;  // (wi = -2: the early bits of the first segment)
        if (__builtin_expect(wi + (int32_t)(4 * kLoads) <= nwords, 1)) {
            // dword-aligned 16-byte loads straight from the lane's position (no alignment waste)
            gptr g = reinterpret_cast<gptr>(bits_addr + 4ll * wi);
            u32x4 x[kLoads];
#pragma unroll
            for (uint32_t k = 0; k < kLoads; k++) x[k] = g[k];
            wait_loads();
            put_window(x);
        } else {
            // near the end of the bitstream: word by word, indices clamped to the last word
            typedef const uint32_t __attribute__((address_space(1))) * wptr;
            wptr w = reinterpret_cast<wptr>(bits_addr);
            const int32_t last = nwords - 1;
#pragma unroll 1
            for (int32_t j = 0; j < (int32_t)W; j++) win[j * NT] = w[wi + j < last ? wi + j : last];
        }
        place(cur);
    }
    // Scheduled refill of all windows of the wavefront in two halves, so that the global-load latency passes while it does
    // something else: request() issues the loads for the windows at the current positions, install() makes them the windows of
    // lanes that have moved on since.  SHARED: a window's 48 bytes are loaded by three neighbouring lanes, whichever segment
    // they decode, so that a load touches 22 places, not 64.  That pays where windows are renewed every few symbols, which
    // is what the passes of a reduce over streams of many bits a symbol do; where they are renewed every 32 the exchange of positions costs
    // as much as it saves.
    // A lane too close to the end of the bitstream for 16-byte loads has 48 harmless bytes in front of the bitstream read
    // instead and refills the slow way at install time.  Only readers of an accepted HUFFMAN frame request windows; its
    // bitstream (at least one word) is preceded by the 32-byte frame header, at least 8 bytes of tables and the stream
    // header, so those 48 bytes lie inside the stream.
    struct Pending { u32x4 x[kLoads]; int32_t cur; bool ok; };
    static __device__ inline uint32_t me() { uint32_t l = lane_id(); asm volatile("" : "+v"(l)); return l; }       // (what follows from it is not kept in registers)
    static __device__ inline void piece(uint32_t r, uint32_t me, uint32_t& lane, uint32_t& part) {       // of load r: whose window, which 16 bytes
        const uint32_t j = r * 64u + me;
        lane = (j * 171u) >> 9;                                          // j / 3 for j < 192
        part = j - 3u * lane;
    }
    __device__ inline void request(Pending& P) const {
        static_assert(kLoads == 3, "three lanes a window");
        P.cur = win_bit0 + (int32_t)p;
        const int32_t wi = (P.cur >> 5) - 1;
        P.ok = wi + (int32_t)(4 * kLoads) <= nwords;
        const int32_t src = P.ok ? wi : -(int32_t)(4 * kLoads);
        const uint32_t self = SHARED ? me() : 0u;
#pragma unroll
        for (uint32_t r = 0; r < kLoads; r++) {
            uint32_t l, part;
            piece(r, self, l, part);
            P.x[r] = SHARED ? *reinterpret_cast<gptr>(bits_addr + 4ll * (__shfl(src, (int)l, 64) + (int32_t)(4u * part)))
                            : reinterpret_cast<gptr>(bits_addr + 4ll * src)[r];
        }
    }
    __device__ inline void install(const Pending& P) {
        wait_loads();
        if (SHARED) {
            const uint32_t self = me();
#pragma unroll
            for (uint32_t r = 0; r < kLoads; r++) {
                uint32_t l, part;
                piece(r, self, l, part);
                uint32_t* w = win - self + l + part * (4u * NT);
#pragma unroll
                for (uint32_t i = 0; i < 4; i++)
                    if (4 * (kLoads - 1) + i < W || part + 1u < kLoads) w[i * NT] = P.x[r][i];
            }
        }
        const int32_t cur = win_bit0 + (int32_t)p, bit0 = P.cur & ~31;
        if (__builtin_expect(P.ok && cur - bit0 < (int32_t)limit, 1)) {
            if (!SHARED) put_window(P.x);
            win_bit0 = bit0; p = (uint32_t)(cur - bit0);                 // (P.cur <= cur: positions only grow)
        } else reload();
        look();
    }
    __device__ inline const uint32_t* word_at(uint32_t at) const {
        // (a row of words is a power of two of bytes and a lane's place in it lies below: the address takes a shift and an and-or)
        static_assert((NT & (NT - 1)) == 0, "rows of a power of two");
        const uint32_t off = ((at * (NT / 8u)) & ~(4u * NT - 1u)) | lane4;
        return reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(win0) + off);
    }
    __device__ inline void look() {
        const uint32_t* w = word_at(p);
        const uint32_t b = w[NT], d = w[2 * NT], f = w[3 * NT];
        c = __builtin_amdgcn_alignbit(d, b, p);
        c1 = __builtin_amdgcn_alignbit(f, d, p);
    }
    __device__ inline uint32_t consumed() const { return (uint32_t)(win_bit0 + (int32_t)p - start_bit); }
    __device__ inline int32_t entry(uint32_t off) const {
        return *reinterpret_cast<const int32_t*>(reinterpret_cast<const uint8_t*>(T->tab) + off);
    }
    // A code that neither table resolves (longer than 17 bits, unassigned, or no second-level table left), from the 30 bits w of the
    // stream: its symbol and the bits to go on by.  Found in the second-level table at `from` it has its first 11 bits
    // behind it: they are that table's prefix.  Bits that start no code take their lane one bit on from where it is: positions never
    // go back, which the windows requested ahead rely on (install).  v = the 28 stream bits from its start as a number, first bit most significant.  Canonical codes left-justified to 28 bits are ordered by length, so the length is 12 + the number of
    // lengths 12..27 whose range ends at or below v; the symbol follows from the canonical order.  All limits are read at
    // once (no dependent loop).
    __device__ inline uint32_t deep_symbol(uint32_t w, uint32_t from, uint32_t& L) {
        uint32_t li = 0;
        asm volatile("" : "+v"(li));                                     // keeps the limit reads inside this rare path
        const uint4* lp = reinterpret_cast<const uint4*>(T->lim + li);
        const uint4 l3 = lp[3], l4 = lp[4], l5 = lp[5], l6 = lp[6], l7 = lp[7];     // lim[12..31]
        uint32_t v = __brev(w) >> 4;
        if (from) v = (T->lim[kPrimaryBits] + (((from - kPlaceSub) >> 8) << (kMaxLen - kPrimaryBits))) | (v >> kPrimaryBits);
        static_assert(kPrimaryBits == 11 && kMaxLen == 28, "limits 12..27 are compared below");
        L = 12u + (v >= l3.x) + (v >= l3.y) + (v >= l3.z) + (v >= l3.w) + (v >= l4.x) + (v >= l4.y) + (v >= l4.z) + (v >= l4.w) +
            (v >= l5.x) + (v >= l5.y) + (v >= l5.z) + (v >= l5.w) + (v >= l6.x) + (v >= l6.y) + (v >= l6.z) + (v >= l6.w);
        if (v >= l7.x) { bad = 1; L = 1; return 1u; }                    // no code starts with these bits
        const uint32_t sy = T->sorted[(uint32_t)((int32_t)(v >> (kMaxLen - L)) + T->base[L])];
        if (from) L -= kPrimaryBits;
        return sy;
    }
    // Two steps without a branch: what is rare (a code for deep_symbol, a value of more than 16 bits, the end of the window) is asked for behind them,
    // and lanes that it concerns make their steps (or the second) again, one by one.  A lane goes on while t < lim; its entries count as
    // nothing otherwise (ALL: every lane does).  PAIRS: the frame has entries of two codes; ESC: escapes; SUB: second-level tables.
    // RARE (without ESC): an escape is one of the rare things.
    // A lane at a code for deep_symbol is helped on where it stood still in both steps or, with alphabets that have many such codes (WIDE), in the second one
    // (alphabet of 1024, 8.2 bits a symbol, either way: decompression of 256 MB 177 / 158 us, sum of four 64 MB messages 572 / 530; for the others it
    // is code to fetch: 4 MB at 6.6 bits 47.3 / 48.5).
    template <bool PAIRS, bool ESC, bool SUB, bool ALL, bool RARE, bool BACK, typename F>
    __device__ inline void two_steps(uint8_t* tile, uint32_t row0, uint32_t& t, int32_t lim, F&& wide) {
        auto store = [&](uint32_t at, uint32_t v) { *reinterpret_cast<uint16_t*>(tile + at) = (uint16_t)v; };
        auto apart = []() { asm volatile("" ::: "memory"); };            // (two stores: one of 32 bits at an odd halfword stalls the shared memory)
        // Without escapes the bits of both steps were in the window when the first began, and only the second is made again where the window ended
        // (a field whose dense segments outrun their windows, 125 MB at 4.4 bits a symbol: 52 -> 50 us; sum of two 64 MB messages in frames of 16384 241 -> 236).
        // BACK: not in the ring step's pass of 512 threads, where the registers fall out worse for it (in frames of 16384, 64 MB 170 -> 175, 256 MB 637 -> 655).
        constexpr int kBack = ESC || RARE || !BACK ? 0 : 1;
        uint32_t p0 = p, t0 = t, base0 = base;
        uint32_t pb = p, tb = t;                                         // where the step that may be stuck began
        bool far = false;
        uint32_t entries = 0;                                            // (RARE) bit 5: an escape
        // A step stores behind the next one's first lookup, which would wait for the stores in the shared memory's queue (4 MB at 4.9 bits 34.7 -> 34.0 us, sum of
        // two 64 MB messages in frames of 16384 231 -> 228).
        uint32_t sv = 0, sv1 = 0, st = 0, st1 = 0;
        auto put_step = [&]() {
            store(st, sv);
            if (PAIRS) { apart(); store(st + 2u, sv >> 16); }
            store(st1, sv1);
            if (PAIRS) { apart(); store(st1 + 2u, sv1 >> 16); }
        };
#pragma unroll
        for (int k = 0; k < 2; k++) {
            if (WIDE && k == 1) { pb = p; tb = t; }
            if (k == kBack) { p0 = p; t0 = t; base0 = base; }
            const bool go = ALL || (int32_t)t < lim;
            int32_t e = entry(SUB ? (c & mask) | base : c & kMainMask);
            if (!ESC && k == 1) { apart(); put_step(); }
            int32_t e1 = entry((c >> ((uint32_t)e & 31u)) & kMainMask);
            if (!ALL) e = go ? e : 0;
            const bool ends = (ESC || SUB) && e < kStops;                // (an escape or a long code ends the step)
            e1 = ends || !go ? 0 : e1;
            const uint32_t t1 = t + (((uint32_t)e >> 16) & 0xFFu), t2 = t1 + (((uint32_t)e1 >> 16) & 0xFFu);
            const uint32_t used = ((uint32_t)e & 0xFFu) + ((uint32_t)e1 & 0xFFu);
            p += used;
            uint32_t a, b, d;
            if (ESC) read_words(p, a, b, d);
            else if (k == 0) c = __builtin_amdgcn_alignbit(c1, c, used); // (at most 22 bits: no trip to the window between the two steps)
            else look();
            sv = __builtin_amdgcn_perm(e, e, kSel); sv1 = __builtin_amdgcn_perm(e1, e1, kSel); st = t; st1 = t1;
            if (ESC || k == 1) put_step();
            if (RARE) entries |= (uint32_t)e | (uint32_t)e1;
            e = ends ? e : e1;
            if (SUB) {
                const uint32_t place = (uint32_t)min(e, kStops) & kPlaceMask;
                base = go ? place : base;
                mask = base ? kSubMask : kMainMask;
            }
            if (ESC) {
                c = __builtin_amdgcn_alignbit(d, b, p);
                const bool esc = ((uint32_t)e & 32u) != 0;
                const uint32_t z = __builtin_amdgcn_alignbit(c, __builtin_amdgcn_alignbit(b, a, p), 2u);     // the 32 bits in front of the next stream bit
                store((esc ? t2 : row0 + row_spare(WIDE) + 2u) - 2u, (uint32_t)unzigzag(z));
                far = far || (esc && z >= 0xFFFFu);
            }
            t = t2;
        }
        if (RARE) far = (entries & 32u) != 0;
        const bool again = far || p >= limit;
        if (__builtin_expect(__ballot(again || (p == pb && (ALL || (int32_t)tb < lim))) != 0, 0)) {
            if (RARE) seen = seen || far;
            if (again) { p = p0; t = t0; base = base0; mask = base ? kSubMask : kMainMask; look(); }
            if (again || p == pb) {
#pragma unroll 1
                for (int k = 0; k < (again ? 2 - kBack : 1); k++) if ((int32_t)t < lim) step<false>(tile, t, wide);
            }
        }
    }
    // Two lookups, whose symbols (up to four) go to the tile of 16-bit codes from byte t on; ONE: one lookup, of which one symbol counts.
    // wide(q, t) takes a value of more than 16 bits and returns what the tile is to hold.
    template <bool ONE, typename F>
    __device__ inline void step(uint8_t* tile, uint32_t& t, F&& wide) {
        auto put = [&](uint32_t at, uint32_t v) { *reinterpret_cast<uint16_t*>(tile + at) = (uint16_t)v; };
        auto put2 = [&](uint32_t at, uint32_t e) {                       // (the second code is written over where it is none)
            const uint32_t v = __builtin_amdgcn_perm(e, e, kSel);
            put(at, v);
            if (WIDE) return;
            asm volatile("" ::: "memory");
            put(at + 2u, v >> 16);
        };
        auto bits = [](int32_t e) { return (uint32_t)e & 0xFFu; };
        auto room = [](int32_t e) { return ((uint32_t)e >> 16) & 0xFFu; };
        const uint32_t from = base, p0 = p;
        int32_t e = entry((c & mask) | base);                            // (at the end: the entry that the step ends with)
        if (ONE && !WIDE) {
            if (room(e) == 2u * (kOneCode >> 16))                        // two symbols: the length of the first one's code alone
                e = (int32_t)(kOneCode | ((uint32_t)e & 0xFF00u) | T->lens()[zigzag((int32_t)((uint32_t)e << 16) >> 24) + 1u]);
        }
        put2(t, (uint32_t)e);
        uint32_t next = t + room(e);
        p += bits(e);
        if (!ONE) {
            const int32_t e1 = entry((c >> (bits(e) & 31u)) & kMainMask);
            const bool ends = e < kStops;                                // (an escape or a long code ends the step)
            const int32_t e2 = ends ? 0 : e1;
            put2(next, (uint32_t)e2);
            next += room(e2);
            p += bits(e2);
            e = ends ? e : e1;
        }
        base = e < kStops ? (uint32_t)e & kPlaceMask : 0u;
        mask = base ? kSubMask : kMainMask;
        bool esc = ((uint32_t)e & 32u) != 0;
        // A code for deep_symbol uses no bits up and stays in its table: here only if it is what the step began with (else the next step does).
        const bool stuck = p == p0;
        uint32_t a, b, d;
        read_words(p, a, b, d);
        asm volatile("" : "+v"(a));                                      // (read along with the others, not once an escape is known)
        if (__builtin_expect(__ballot(stuck || p >= limit) != 0, 0)) {
            if (stuck) {
                uint32_t L;
                const uint32_t sy = deep_symbol(c >> 2, from, L);
                put(t, (uint32_t)unzigzag(sy - 1u));
                esc = sy == 0;
                p += L + (esc ? 32u : 0u); next = t + 2u; mask = kMainMask; base = 0;
            }
            if (p >= limit) reload();
            read_words(p, a, b, d);
        }
        c = __builtin_amdgcn_alignbit(d, b, p);
        c1 = __builtin_amdgcn_alignbit(word_at(p)[3 * NT], d, p);
        t = next;
        if (esc) {
            const uint32_t z = __builtin_amdgcn_alignbit(c, __builtin_amdgcn_alignbit(b, a, p), 2u);     // the 32 bits in front of the next stream bit
            int32_t q = unzigzag(z);
            if (__builtin_expect(z >= 0xFFFFu, 0)) q = wide(q, t - 2u);
            put(t - 2u, (uint32_t)q);
        }
    }
};

// Position-addressed fetch of element e of a RAW / FIXEDLEN (or rejected = all-zero) frame.
struct DirectFetch {
    const uint32_t* words; uint32_t last, w, mask, kind;
    __device__ inline void init(const FrameView& V, const uint32_t* safe_word) {
        words = V.words; kind = V.kind; w = V.w;
        uint32_t nwords = V.nwords;
        if (kind == KIND_ZERO) { nwords = 0; w = 0; kind = KIND_FIXED; }
        if (nwords == 0) { words = safe_word; nwords = 1; }
        last = nwords - 1;
        mask = (w >= 32u) ? 0xFFFFFFFFu : ((1u << w) - 1u);
    }
    // zigzag code (FIXEDLEN) or fp32 bit pattern (RAW)
    __device__ inline uint32_t get(uint32_t e) const {
        if (kind == KIND_RAW) return words[e < last ? e : last];
        const uint64_t bp = (uint64_t)e * w;
        const uint32_t i = (uint32_t)(bp >> 5), sh = (uint32_t)(bp & 31u);
        const uint32_t lo = words[i < last ? i : last], hi = words[i + 1 < last ? i + 1 : last];
        return __builtin_amdgcn_alignbit(hi, lo, sh) & mask;
    }
};

enum : int { MODE_DECOMPRESS = 0, MODE_STAGE_A = 1, MODE_ADD_B = 2, MODE_ADD_LOCAL = 3, MODE_ADD_LOCAL_SR = 4,
             MODE_ADD_LOCAL_PLAIN = 5, MODE_ACC = 6 };
// the adding passes: ADD_B adds the staged codes of operand A, ADD_LOCAL the rank's own fp32 data, quantized on the fly
// (ADD_LOCAL_SR: by the stochastic quantizer; ADD_LOCAL_PLAIN: without the statistics of the sums, for the sampled
// arbitration, which profiles a prefix of the staged sums instead)
#define NZ_LOCAL(M) ((M) == MODE_ADD_LOCAL || (M) == MODE_ADD_LOCAL_SR || (M) == MODE_ADD_LOCAL_PLAIN)
#define NZ_STATS(M) ((M) == MODE_ADD_B || (M) == MODE_ADD_LOCAL || (M) == MODE_ADD_LOCAL_SR)
#define NZ_ADDS(M) ((M) == MODE_ADD_B || (M) == MODE_ACC || NZ_LOCAL(M))
// the passes whose other operand is the staged running value (operand A of the two-stream reduce); ACC, the
// accumulating pass of the k-ary reduce, stages its sums in operand A's format again, without statistics
#define NZ_STAGED(M) ((M) == MODE_ADD_B || (M) == MODE_ACC)

// Shared memory of one decode workgroup: the windows, and behind them (a reader's requests may touch a few rows past its
// window, whose values it does not use) the tile.  The adding passes take smaller windows and fewer second-level tables: they
// have a histogram too, and two workgroups of 512 threads are to share a compute unit.
constexpr uint32_t resident(uint32_t threads) { return threads > kDecThreads ? 2u : 3u; }      // decompressing or staging workgroups a compute unit
constexpr uint32_t win_words(int mode, int threads) { return threads > 256 && NZ_STATS(mode) ? 10u : 12u; }
constexpr bool shared_loads(int mode) { return mode == MODE_STAGE_A || NZ_STAGED(mode); }
// How many of its eight groups of the other operand an adding pass requests before it decodes a phase (the others: behind it,
// where the decoder's registers are free): what the registers hold, and with 512 threads there are 128.  All of them fit with 256
// threads and in the accumulating pass, four where the last operand's sums are counted too, three of the rank's own fp32 values (any number from none to
// four is within a hundredth there, but four spills 24: ring step on 256 MB with none / three / four 220.0 / 218.9 / 217.9, 512 MB at ten bits 543 / 550 / 551); with
// a predictor the row of running sums wants the room (none or two in the ring step: 128 MB 187 either way).  Spilled registers cost more than the groups' latency where there are many (an earlier decoder, all / this
// many, us and registers spilled: ring step on 256 MB with the predictor 303.4 / 296, 128 / 0).
constexpr uint32_t groups_ahead(int mode, int threads, int delta) {
    return mode == MODE_ADD_LOCAL_SR ? 0u : threads <= 256 ? 8u : delta ? (mode == MODE_ACC ? 2u : 0u) : NZ_LOCAL(mode) ? 3u : mode == MODE_ADD_B ? 4u : 8u;
}
// Second-level tables: what the shared memory has room for with so many workgroups to a compute unit (shapes_fit).  WIDE: the rows are shorter by
// four symbols, and the room goes to the tables, of which a large alphabet wants more: prefixes that have none go through deep_symbol, lane by lane.
constexpr uint32_t sub_tables(int mode, int threads, int wide) {
    return wide ? (!NZ_ADDS(mode) ? (threads <= 256 ? 51u : 40u) : threads <= 256 ? 34u : NZ_STATS(mode) ? 28u : 36u)
                : (!NZ_ADDS(mode) ? (threads <= 256 ? 43u : 24u) : threads <= 256 ? 26u : NZ_STATS(mode) ? 12u : 20u);
}
template <int NT, uint32_t W, int WIDE>
struct __align__(16) DecShared {
    uint32_t win[NT * W];
    union { uint16_t tile[NT * tile_stride(WIDE)]; BuildScratch build; } u;
    uint32_t zmax[2], cwide[2], lunq[2], ovf, late;
};
template <int MODE, int NT, int WIDE> using ModeTables = DecTables<sub_tables(MODE, NT, WIDE)>;
template <int MODE, int NT, int WIDE> using ModeShared = DecShared<NT, win_words(MODE, NT), WIDE>;
template <int MODE, int NT, int WIDE> using ModeReader = HuffReader<NT, sub_tables(MODE, NT, WIDE), win_words(MODE, NT), shared_loads(MODE), WIDE>;

struct SegCtx {
    uint32_t tid, lane, first_seg, nf, cntseg, e0, blk0;
    uint64_t f0;
    bool vec_ok;
};

// Second reduce pass, one element the general way: fetch A, combine, stage the sum, count its symbol.
// The sums are staged for the encoder as 16-bit codes in c16 (message order), kWideMarker where a sum needs 32
// bits, which then sits in codes; a frame with a RAW operand keeps its fp32 sums in codes.  wide[h] is raised when
// half h of the workgroup's block holds a marker.
// In the ring-step pass the other operand is the rank's own fp32 message (`local`), quantized here; an element
// that cannot be quantized counts as code 0 and raises lunq[h]: its frame becomes RAW and is redone by fix_elements.
struct AddCtx {
    StageA sa; uint32_t* codes; int16_t* c16; uint32_t* s_h; uint32_t* s_cwide; uint32_t* s_lunq;
    StageA so; bool acc;       // accumulating pass of the k-ary reduce: the sums go to this staging set, in operand A's format
    const float* local; float eb, inv;
    bool sr; SrKeys keys;      // stochastic local quantizer: draws by element offset from the workgroup's block
    bool stats;                // the pass gathers the statistics of the sums
    uint32_t ncs, copy, K; float step; bool a_raw, b_raw;
    __device__ inline void finish(const SegCtx& C, uint32_t i, uint32_t tb, uint32_t (&zmax)[2], uint32_t& overflow) const {
        const uint64_t g = C.f0 + i;
        const uint32_t h = (i - C.blk0) >> 16;
        uint32_t ta;
        if (local) {
            int32_t q;
            const bool okq = sr ? sr_quantize1(local[g], step, inv, keys.draw(i - C.blk0), q) : quantize1(local[g], eb, step, inv, q);
            if (!okq) s_lunq[h] = 1u;
            ta = (uint32_t)q;
        } else ta = sa.get(C.f0, C.nf, i, a_raw);
        if (acc) {
            if (a_raw || b_raw) { so.a32[g] = combine<true>(ta, a_raw, tb, b_raw, step, overflow); return; }
            uint32_t wide_seen = 0;
            so.put_code(C.f0, C.nf, i, (int32_t)combine<false>(ta, false, tb, false, step, overflow), wide_seen);
            if (wide_seen) s_cwide[h] = 1u;
            return;
        }
        if (a_raw || b_raw) { codes[g] = combine<true>(ta, a_raw, tb, b_raw, step, overflow); return; }
        const uint32_t t = combine<false>(ta, false, tb, false, step, overflow);
        const int32_t Q = (int32_t)t;
        if (Q > 32767 || Q <= kWideMarker) { c16[g] = (int16_t)kWideMarker; codes[g] = t; s_cwide[h] = 1u; }
        else c16[g] = (int16_t)Q;
        if (!stats) return;
        const uint32_t z = zigzag(Q);
        zmax[h] = z > zmax[h] ? z : zmax[h];
        atomicAdd(&s_h[h * 1024u + (bin_of(z, K) << ncs) + copy], 1u);
    }
};

// Four consecutive sums of an adding pass: counted (h: the half of the workgroup's block, zm: its largest symbol), then
// stored as 16-bit codes at `at`; a sum outside them goes to c32 and leaves a marker.  A wavefront comes here with all
// its lanes or, at the end of a frame, with the low ones.
template <int MODE, bool WHOLE_LINES = true>
__device__ inline void put_sums(const AddCtx& X, uint32_t lane, bool hot_esc, uint32_t h, const int32_t (&Q)[4], uint32_t& zm,
                                int16_t* at, uint32_t* c32) {
    if (!NZ_STATS(MODE)) {
        // (no statistics in this pass)
    } else if (hot_esc) {
        // Where escapes are frequent (sums of many peers: most codes leave the alphabet) they all hit one
        // bin, whose few copies serialise the wave.  They are counted per wavefront and added once; h is the
        // same for all of it.  (Uniform branch: the incoming frame's kind.)
        uint32_t wave_esc = 0;
#pragma unroll
        for (uint32_t j = 0; j < 4; j++) {
            const uint32_t z = zigzag(Q[j]);
            zm = z > zm ? z : zm;
            const bool esc = z >= X.K - 1u;
            wave_esc += (uint32_t)__builtin_popcountll(__ballot(esc));
            if (!esc) atomicAdd(&X.s_h[h * 1024u + (z << X.ncs) + X.copy], 1u);
        }
        if (lane == 0 && wave_esc) atomicAdd(&X.s_h[h * 1024u + ((X.K - 1u) << X.ncs)], wave_esc);
    } else {
#pragma unroll
        for (uint32_t j = 0; j < 4; j++) {
            const uint32_t z = zigzag(Q[j]);
            zm = z > zm ? z : zm;
            atomicAdd(&X.s_h[h * 1024u + (bin_of(z, X.K) << X.ncs) + X.copy], 1u);
        }
    }
    const int32_t qhi = max(max(Q[0], Q[1]), max(Q[2], Q[3])), qlo = min(min(Q[0], Q[1]), min(Q[2], Q[3]));
    uint32_t w0 = ((uint32_t)Q[0] & 0xFFFFu) | ((uint32_t)Q[1] << 16), w1 = ((uint32_t)Q[2] & 0xFFFFu) | ((uint32_t)Q[3] << 16);
    if (__builtin_expect(qhi > 32767 || qlo <= kWideMarker, 0)) {
        uint32_t hw[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; j++) {
            const bool wd = Q[j] > 32767 || Q[j] <= kWideMarker;
            if (wd) c32[j] = (uint32_t)Q[j];
            hw[j] = wd ? (uint32_t)(uint16_t)kWideMarker : ((uint32_t)Q[j] & 0xFFFFu);
        }
        w0 = hw[0] | (hw[1] << 16); w1 = hw[2] | (hw[3] << 16);
        X.s_cwide[h] = 1u;
    }
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef u32x2 u32x2_a2 __attribute__((aligned(2)));
    u32x2 v; v.x = w0; v.y = w1;
    if constexpr (MODE == MODE_ACC || !WHOLE_LINES) *reinterpret_cast<u32x2_a2*>(at) = v;   // (read again by the next pass; parts of lines)
    else __builtin_nontemporal_store(v, reinterpret_cast<u32x2_a2*>(at));   // streaming: should not displace the bitstream in L2
}

// Orders a wavefront's own accesses to shared memory for the compiler (the hardware keeps them in order): what its lanes
// wrote before is read by its other lanes after.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// HUFFMAN frame: every thread decodes its 256-symbol segment 32 symbols at a time into its tile row, and its wavefront
// consumes its own 64 rows with coalesced accesses (eight lanes per row).  The wavefronts of a workgroup share the tables
// only: none waits for another between the tables and the last symbol.
//   MODE_DECOMPRESS  dequantize and store fp32
//   MODE_STAGE_A     store the 16-bit codes
//   MODE_ADD_B       add the staged codes of A, store the sums as 16-bit codes, count their symbols per half of
//                    kHalf elements
//   MODE_ADD_LOCAL   the same with the rank's own fp32 data, quantized here, in the place of A
// A code that does not fit 16 bits (an escape with a large value) goes to memory and leaves kWideMarker in the tile; only
// then does the consumer look for markers.  Decompression is done with it by that; the adding passes keep it in the 32-bit
// word of its sum, where the consumer finds it.
// DELTA: the stream carries differences; the thread keeps the running sum of its segment (modulo 2^32) and a sum
// that does not fit 16 bits is finished by the decoding lane like a wide escape.
template <int MODE, int NT, int DELTA, int WIDE>
__device__ inline void run_huff(const DecodeArgs& A, const SegCtx& C, ModeReader<MODE, NT, WIDE>& ra, ModeShared<MODE, NT, WIDE>* S, const FrameView& V,
                                bool hot_esc, const AddCtx& X, bool a_wide, uint32_t (&zmax)[2], uint32_t& overflow) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef u32x2 u32x2_a2 __attribute__((aligned(2)));
    typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
    constexpr uint32_t LPR = kTile16R / 4;            // 8 lanes consume one row
    constexpr uint32_t RPK = 64 / LPR;                // rows covered by one step k of the consumer
    const uint32_t wrow = __builtin_amdgcn_readfirstlane(C.tid & ~63u);   // first row (= segment of the block) of this wavefront
    if ((C.first_seg + wrow) * kSeg >= C.nf) return;
    constexpr uint32_t kTile16Stride = tile_stride(WIDE), kAheadSyms = ahead(WIDE);
    uint16_t* tile = S->u.tile;
    uint32_t* far = MODE == MODE_DECOMPRESS ? reinterpret_cast<uint32_t*>(A.out) : MODE == MODE_STAGE_A || MODE == MODE_ACC ? (MODE == MODE_ACC ? X.so.a32 : X.sa.a32) : X.codes;
    const uint32_t renew = V.renew;
    const int32_t ask = 2 * ask_late(win_words(MODE, NT), V.bits, C.nf);
    uint32_t mark = 0;                                // bit 0: this lane left a marker in the phase's tile; bit 1: in the symbols that are ahead
    typename ModeReader<MODE, NT, WIDE>::Pending pend;
    if (DELTA && V.starts) ra.limit = ra.kLimit - 21u;
    // Streams of differences: a segment's first symbol is the code itself and escapes more often than not, the others may never.  Where the escape's
    // code is as rare as that (V.starts), a wavefront takes the steps without escapes from its second phase on, until it comes to one.
    // us, with escapes all along / this: decompression of a 4 MB line 40.9 / 39.1, of 128 MB 52 / 49.5, with a jump in 3000 symbols besides 40.8 / 41.7, in 1400 41.0 / 43.8.
    bool escapes = V.escapes;
    ra.request(pend);
    ra.install(pend);
    auto wide_code = [&](int32_t q, uint32_t i) -> int32_t {     // element i's code is outside the tile's 16 bits: kept elsewhere, marked there
        if (MODE == MODE_DECOMPRESS) A.out[C.f0 + i] = dequantize1(q, A.step);
        else if (MODE == MODE_STAGE_A) { X.sa.a32[C.f0 + i] = (uint32_t)q; S->cwide[wrow / (kHalf / kSeg)] = 1u; }
        else (MODE == MODE_ACC ? X.so.a32 : X.codes)[C.f0 + i] = (uint32_t)q;       // (the place of the sum, until the consumer has made it)
        return kWideMarker;
    };
    uint32_t acc = 0;                                 // DELTA: the code before this one (0 at the segment start)
    // consumer: lane (row rw0 + RPK k, columns c .. c+3) for k = 0..7
    const uint32_t rw0 = wrow + C.lane / LPR, c = (C.lane % LPR) * 4;
    const uint32_t* src0 = reinterpret_cast<const uint32_t*>(tile + rw0 * kTile16Stride + c);
    const uint32_t eo0 = (C.first_seg + rw0) * kSeg + c;
    const bool whole = C.vec_ok && (C.first_seg + wrow + 64u) * kSeg <= C.nf;   // every access is a full, aligned group of 4
    const bool fast_add = NZ_ADDS(MODE) && whole && !a_wide && !X.a_raw;
    // staged codes (StageA::at16): a row of the wavefront's half, phase-major if the frame fills the half
    const uint32_t h = wrow / (kHalf / kSeg), h0 = C.blk0 + h * kHalf;
    const bool half_full = h0 + kHalf <= C.nf;
    const uint32_t st_row = half_full ? kTile16R : kSeg, st_phase = half_full ? kHalf / 8u : kTile16R;
    const uint64_t st_at = C.f0 + h0 + (rw0 % (kHalf / kSeg)) * st_row + c;
    uint32_t zm = 0;
    // what a lane does with its four codes of step k of the phase that starts at r0 (whole_lines: eight lanes write a whole 128-byte
    // line or an aligned half; a constant of the type, since of two stores that differ in the streaming hint alone the compiler keeps the plain one)
    auto out4 = [&](uint32_t k, uint32_t r0, auto whole_lines) {
        const uint32_t* src = src0 + k * RPK * (kTile16Stride / 2);
        const uint32_t p0 = src[0], p1 = src[1];
        // streaming store: the output is not read again here and should not displace the bitstream in L2
        f32x4 v;
        v.x = dequantize1((int32_t)(int16_t)(p0 & 0xFFFFu), A.step); v.y = dequantize1((int32_t)p0 >> 16, A.step);
        v.z = dequantize1((int32_t)(int16_t)(p1 & 0xFFFFu), A.step); v.w = dequantize1((int32_t)p1 >> 16, A.step);
        f32x4_a4* at = reinterpret_cast<f32x4_a4*>(A.out + C.f0 + eo0 + r0 + k * RPK * kSeg);
        if constexpr (decltype(whole_lines)::value) __builtin_nontemporal_store(v, at); else *at = v;
    };
    auto stage4 = [&](uint32_t k, uint32_t r0, auto whole_lines) {       // (markers are staged as they are)
        const uint32_t* src = src0 + k * RPK * (kTile16Stride / 2);
        u32x2 v; v.x = src[0]; v.y = src[1];
        u32x2_a2* at = reinterpret_cast<u32x2_a2*>(X.sa.a16 + st_at + (r0 / kTile16R) * st_phase + k * RPK * st_row);
        if constexpr (decltype(whole_lines)::value) __builtin_nontemporal_store(v, at); else *at = v;
    };
    auto add4 = [&](uint32_t k, uint32_t r0, u32x2 va, f32x4 vl, auto whole_lines) {
        const uint32_t* src = src0 + k * RPK * (kTile16Stride / 2);
        const uint32_t p0 = src[0], p1 = src[1];
        int32_t Q[4];
        if (NZ_LOCAL(MODE)) {
            // quantize the rank's own values; one that cannot be quantized counts as 0 and flags its half
            int32_t ql[4];
            const float xl[4] = { vl.x, vl.y, vl.z, vl.w };
            bool ok = true;
            const uint32_t off = eo0 + r0 + k * RPK * kSeg - C.blk0;              // element offset inside the workgroup's block
#pragma unroll
            for (uint32_t j = 0; j < 4; j++)
                ok = (MODE == MODE_ADD_LOCAL_SR ? sr_quantize1(xl[j], X.step, X.inv, X.keys.draw(off + j), ql[j])
                                                : quantize1(xl[j], X.eb, X.step, X.inv, ql[j])) && ok;
            if (!ok) X.s_lunq[h] = 1u;
            Q[0] = (int32_t)(int16_t)(p0 & 0xFFFFu) + ql[0]; Q[1] = ((int32_t)p0 >> 16) + ql[1];
            Q[2] = (int32_t)(int16_t)(p1 & 0xFFFFu) + ql[2]; Q[3] = ((int32_t)p1 >> 16) + ql[3];
        } else {
            Q[0] = (int32_t)(int16_t)(p0 & 0xFFFFu) + (int32_t)(int16_t)(va.x & 0xFFFFu);
            Q[1] = ((int32_t)p0 >> 16) + ((int32_t)va.x >> 16);
            Q[2] = (int32_t)(int16_t)(p1 & 0xFFFFu) + (int32_t)(int16_t)(va.y & 0xFFFFu);
            Q[3] = ((int32_t)p1 >> 16) + ((int32_t)va.y >> 16);
        }
        // (the accumulating pass keeps operand A's layout: the position the codes of A came from)
        int16_t* at = MODE == MODE_ACC ? X.so.a16 + st_at + (r0 / kTile16R) * st_phase + k * RPK * st_row
                                       : X.c16 + C.f0 + eo0 + r0 + k * RPK * kSeg;
        put_sums<MODE, decltype(whole_lines)::value>(X, C.lane, hot_esc, h, Q, zm, at, (MODE == MODE_ACC ? X.so.a32 : X.codes) + C.f0 + eo0 + r0 + k * RPK * kSeg);
    };
    uint32_t t = 2u * kTile16Stride * C.tid;          // where this lane's next symbol goes (bytes from the start of the tile)
    for (uint32_t r0 = 0; r0 < kSeg; r0 += kTile16R) {
        // Instruction issue favours the wavefronts that were started first, so the workgroups that share a compute unit
        // would finish one after the other and leave it half empty towards the end of the kernel (there is nothing left
        // to start in their place).  A wavefront's priority falls as it gets through its segment, which lets the ones
        // that are behind catch up: the workgroups of a compute unit finish closer together.
        // (the levels get shorter towards the end -- phases 0-3, 4-5, 6, 7 -- so that the workgroups draw level at every
        // boundary and can only drift apart again inside the last phase)
        switch (r0 / kTile16R) {
            case 0: case 1: case 2: case 3: __builtin_amdgcn_s_setprio(3); break;
            case 4: case 5: __builtin_amdgcn_s_setprio(2); break;
            case 6: __builtin_amdgcn_s_setprio(1); break;
            default: __builtin_amdgcn_s_setprio(0); break;
        }
        u32x2 pa[NZ_STAGED(MODE) ? LPR : 1];          // the staged codes of A this lane will add
        f32x4 pl[NZ_LOCAL(MODE) ? LPR : 1];           // ring step: the rank's own values this lane will add
        const int16_t* ap = NZ_STAGED(MODE) ? X.sa.a16 + st_at + (r0 / kTile16R) * st_phase : nullptr;
        const float* lp = NZ_LOCAL(MODE) ? X.local + C.f0 + eo0 + r0 : nullptr;
        auto fetch = [&](uint32_t from, uint32_t to) {
#pragma unroll
            for (uint32_t k = 0; k < LPR; k++) {
                if (k < from || k >= to) continue;
                if (NZ_STAGED(MODE)) pa[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x2_a2*>(ap + k * RPK * st_row));
                if (NZ_LOCAL(MODE)) pl[k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_a4*>(lp + k * RPK * kSeg));
            }
        };
        constexpr uint32_t kAhead = groups_ahead(MODE, NT, DELTA);
        if (NZ_ADDS(MODE) && fast_add) fetch(0, kAhead);
        const uint32_t row0 = 2u * kTile16Stride * C.tid;                 // (t counts from the tile's first byte)
        const int32_t left = (int32_t)C.cntseg - (int32_t)r0;             // symbols of the segment from here on
        const uint32_t nr = left < (int32_t)kTile16R ? (left > 0 ? (uint32_t)left : 0u) : kTile16R;
        uint16_t* row = tile + C.tid * kTile16Stride;
        uint8_t* tileb = reinterpret_cast<uint8_t*>(tile);
        // (DELTA: differences of more than 16 bits are kept where the sums of more than 16 bits go, until they are added up)
        auto wide = [&](int32_t q, uint32_t at) -> int32_t {
            const uint32_t pl = (at - row0) / 2u;
            mark |= pl < kTile16R ? 1u : 2u;
            if (!DELTA) return wide_code(q, C.e0 + r0 + pl);
            far[C.f0 + C.e0 + r0 + pl] = (uint32_t)q;
            return kWideMarker;
        };
        // A step takes up to four symbols (two), so the last ones of a segment are taken one by one.
        const int32_t lim = (int32_t)row0 + 2 * (left - (int32_t)kAheadSyms < (int32_t)kTile16R ? left - (int32_t)kAheadSyms : (int32_t)kTile16R);
        // Windows are installed before the output's stores are issued: the wait for a window would be for them too.  And on every path from their
        // request, or the compiler has loads in flight to wait for, and the stores with them, where the next phase begins.
        auto go_on = [&]() { return __ballot((int32_t)t < lim) != 0; };
        if (renew) {
            auto steps = [&](auto sub) {
                auto two = [&]() { ra.template two_steps<false, true, decltype(sub)::value, false, false, false>(tileb, row0, t, lim, wide); };
#pragma unroll 1
                while (go_on()) {
#pragma unroll 1
                    for (uint32_t k = 2; k < renew && go_on(); k += 2) two();
                    if (!go_on()) break;
                    ra.request(pend);
                    two();
                    ra.install(pend);
                }
            };
            if (V.subs) steps(std::true_type{}); else steps(std::false_type{});
        } else {
            auto steps = [&](auto esc) {
                constexpr bool kGiveBackOne = !(NZ_LOCAL(MODE) && NT > 256);
                constexpr bool kRare = DELTA && !decltype(esc)::value;
                // (eight steps at least, for lanes that need 32 symbols and may have three; sixteen of at most two, for 31)
                if (__ballot(left < (int32_t)(kTile16R + 4u)) == 0) {
#pragma unroll 1
                    for (uint32_t k = 0; k < (WIDE ? 6 : 3); k++) ra.template two_steps<!WIDE, decltype(esc)::value, true, true, kRare, kGiveBackOne>(tileb, row0, t, lim, wide);
                }
                // Asked at the end of a turn the loop copies no registers, 52 vector instructions a turn for 67 (decompression of 4 MB at 4.9 bits 36.1 -> 34.6 us, sum of
                // two 42 MB messages 154.3 -> 150.5); the ring step's pass of 256 threads is better off with the copies (44 MB at ten bits 125 / 128).
                auto turns = [&](auto more) {
                    auto two = [&]() { ra.template two_steps<!WIDE, decltype(esc)::value, true, false, kRare, kGiveBackOne>(tileb, row0, t, lim, wide); };
                    if constexpr (NZ_LOCAL(MODE) && NT <= 256) {
#pragma unroll 1
                        while (more()) two();
                    } else if (more()) {
#pragma unroll 1
                        do two(); while (more());
                    }
                };
                turns([&]() { return __ballot((int32_t)t < lim - ask) != 0; });
                ra.request(pend);
                turns(go_on);
                ra.install(pend);
            };
            if (escapes) steps(std::true_type{}); else steps(std::false_type{});
            if (DELTA) escapes = V.escapes && (!V.starts || __ballot(ra.seen) != 0);
        }
        while (t < row0 + 2u * nr) ra.template step<true>(tileb, t, wide);
        if (DELTA) {
            // differences to running sums: a row at once, half a row where registers are short, or one by one where a code does not fit the row
            uint32_t* row32 = reinterpret_cast<uint32_t*>(row);
            uint32_t r = 0;
            if (__builtin_expect(nr == kTile16R && !(mark & 1u), 1)) {
                constexpr uint32_t kPart = NT <= 256 ? kTile16R / 2 : kTile16R / 4;              // words
#pragma unroll
                for (uint32_t at = 0; at < kTile16R / 2; at += kPart) {
                    uint32_t d[kPart], sum = acc;
                    int32_t most = 0, least = 0;
#pragma unroll
                    for (uint32_t i = 0; i < kPart; i++) d[i] = row32[at + i];
#pragma unroll
                    for (uint32_t i = 0; i < kPart; i++) {
                        const uint32_t lo = sum + (uint32_t)(int32_t)(int16_t)d[i];
                        sum = lo + (uint32_t)((int32_t)d[i] >> 16);
                        most = max(most, max((int32_t)lo, (int32_t)sum)); least = min(least, min((int32_t)lo, (int32_t)sum));
                        d[i] = __builtin_amdgcn_perm(sum, lo, 0x05040100u);
                    }
                    if (r == 2u * at && most <= 32767 && least > kWideMarker) {
#pragma unroll
                        for (uint32_t i = 0; i < kPart; i++) row32[at + i] = d[i];
                        acc = sum; r = 2u * (at + kPart);
                    }
                }
            }
#pragma unroll 1
            for (; r < nr; r++) {
                int32_t q = (int16_t)row[r];
                if (q == kWideMarker) q = (int32_t)far[C.f0 + C.e0 + r0 + r];
                acc += (uint32_t)q; q = (int32_t)acc;
                if (q > 32767 || q <= kWideMarker) { q = wide_code(q, C.e0 + r0 + r); mark |= 1u; }
                row[r] = (uint16_t)q;
            }
        }
        wave_sync();
        const bool marked = __ballot((mark & 1u) != 0) != 0, plain = whole && !marked;      // no markers in the tile, no bounds to watch
        if (NZ_ADDS(MODE) && marked) __threadfence_block();      // (the codes behind the markers are read by other lanes)
        if (MODE == MODE_DECOMPRESS && __builtin_expect(plain, 1)) {
#pragma unroll
            for (uint32_t k = 0; k < LPR; k++) out4(k, r0, std::true_type{});
        } else if (MODE == MODE_STAGE_A && __builtin_expect(whole, 1)) {
#pragma unroll
            for (uint32_t k = 0; k < LPR; k++) stage4(k, r0, std::true_type{});
        } else if (NZ_ADDS(MODE) && __builtin_expect(fast_add && plain, 1)) {
            fetch(kAhead, LPR);
#pragma unroll
            for (uint32_t k = 0; k < LPR; k++) add4(k, r0, pa[NZ_STAGED(MODE) ? k : 0], pl[NZ_LOCAL(MODE) ? k : 0], std::true_type{});
        } else {
            // A block that the frame fills in part or that starts off a multiple of four, markers in the tile, wide or raw codes of A: four
            // at a time where that can be done, else element by element.  The stores are not streamed here: groups off a multiple of four
            // meet in their lines, which then go to memory once (decompression of 64 MB in frames of 100003 elements 81 -> 58 us).  This is
            // one wavefront's work, so it shows where frames are short or none of them starts at a multiple of four (us element by element /
            // these; all wavefronts together, element by element, before: frames of 65537, 136 MB, decompression 182 / 124 (201), ring step
            // 600 / 420 (485), sum of two 693 / 500 (650); of 10001, 128 MB, 300 / 253 (238), 1162 / 850 (778), 1430 / 1033 (1000)).
            const bool four = (MODE == MODE_STAGE_A || !marked) && (!NZ_ADDS(MODE) || (!a_wide && !X.a_raw));
#pragma unroll 1
            for (uint32_t k = 0; k < LPR; k++) {
                const uint32_t eo = eo0 + k * RPK * kSeg + r0;                    // element index in the frame
                if (four && eo + 4u <= C.nf) {
                    if (MODE == MODE_DECOMPRESS) out4(k, r0, std::false_type{});
                    else if (MODE == MODE_STAGE_A) stage4(k, r0, std::false_type{});
                    else {
                        u32x2 va = { 0u, 0u };
                        f32x4 vl = { 0.0f, 0.0f, 0.0f, 0.0f };
                        if (NZ_STAGED(MODE)) va = *reinterpret_cast<const u32x2_a2*>(ap + k * RPK * st_row);
                        if (NZ_LOCAL(MODE)) vl = *reinterpret_cast<const f32x4_a4*>(lp + k * RPK * kSeg);
                        add4(k, r0, va, vl, std::false_type{});
                    }
                    continue;
                }
                const uint16_t* src = tile + (rw0 + k * RPK) * kTile16Stride + c;
                for (uint32_t j = 0; j < 4; j++) {
                    if (eo + j >= C.nf) break;
                    int32_t q = (int16_t)src[j];
                    if (MODE == MODE_STAGE_A) X.sa.a16[StageA::at16(C.f0, C.nf, eo + j)] = (int16_t)q;
                    else if (MODE == MODE_DECOMPRESS) { if (q != kWideMarker) A.out[C.f0 + eo + j] = dequantize1(q, A.step); }
                    else {
                        if (q == kWideMarker) q = (int32_t)(MODE == MODE_ACC ? X.so.a32 : X.codes)[C.f0 + eo + j];
                        X.finish(C, eo + j, (uint32_t)q, zmax, overflow);
                    }
                }
            }
        }
        wave_sync();
        // the symbols that the steps took beyond the phase become the first ones of the next
        {
            uint32_t* row32 = reinterpret_cast<uint32_t*>(row);
            const uint32_t a0 = row32[kTile16R / 2], a1 = WIDE ? 0u : row32[kTile16R / 2 + 1];
            row32[0] = a0;
            if (!WIDE) row32[1] = a1;
            t = t > row0 + 2u * kTile16R ? t - 2u * kTile16R : row0;
            mark >>= 1;
        }
    }
    if (h) zmax[1] = zm > zmax[1] ? zm : zmax[1]; else zmax[0] = zm > zmax[0] ? zm : zmax[0];
}

// RAW frames and rejected frames (= all zero): element-parallel.  RAW frames that start at a multiple of four go four elements at a
// time, and a thread has several such groups on their way at once: what bounds them is memory, and three workgroups of 256 threads
// to a compute unit, which the tables of HUFFMAN frames leave room for, do not cover its latency otherwise (us, one group at a
// time / these: decompression in frames of 65536 elements of 16 MB 44 / 21, of 256 MB 129 / 103; element by element before: sum of
// two messages of 64 MB 253 / 96, of 256 MB 726 / 380, ring step on 64 MB 198 / 71).
template <int MODE, int NT, typename SHARED>
__device__ inline void run_elementwise(const DecodeArgs& A, const SegCtx& C, const DirectFetch& da, SHARED* S,
                                       const AddCtx& X, bool a_wide, uint32_t (&zmax)[2], uint32_t& overflow) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const uint32_t cnt = (C.nf - C.blk0 < NT * kSeg) ? (C.nf - C.blk0) : NT * kSeg;
    const bool raw = da.kind == KIND_RAW;
    const uint64_t g0 = C.f0 + C.blk0;                                   // the block's first element in the message
    uint32_t wide_seen = 0;
    uint32_t i = C.tid * 4;
    if (raw && C.vec_ok) {
        constexpr uint32_t kGroups = NZ_ADDS(MODE) ? 4 : 8, kStep = NT * 4;
        const uint32_t* words = da.words + C.blk0;
        for (; i + (kGroups - 1u) * kStep + 4u <= cnt; i += kGroups * kStep) {
            u32x4 b[kGroups];
#pragma unroll
            for (uint32_t k = 0; k < kGroups; k++) b[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(words + i + k * kStep));
            if (!NZ_ADDS(MODE)) {
                uint32_t* to = (MODE == MODE_DECOMPRESS ? reinterpret_cast<uint32_t*>(A.out) : X.sa.a32) + g0 + i;
#pragma unroll
                for (uint32_t k = 0; k < kGroups; k++) {
                    if (MODE == MODE_DECOMPRESS) __builtin_nontemporal_store(b[k], reinterpret_cast<u32x4*>(to + k * kStep));
                    else *reinterpret_cast<u32x4*>(to + k * kStep) = b[k];
                }
                continue;
            }
            u32x4 a[kGroups];                                            // the other operand: fp32 bits, or codes
            if (NZ_LOCAL(MODE) || X.a_raw) {
                const uint32_t* from = (NZ_LOCAL(MODE) ? reinterpret_cast<const uint32_t*>(X.local) : X.sa.a32) + g0 + i;
#pragma unroll
                for (uint32_t k = 0; k < kGroups; k++) a[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(from + k * kStep));
            } else {
                u32x2 h[kGroups];
#pragma unroll
                for (uint32_t k = 0; k < kGroups; k++)
                    h[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(X.sa.a16 + StageA::at16(C.f0, C.nf, C.blk0 + i + k * kStep)));
#pragma unroll
                for (uint32_t k = 0; k < kGroups; k++) {
                    a[k].x = (uint32_t)(int32_t)(int16_t)(h[k].x & 0xFFFFu); a[k].y = (uint32_t)((int32_t)h[k].x >> 16);
                    a[k].z = (uint32_t)(int32_t)(int16_t)(h[k].y & 0xFFFFu); a[k].w = (uint32_t)((int32_t)h[k].y >> 16);
                    if (a_wide) {
#pragma unroll
                        for (uint32_t j = 0; j < 4; j++) if ((int32_t)a[k][j] == kWideMarker) a[k][j] = X.sa.a32[g0 + i + k * kStep + j];
                    }
                }
            }
#pragma unroll
            for (uint32_t k = 0; k < kGroups; k++) {
                const uint32_t at = i + k * kStep;
                if (NZ_LOCAL(MODE)) {
                    bool ok = true;
#pragma unroll
                    for (uint32_t j = 0; j < 4; j++) {
                        int32_t q;
                        const float x = __uint_as_float(a[k][j]);
                        ok = (MODE == MODE_ADD_LOCAL_SR ? sr_quantize1(x, X.step, X.inv, X.keys.draw(at + j), q)
                                                        : quantize1(x, X.eb, X.step, X.inv, q)) && ok;
                        a[k][j] = (uint32_t)q;
                    }
                    if (!ok) X.s_lunq[at >> 16] = 1u;
                }
                u32x4 v;
#pragma unroll
                for (uint32_t j = 0; j < 4; j++) v[j] = combine<true>(a[k][j], X.a_raw, b[k][j], true, X.step, overflow);
                *reinterpret_cast<u32x4*>((MODE == MODE_ACC ? X.so.a32 : X.codes) + g0 + at) = v;
            }
        }
    }
    for (; i < cnt; i += NT * 4) {
        const uint32_t m = (cnt - i < 4) ? (cnt - i) : 4u;
        if (MODE == MODE_DECOMPRESS && raw && m == 4u && C.vec_ok) {      // a RAW frame is a copy (payload and output 16-byte aligned)
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(da.words + C.blk0 + i));
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(A.out + g0 + i));
            continue;
        }
        for (uint32_t j = 0; j < m; j++) {
            const uint32_t e = C.blk0 + i + j;
            uint32_t t = da.get(e);                                               // fp32 bits (RAW) or zero
            if (!raw) t = (uint32_t)unzigzag(t);
            if (MODE == MODE_DECOMPRESS) A.out[C.f0 + e] = raw ? __uint_as_float(t) : dequantize1((int32_t)t, A.step);
            else if (MODE == MODE_STAGE_A) { if (raw) X.sa.a32[C.f0 + e] = t; else X.sa.put_code(C.f0, C.nf, e, (int32_t)t, wide_seen); }
            else X.finish(C, e, t, zmax, overflow);
        }
    }
    if (MODE == MODE_STAGE_A && wide_seen) { S->cwide[0] = 1u; S->cwide[1] = 1u; }   // (both halves: some code of the block is wide)
}

// FIXEDLEN frames, the streaming way: a pass of NT * 4 elements is NT * w / 8 whole words of the payload (at a 16-byte
// boundary), which the workgroup copies into shared memory with 16-byte loads (a later pass's words are requested
// before this pass is worked on); every thread then cuts its four consecutive codes out of the copy.  Two copies
// alternate (they live in the window area, which only HUFFMAN frames use), so one barrier per pass is enough.
// DELTA: the running sums of a segment are a scan over the wavefront that holds it.
// The reduce passes are bound by memory where they take four codes at a time -- the other operand's four are requested with
// the next pass's words -- and were bound by 2-byte accesses and by escapes meeting in one histogram counter while they
// went element by element: nz_reduce_k over eight 16 MB messages of 14-bit codes 1193 -> 584 us, nz_reduce_local over
// 44 MB 201 -> 155 us.  That way is left for frames that start off a multiple of four, a RAW operand, and the ends.
// Decompression and staging are bound by memory, and three workgroups of 256 threads to a compute unit, which the tables of HUFFMAN
// frames leave room for, do not cover its latency where a block is short (a header to wait for every sixteen passes) or where the
// last round leaves compute units with less.  There the words of four passes are on their way; where the chip is full one pass
// is faster (four instead: decompression of 192 MB 48.5 -> 52, of 384 MB 90 -> 95), and the adding passes gain nothing.
// us with one / four, four workgroups a compute unit before (14-bit codes): decompression in frames of 16384 elements of 64 MB 26.5 /
// 25.5 (21.7), of 256 MB 74.7 / 70.5 (68), in frames of 65536 of 128 MB 39.8 / 36.5 (40.5), of 256 MB 78.3 / 76.1 (66); sum of two
// messages of 256 MB in frames of 16384 428 / 402 (407), of 65536 370 / 333 (327).
template <int MODE, int NT, int DELTA, typename SHARED>
__device__ inline void run_fixed(const DecodeArgs& A, const SegCtx& C, const FrameView& V, SHARED* S,
                                 const AddCtx& X, bool a_wide, uint32_t (&zmax)[2], uint32_t& overflow) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    constexpr uint32_t kPass = NT * 4;                                   // elements per pass
    const bool vec = C.vec_ok && !X.a_raw;                               // staged codes and local values in groups of four
    static_assert(2 * (kPass + 8) <= sizeof(S->win) / 4, "two pass copies fit the window area");
    const uint32_t cnt = (C.nf - C.blk0 < NT * kSeg) ? (C.nf - C.blk0) : NT * kSeg;
    const uint32_t w = V.w, tid = C.tid;
    const uint32_t mask = (w >= 32u) ? 0xFFFFFFFFu : ((1u << w) - 1u);
    const uint32_t pass_words = (kPass / 32u) * w;                       // words of a whole pass (at most kPass)
    uint32_t wide_seen = 0;
    // words [4 tid, 4 tid + 4) of the pass that starts at element `base` of the block (zero where the payload ends)
    auto fetch = [&](uint32_t base) -> u32x4 {
        u32x4 x = { 0u, 0u, 0u, 0u };
        if (base >= cnt) return x;
        const uint32_t g0 = ((C.blk0 + base) >> 5) * w + 4u * tid;        // first of my words in the payload
        if (4u * tid >= pass_words || g0 >= V.nwords) return x;
        if (g0 + 4u <= V.nwords) return *reinterpret_cast<const u32x4*>(V.words + g0);
        x.x = V.words[g0];
        if (g0 + 1u < V.nwords) x.y = V.words[g0 + 1u];
        if (g0 + 2u < V.nwords) x.z = V.words[g0 + 2u];
        return x;
    };
    auto passes = [&](auto ahead) __attribute__((always_inline)) {
        constexpr uint32_t kDeep = decltype(ahead)::value;                   // passes whose words are on their way
        u32x4 nxt[kDeep];
#pragma unroll
        for (uint32_t k = 0; k < kDeep; k++) nxt[k] = fetch(k * kPass);
        for (uint32_t base0 = 0; base0 < cnt; base0 += kDeep * kPass)
#pragma unroll
        for (uint32_t it = 0; it < kDeep; it++) {
            const uint32_t base = base0 + it * kPass;
            if (base >= cnt) break;
            uint32_t* buf = S->win + (base / kPass & 1u) * (kPass + 8u);
            *reinterpret_cast<u32x4*>(buf + 4u * tid) = nxt[it];
            const uint32_t i = base + tid * 4u;
            const uint32_t m = (i < cnt) ? ((cnt - i < 4u) ? (cnt - i) : 4u) : 0u;
            const bool quad = vec && m == 4u;
            u32x2 pa; pa.x = 0; pa.y = 0;                                     // the other operand, requested before the next pass's words
            f32x4 pl = { 0.0f, 0.0f, 0.0f, 0.0f };
            if (NZ_STAGED(MODE) && quad) pa = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(X.sa.a16 + StageA::at16(C.f0, C.nf, C.blk0 + i)));
            if (NZ_LOCAL(MODE) && quad) pl = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(X.local + C.f0 + C.blk0 + i));
            nxt[it] = fetch(base + kDeep * kPass);
            __syncthreads();
            uint32_t tv[4];
            uint32_t pos = tid * 4u * w;
#pragma unroll
            for (uint32_t j = 0; j < 4; j++) {
                const uint32_t k = pos >> 5;                                  // (k + 1 <= kPass + 3: inside the copy's slack)
                tv[j] = (uint32_t)unzigzag(__builtin_amdgcn_alignbit(buf[k + 1u], buf[k], pos & 31u) & mask);
                pos += w;
            }
            if (DELTA) {
#pragma unroll
                for (uint32_t j = 0; j < 4; j++) if (j >= m) tv[j] = 0;       // (elements past the end add nothing)
                tv[1] += tv[0]; tv[2] += tv[1]; tv[3] += tv[2];
                const uint32_t before = wave_incl_scan_dpp(tv[3]) - tv[3];
                tv[0] += before; tv[1] += before; tv[2] += before; tv[3] += before;
            }
            if (MODE == MODE_DECOMPRESS && m == 4u && C.vec_ok) {
                f32x4 v;
                v.x = dequantize1((int32_t)tv[0], A.step); v.y = dequantize1((int32_t)tv[1], A.step);
                v.z = dequantize1((int32_t)tv[2], A.step); v.w = dequantize1((int32_t)tv[3], A.step);
                __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(A.out + C.f0 + C.blk0 + i));
            } else if (MODE == MODE_STAGE_A && quad) {
                uint32_t hw[4];
#pragma unroll
                for (uint32_t j = 0; j < 4; j++) {
                    const int32_t q = (int32_t)tv[j];
                    const bool wd = q > 32767 || q <= kWideMarker;
                    if (__builtin_expect(wd, 0)) { X.sa.a32[C.f0 + C.blk0 + i + j] = tv[j]; wide_seen = 1; }
                    hw[j] = wd ? (uint32_t)(uint16_t)kWideMarker : (tv[j] & 0xFFFFu);
                }
                u32x2 v; v.x = hw[0] | (hw[1] << 16); v.y = hw[2] | (hw[3] << 16);
                __builtin_nontemporal_store(v, reinterpret_cast<u32x2*>(X.sa.a16 + StageA::at16(C.f0, C.nf, C.blk0 + i)));
            } else if (NZ_ADDS(MODE) && quad) {
                // (the operand's codes have up to 31 bits here, the staged value too: the general range check)
                const uint32_t h = base >> 16;                                // (a pass lies in one half)
                static_assert(kHalf % kPass == 0 && kHalf == 65536, "a pass of the workgroup lies in one half of its block");
                uint32_t ta[4];
                if (NZ_LOCAL(MODE)) {
                    const float xl[4] = { pl.x, pl.y, pl.z, pl.w };
                    bool ok = true;
#pragma unroll
                    for (uint32_t j = 0; j < 4; j++) {
                        int32_t q;
                        ok = (MODE == MODE_ADD_LOCAL_SR ? sr_quantize1(xl[j], X.step, X.inv, X.keys.draw(i + j), q)
                                                        : quantize1(xl[j], X.eb, X.step, X.inv, q)) && ok;
                        ta[j] = (uint32_t)q;
                    }
                    if (!ok) X.s_lunq[h] = 1u;
                } else {
                    ta[0] = (uint32_t)(int32_t)(int16_t)(pa.x & 0xFFFFu); ta[1] = (uint32_t)((int32_t)pa.x >> 16);
                    ta[2] = (uint32_t)(int32_t)(int16_t)(pa.y & 0xFFFFu); ta[3] = (uint32_t)((int32_t)pa.y >> 16);
                    if (a_wide) {
#pragma unroll
                        for (uint32_t j = 0; j < 4; j++) if ((int32_t)ta[j] == kWideMarker) ta[j] = X.sa.a32[C.f0 + C.blk0 + i + j];
                    }
                }
                int32_t Q[4];
#pragma unroll
                for (uint32_t j = 0; j < 4; j++) Q[j] = (int32_t)combine<false>(ta[j], false, tv[j], false, X.step, overflow);
                int16_t* at = MODE == MODE_ACC ? X.so.a16 + StageA::at16(C.f0, C.nf, C.blk0 + i) : X.c16 + C.f0 + C.blk0 + i;
                uint32_t zm = 0;
                put_sums<MODE>(X, C.lane, V.hot_esc, h, Q, zm, at, (MODE == MODE_ACC ? X.so.a32 : X.codes) + C.f0 + C.blk0 + i);
                if (h) zmax[1] = zm > zmax[1] ? zm : zmax[1]; else zmax[0] = zm > zmax[0] ? zm : zmax[0];
            } else {
                for (uint32_t j = 0; j < m; j++) {
                    const uint32_t e = C.blk0 + i + j;
                    if (MODE == MODE_DECOMPRESS) A.out[C.f0 + e] = dequantize1((int32_t)tv[j], A.step);
                    else if (MODE == MODE_STAGE_A) X.sa.put_code(C.f0, C.nf, e, (int32_t)tv[j], wide_seen);
                    else X.finish(C, e, tv[j], zmax, overflow);
                }
            }
        }
    };
    constexpr uint32_t kResident = resident(NT) * kComputeUnits;
    const uint32_t rounds = (gridDim.x + kResident - 1) / kResident;
    const bool full = cnt > 16u * kPass && 4u * gridDim.x > 3u * kResident * rounds;       // long blocks, rounds filled by three quarters
    if (!NZ_ADDS(MODE) && !full) passes(std::integral_constant<uint32_t, 4>{});
    else passes(std::integral_constant<uint32_t, 1>{});
    if (MODE == MODE_STAGE_A && wide_seen) { S->cwide[0] = 1u; S->cwide[1] = 1u; }   // (both halves: some code of the block is wide)
}

// One workgroup per NT segments of one frame.
// FORM: bit 0 the stream carries differences (DELTA), bit 1 its alphabet has more than kPairAlphabet symbols (WIDE).
template <int MODE, int NT, int FORM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void k_decode(DecodeArgs A) {
    constexpr int DELTA = FORM & 1, WIDE = FORM >> 1;
    __shared__ ModeTables<MODE, NT, WIDE> s_t;
    __shared__ ModeShared<MODE, NT, WIDE> S;
    static_assert(sizeof(S.u) >= kWinOver * NT * sizeof(uint32_t) && offsetof(decltype(S), u) == sizeof(S.win), "what a request may touch");
    constexpr uint32_t kHist = NT * kSeg / kHalf * 1024u;               // counters: 1024 per half of the workgroup's block
    __shared__ uint32_t s_h[NZ_STATS(MODE) ? kHist : 1u];

    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const uint32_t frame = blockIdx.x / A.dbpf, db = blockIdx.x % A.dbpf;
    const uint64_t f0 = (uint64_t)frame * A.chunk;
    const uint32_t nf = (uint32_t)((A.n - f0 < A.chunk) ? (A.n - f0) : A.chunk);
    const uint32_t blk0 = db * NT * kSeg;
    if (blk0 >= nf) return;
    ResultRec* res = reinterpret_cast<ResultRec*>(A.res);
    const uint32_t first_seg = db * NT;
    const uint32_t nseg = (nf + kSeg - 1) / kSeg;
    const uint32_t gseg = first_seg + tid;
    const bool seg_valid = gseg < nseg;
    const uint32_t e0 = gseg * kSeg;                                    // first element of my segment in the frame
    const uint32_t cntseg = seg_valid ? ((nf - e0 < kSeg) ? (nf - e0) : kSeg) : 0u;
    const uint32_t hpf = (A.chunk + kHalf - 1) / kHalf;                 // halves (statistics blocks) per frame

    // the frame's entry of the offsets table is requested before the stream header is looked at (its place does not
    // depend on the header; the entry is only believed once the header is)
    uint64_t frame_off = 0;
    {
        const uint8_t* sp = NZ_STAGED(MODE) ? A.b : A.a;
        const uint64_t sb = NZ_STAGED(MODE) ? A.b_bytes : A.a_bytes;
        if (kStreamHdr + 8ull * frame + 8ull <= sb) frame_off = *reinterpret_cast<const uint64_t*>(sp + kStreamHdr + 8ull * frame);
    }
    // stream headers: the reduce passes look at both operands, so that neither goes on after a stream-level error
    uint64_t total_a = 0, total_b = 0;
    const uint32_t st_a = check_stream(A.a, A.a_bytes, A, total_a);
    uint32_t st_b = ST_OK;
    if (MODE == MODE_STAGE_A || NZ_STAGED(MODE)) st_b = check_stream(A.b, A.b_bytes, A, total_b);
    // decompress: one verdict word per workgroup (status | kind << 8), summed up by k_decode_finish; nothing here
    // touches the result record.  The reduce passes hand the worst status of what they have seen on with the words of every half, to the codebook
    // kernel; the sampled ring step's reports through a (pre-cleared) record with atomics.
    uint32_t* verdict = reinterpret_cast<uint32_t*>(A.ws + A.L.pmeta);
    if (MODE == MODE_ADD_LOCAL_PLAIN && blockIdx.x == 0 && tid == 0 && st_a) atomicMax(&res->status, st_a);
    if ((MODE == MODE_STAGE_A || MODE == MODE_ADD_LOCAL || MODE == MODE_ADD_LOCAL_SR) && blockIdx.x == 0) {
        // The first pass of a reduce clears the control block, the frame descriptors and the result record on the side: the codebook kernel is the
        // first to use them (a kernel of its own for that took 4.5 us).
        uint32_t* z = reinterpret_cast<uint32_t*>(A.ws + A.L.ctrl);
        const uint32_t words = (uint32_t)((A.L.zero_end - A.L.ctrl) / 4);
        for (uint32_t i = tid; i < words; i += NT) z[i] = 0;
        if (tid == 0) { res->bytes = 0; res->status = ST_OK; res->n_frames = A.n_frames; res->n_raw = 0; res->n_fixed = 0; res->n_huff = 0; res->reserved = 0; }
    }
    if (MODE == MODE_DECOMPRESS && st_a) {                              // nothing is written on a stream-level error
        if (tid == 0) verdict[blockIdx.x] = st_a;
        return;
    }

    FrameView V;
    V.status = ST_OK; V.kind = KIND_ZERO; V.w = 0; V.words = nullptr; V.nwords = 0; V.bits = 0; V.seglen = 0; V.bit0 = 0; V.renew = 0; V.escapes = false; V.starts = false; V.subs = false;
    V.hot_esc = false;
    if (st_a == ST_OK && st_b == ST_OK) {
        open_frame<NT, sub_tables(MODE, NT, WIDE), WIDE>(NZ_STAGED(MODE) ? A.b : A.a, NZ_STAGED(MODE) ? total_b : total_a, frame_off,
                       NZ_STAGED(MODE) ? A.b_bytes : A.a_bytes, nf, first_seg, A, &s_t, &S.u.build, V);
        if (MODE == MODE_ADD_LOCAL_PLAIN && tid == 0 && V.status) atomicMax(&res->status, V.status);
    }
    const uint32_t found_kind = V.kind;
    if (V.status) V.kind = KIND_ZERO;                                   // a rejected frame counts as zeros (and decodes to zeros)

    const uint32_t bit0 = V.bit0, seglen = V.kind == KIND_HUFF ? V.seglen : 0u;
    if (tid == 0) { S.zmax[0] = 0; S.zmax[1] = 0; S.cwide[0] = 0; S.cwide[1] = 0; S.lunq[0] = 0; S.lunq[1] = 0; S.ovf = 0; S.late = 0; }
    __syncthreads();
    const uint32_t* safe = reinterpret_cast<const uint32_t*>(A.res);
    ModeReader<MODE, NT, WIDE> ra;
    DirectFetch da;
    ra.init(V, &s_t, bit0, safe, S.win);
    da.init(V, safe);
    SegCtx C;
    C.tid = tid; C.lane = lane; C.first_seg = first_seg; C.nf = nf; C.cntseg = cntseg; C.e0 = e0; C.f0 = f0; C.blk0 = blk0;
    C.vec_ok = ((f0 & 3u) == 0);
    uint32_t overflow = 0;
    uint32_t zmax[2] = { 0, 0 };

    // Two staging sets in operand A's format: set 0 = (a16, a32, akind, awide), set 1 = the arrays of the sums (c16,
    // codes) with flag arrays of its own.  The two-stream reduce only knows set 0.  In the k-ary reduce the running
    // value alternates: the staging pass writes set A.set_in, an accumulating pass reads set A.set_in and writes the
    // other one, and the last accumulating pass ends in set 0, where the statistics pass (ADD_B) reads operand A
    // while it writes the sums in their own format to c16 / codes.
    const uint32_t si = (MODE == MODE_STAGE_A || MODE == MODE_ACC) ? (A.set_in & 1u) : 0u;
    AddCtx X;
    X.sa.a16 = reinterpret_cast<int16_t*>(A.ws + (si ? A.L.c16 : A.L.a16)); X.sa.a32 = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.codes : A.L.a32));
    X.so.a16 = reinterpret_cast<int16_t*>(A.ws + (si ? A.L.a16 : A.L.c16)); X.so.a32 = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.a32 : A.L.codes));
    X.acc = (MODE == MODE_ACC);
    X.codes = reinterpret_cast<uint32_t*>(A.ws + A.L.codes); X.c16 = reinterpret_cast<int16_t*>(A.ws + A.L.c16);
    X.s_cwide = S.cwide; X.s_lunq = S.lunq;
    X.local = NZ_LOCAL(MODE) ? A.local : nullptr; X.eb = A.eb; X.inv = A.inv_step;
    X.sr = (MODE == MODE_ADD_LOCAL_SR); X.stats = NZ_STATS(MODE);
    if (MODE == MODE_ADD_LOCAL_SR) X.keys.init(A.seed, f0 + blk0); else { X.keys.base_lo = 0; X.keys.key0 = 0; X.keys.key1 = 0; }
    X.s_h = s_h; X.K = A.K; X.step = A.step; X.ncs = 0; X.copy = 0; X.a_raw = false; X.b_raw = false;
    uint32_t* akind = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.akind1 : A.L.akind));   // per frame: operand A is RAW
    uint32_t* awide = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.awide1 : A.L.awide));   // per half: some code of A needs 32 bits
    uint32_t* akind_out = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.akind : A.L.akind1));   // (accumulating pass: the set it writes)
    uint32_t* awide_out = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.awide : A.L.awide1));
    bool a_wide = false;
    uint32_t a_status = ST_OK;
    if (NZ_ADDS(MODE)) {
        while ((A.K << (X.ncs + 1)) <= 1024u && X.ncs < 5) X.ncs++;
        X.copy = lane & ((1u << X.ncs) - 1u);
        if (NZ_STATS(MODE)) for (uint32_t i = tid; i < kHist; i += NT) s_h[i] = 0;
        X.b_raw = V.kind == KIND_RAW;
        if (NZ_STAGED(MODE)) {
            X.a_raw = akind[frame] != 0;
            for (uint32_t h = 0; h < NT * kSeg / kHalf; h++)
                if (blk0 + h * kHalf < nf) {
                    const uint32_t word = awide[(size_t)frame * hpf + blk0 / kHalf + h];
                    a_wide = a_wide || (word & 1u) != 0;
                    a_status = max(a_status, word >> 8);
                }
        } else if (db == 0 && tid == 0) akind[frame] = X.b_raw ? 1u : 0u;   // ring step: "the incoming frame is RAW"
        __syncthreads();
    }

    bool late = false;                                                  // a segment that did not use exactly its recorded bits
    if (V.kind == KIND_HUFF) {
        run_huff<MODE, NT, DELTA, WIDE>(A, C, ra, &S, V, V.hot_esc, X, a_wide, zmax, overflow);
        late = seg_valid && (ra.bad || ra.consumed() != seglen);
        if (MODE == MODE_ADD_LOCAL_PLAIN && late) atomicMax(&res->status, (uint32_t)ST_CORRUPT);
    } else if (V.kind == KIND_FIXED) {
        run_fixed<MODE, NT, DELTA>(A, C, V, &S, X, a_wide, zmax, overflow);
    } else {
        run_elementwise<MODE, NT>(A, C, da, &S, X, a_wide, zmax, overflow);
    }
    if (MODE != MODE_DECOMPRESS && late) S.late = 1u;
    if (MODE == MODE_DECOMPRESS) {
        // a frame found corrupt only now has been written already: k_decode_finish clears it again
        if (late) S.ovf = 1u;                                           // (cleared before the first barrier; otherwise unused here)
        __syncthreads();
        const uint32_t any_late = S.ovf;
        if (tid == 0) verdict[blockIdx.x] = (V.status ? V.status : (any_late ? (uint32_t)ST_CORRUPT : (uint32_t)ST_OK)) | (found_kind << 8);
        return;
    }

    // worst status so far: the stream headers', the frame's, this workgroup's segments', and what the passes before found (a_status)
    auto worst = [&]() -> uint32_t { return max(max(st_a, st_b), max(max(V.status, a_status), S.late ? (uint32_t)ST_CORRUPT : (uint32_t)ST_OK)); };
    if (MODE == MODE_STAGE_A) {
        __syncthreads();
        if (tid == 0) {
            for (uint32_t h = 0; h < NT * kSeg / kHalf; h++)
                if (blk0 + h * kHalf < nf) awide[(size_t)frame * hpf + blk0 / kHalf + h] = S.cwide[h] | (worst() << 8);
            if (db == 0) akind[frame] = (V.kind == KIND_RAW) ? 1u : 0u;
        }
        return;
    }
    // ---- adding passes: statistics of the sum, per half ----
    // (a sum beyond 2^30 turns the whole frame RAW, which only a later kernel can do once every workgroup of the frame is
    // done; the flag travels with the half's statistics)
    if (overflow) S.ovf = 1u;
#pragma unroll
    for (uint32_t h = 0; h < 2; h++) {
        const uint32_t zm = wave_max(zmax[h]);
        if (lane == 0 && zm) atomicMax(&S.zmax[h], zm);
    }
    __syncthreads();
    const bool out_raw = X.a_raw || X.b_raw;                            // uniform over the frame
    if (MODE == MODE_ACC) {
        // the running value's flags, in the set just written; the range flag goes where k_fix_acc looks for it
        if (tid == 0) {
            for (uint32_t h = 0; h < NT * kSeg / kHalf; h++) {
                if (blk0 + h * kHalf >= nf) break;
                const size_t hb = (size_t)frame * hpf + blk0 / kHalf + h;
                awide_out[hb] = (S.cwide[h] ? 1u : 0u) | (worst() << 8);
                reinterpret_cast<uint2*>(A.ws + A.L.pmeta)[hb] = make_uint2(0u, out_raw ? 1u : 0u);
                reinterpret_cast<uint32_t*>(A.ws + A.L.cwide)[hb] = S.ovf ? 2u : 0u;
            }
            if (db == 0) akind_out[frame] = out_raw ? 1u : 0u;
        }
        return;
    }
    for (uint32_t h = 0; h < NT * kSeg / kHalf; h++) {
        if (blk0 + h * kHalf >= nf) break;
        const size_t hb = (size_t)frame * hpf + blk0 / kHalf + h;
        uint32_t* ph = reinterpret_cast<uint32_t*>(A.ws + A.L.phist) + hb * kMaxK;
        if (NZ_STATS(MODE)) for (uint32_t sy = tid; sy < A.K; sy += NT) {
            uint32_t t = 0;
            for (uint32_t cc = 0; cc < (1u << X.ncs); cc++) t += s_h[h * 1024u + (sy << X.ncs) + cc];
            ph[bin_symbol(sy, A.K)] = t;
        }
        if (tid == 0) {
            // flag word: bit 0 = an operand frame is RAW, bit 1 = the local data of this half cannot be quantized
            reinterpret_cast<uint2*>(A.ws + A.L.pmeta)[hb] = make_uint2(S.zmax[h], (out_raw ? 1u : 0u) | (S.lunq[h] ? 2u : 0u));
            // bit 0 = the half holds sums that need 32 bits, bit 1 = a sum of this workgroup is out of range, from bit 8 on the worst status
            reinterpret_cast<uint32_t*>(A.ws + A.L.cwide)[hb] = (S.cwide[h] ? 1u : 0u) | (S.ovf ? 2u : 0u) | (worst() << 8);
        }
    }
}

// Threads of a decompressing or staging workgroup.  Two workgroups of 512 fit a compute unit, or three of 256: four wavefronts a
// SIMD hold what three would not, but a round of them is longer, the more so the more the decoder has to do for a symbol.  512 where
// that makes one round of two, or two of three: there, unless the stream has four to twelve bits a symbol.  With fewer the codes
// are short, from twelve on frames are FIXEDLEN for the most part, and those lose most by 256.  What the host knows of it is the size of
// the buffer that holds the stream; one for the worst case says nothing, and the stream in it takes 512.
// us with 256 / 512 threads: one round, 224 MB at 3.8 bits a symbol 92 / 69, at ten 143 / 120, 256 MB at 3.7 96 / 74, at 4.9 98 / 94, at 6.6 132 / 133, at
// ten 147 / 161 (the one place where the line is older than the decoder), FIXEDLEN at 14 77 / 64; two rounds, 448 MB at 3.7 bits 140 / 123, at 4.9 145 / 144, at ten 230 / 250, 512 MB at 3.7 146 / 134, at 4.9 150 / 172,
// at 6.6 207 / 250, of a field at 7.8 233 / 252, FIXEDLEN at 14 124 / 120; no round saved, 192 MB 62 / 66, 384 MB
// 114 / 137, 768 MB at 4.9 211 / 250; sums of two messages of 256 MB 269 / 269, at ten bits 397 / 406, of 512 MB at 4.9 bits 495 / 512, at ten 721 / 785.
static uint32_t dec_threads(const DecodeArgs& A) {
    const uint64_t blocks = (A.n + A.chunk - 1) / A.chunk * ((A.chunk + kDecBlock - 1) / kDecBlock);
    constexpr uint64_t kSmall = resident(kDecThreads) * kComputeUnits, kLarge = 2u * resident(2 * kDecThreads) * kComputeUnits;    // blocks of 65536 a round
    const uint64_t small = (blocks + kSmall - 1) / kSmall, large = (blocks + kLarge - 1) / kLarge;
    if (A.chunk <= kDecBlock || large >= small) return kDecThreads;
    const bool long_codes = 2u * A.a_bytes >= A.n && 2u * A.a_bytes < 3u * A.n;
    return large == 1 || (large == 2 && !long_codes) ? 2u * kDecThreads : kDecThreads;
}

// How many workgroups share a compute unit's 160 KB is part of the rules for their width.  It is given out in pieces of 1280 bytes: with a 44th
// second-level table (53920 bytes) two decompressing workgroups of 256 threads fitted where three do now (a 512 MB field at 4.3 bits a symbol 155 / 143 us).
constexpr uint32_t kLds = 160u << 10, kLdsPiece = 1280;
constexpr uint32_t lds_pieces(uint32_t bytes) { return (bytes + kLdsPiece - 1) / kLdsPiece * kLdsPiece; }
template <int MODE, int NT, int WIDE>
constexpr uint32_t lds_of() { return lds_pieces(sizeof(ModeTables<MODE, NT, WIDE>) + sizeof(ModeShared<MODE, NT, WIDE>) + (NZ_STATS(MODE) ? 16u * NT : 16u)); }
template <int WIDE>
constexpr bool shapes_fit() {
    return kLds / lds_of<MODE_DECOMPRESS, kDecThreads, WIDE>() == resident(kDecThreads) && kLds / lds_of<MODE_DECOMPRESS, 2 * kDecThreads, WIDE>() == resident(2 * kDecThreads) &&
           kLds / lds_of<MODE_ADD_B, kAddThreads, WIDE>() == kAddResident && kLds / lds_of<MODE_ADD_B, kAddThreadsSmall, WIDE>() == kAddResidentSmall;
}
static_assert(shapes_fit<0>() && shapes_fit<1>(), "see resident and add_pass_threads");

template <int MODE, int NT, int FORM>
static void launch_blocks(DecodeArgs& D, hipStream_t st) {
    D.dbpf = (D.chunk + NT * kSeg - 1) / (NT * kSeg);
    hipLaunchKernelGGL((k_decode<MODE, NT, FORM>), dim3(D.n_frames * D.dbpf), dim3(NT), 0, st, D);
}

template <int MODE, int FORM>
static void launch_add(DecodeArgs& D, hipStream_t st) {
    // (The passes without statistics are built with 512 threads only.  256 would gain a little on messages that leave compute units idle: sampled
    // ring step on 4 MB 74 / 70 us, on 64 MB 109 / 105, on 128 MB 150 / 147.)
    if constexpr (NZ_STATS(MODE)) {
        if (add_pass_threads(D.n, D.chunk) == kAddThreadsSmall) { launch_blocks<MODE, kAddThreadsSmall, FORM>(D, st); return; }
    }
    launch_blocks<MODE, kAddThreads, FORM>(D, st);
}

template <int FORM>
static void launch_decode_t(DecodeArgs& D, int pass, hipStream_t st) {
    const bool small = dec_threads(D) == kDecThreads;
    if (pass == 0 && small) launch_blocks<MODE_DECOMPRESS, kDecThreads, FORM>(D, st);
    else if (pass == 0) launch_blocks<MODE_DECOMPRESS, 2 * kDecThreads, FORM>(D, st);
    else if (pass == 1 && small) launch_blocks<MODE_STAGE_A, kDecThreads, FORM>(D, st);
    else if (pass == 1) launch_blocks<MODE_STAGE_A, 2 * kDecThreads, FORM>(D, st);
    else if (pass == 2) launch_add<MODE_ADD_B, FORM>(D, st);
    else if (pass == 3) launch_add<MODE_ADD_LOCAL, FORM>(D, st);
    else if (pass == 6) launch_add<MODE_ACC, FORM>(D, st);
    else if constexpr (!(FORM & 1)) {            // (the stochastic and the sampled ring step are not built with the predictor)
        if (pass == 4) launch_add<MODE_ADD_LOCAL_SR, FORM>(D, st); else launch_add<MODE_ADD_LOCAL_PLAIN, FORM>(D, st);
    }
}

}  // namespace nz
