// nz_decode.hip -- gfx950 kernels of the receiver side beside the decoder itself (nz_decode.hpp): frames that leave the integer domain, and
// the verdict on a decompressed stream.
#include "nz_decode.hpp"

namespace nz {

// The sampled ring step, and an exact one whose output lies on an operand: frames that turn RAW late (fix_elements), one workgroup per half, which looks
// at the frame's flags and returns at once otherwise.  (Otherwise the exact reduces' encoder makes them: enc_raw_sums.)
__global__ __launch_bounds__(256) void k_fix(DecodeArgs A) {
    const uint32_t hpf = (A.chunk + kHalf - 1) / kHalf;
    const uint32_t frame = blockIdx.x / hpf, h = blockIdx.x % hpf;
    const uint64_t f0 = (uint64_t)frame * A.chunk;
    const uint32_t nf = (uint32_t)((A.n - f0 < A.chunk) ? (A.n - f0) : A.chunk);
    const uint32_t h0 = h * kHalf;
    if (h0 >= nf) return;
    const uint32_t cnt = (nf - h0 < kHalf) ? (nf - h0) : kHalf;
    const uint2* pm = reinterpret_cast<const uint2*>(A.ws + A.L.pmeta) + (size_t)frame * hpf;
    const uint32_t* cw = reinterpret_cast<const uint32_t*>(A.ws + A.L.cwide) + (size_t)frame * hpf;
    uint32_t flags = 0;
    for (uint32_t j = 0; j < hpf && j * kHalf < nf; j++) flags |= (pm[j].y & (FLAG_RAW | FLAG_UNQUANTIZABLE)) | ((cw[j] & 2u) ? (uint32_t)FLAG_RANGE : 0u);
    if (!needs_fix(flags)) return;
    const FixArgs F = { A.a, A.local, A.sr, A.seed, A.eb, A.step, A.inv_step, A.ws };
    fix_elements(F, A.L, frame, f0, nf, h0, cnt, flags, 256u);
}

// After an accumulating pass of the k-ary reduce: a frame in which a partial sum passed 2^30 in magnitude leaves the
// integer domain at this operand.  Its running value becomes fp32 -- fl(fl(v*step) + fl(q*step)) with v the running
// code before this operand (still in the set the pass read) and q the operand's code, recovered as the staged sum
// minus v -- and the frame counts as RAW for the operands that follow.  One workgroup per half; rare.
__global__ __launch_bounds__(256) void k_fix_acc(DecodeArgs A) {
    const uint32_t tid = threadIdx.x;
    const uint32_t hpf = (A.chunk + kHalf - 1) / kHalf;
    const uint32_t frame = blockIdx.x / hpf, h = blockIdx.x % hpf;
    const uint64_t f0 = (uint64_t)frame * A.chunk;
    const uint32_t nf = (uint32_t)((A.n - f0 < A.chunk) ? (A.n - f0) : A.chunk);
    const uint32_t h0 = h * kHalf;
    if (h0 >= nf) return;
    const uint32_t cnt = (nf - h0 < kHalf) ? (nf - h0) : kHalf;
    const uint2* pm = reinterpret_cast<const uint2*>(A.ws + A.L.pmeta) + (size_t)frame * hpf;
    const uint32_t* cw = reinterpret_cast<const uint32_t*>(A.ws + A.L.cwide) + (size_t)frame * hpf;
    uint32_t ovf = 0, raw = 0;
    for (uint32_t j = 0; j < hpf && j * kHalf < nf; j++) { raw |= pm[j].y & 1u; ovf |= cw[j] & 2u; }
    if (raw || !ovf) return;                  // (a frame that was fp32 already has no integer sums to go out of range)
    const uint32_t si = A.set_in & 1u;
    StageA sa, so;
    sa.a16 = reinterpret_cast<int16_t*>(A.ws + (si ? A.L.c16 : A.L.a16)); sa.a32 = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.codes : A.L.a32));
    so.a16 = reinterpret_cast<int16_t*>(A.ws + (si ? A.L.a16 : A.L.c16)); so.a32 = reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.a32 : A.L.codes));
    uint32_t dummy = 0;
    for (uint32_t i = tid; i < cnt; i += 256) {
        const uint32_t ta = sa.get(f0, nf, h0 + i, false);
        const uint32_t tb = so.get(f0, nf, h0 + i, false) - ta;
        so.a32[f0 + h0 + i] = combine<true>(ta, false, tb, false, A.step, dummy);
    }
    if (h == 0 && tid == 0) reinterpret_cast<uint32_t*>(A.ws + (si ? A.L.akind : A.L.akind1))[frame] = 1u;
}

hipError_t launch_fix_acc(const DecodeArgs& A, hipStream_t st) {
    const uint32_t hpf = (A.chunk + kHalf - 1) / kHalf;
    hipLaunchKernelGGL(k_fix_acc, dim3(A.n_frames * hpf), dim3(256), 0, st, A);
    return hipGetLastError();
}

hipError_t launch_fix(const DecodeArgs& A, hipStream_t st) {
    const uint32_t hpf = (A.chunk + kHalf - 1) / kHalf;
    hipLaunchKernelGGL(k_fix, dim3(A.n_frames * hpf), dim3(256), 0, st, A);
    return hipGetLastError();
}

// Decompress, second kernel: sums the workgroups' verdicts up into the result record (plain stores: the record needs
// no clearing beforehand) and zero-fills every rejected frame -- the ones rejected at the header decode to zeros
// anyway, the ones found corrupt while decoding (a segment that did not use exactly its recorded bits) were written
// before the verdict was known.  A rejected frame never hands untrusted bytes to the caller (the paper's receiver
// copies rawBytes from an invalid frame, Algorithm 2; this format reports the frame and fills it with zeros).
__global__ __launch_bounds__(256) void k_decode_finish(DecodeArgs A) {
    __shared__ uint32_t s_status, s_cnt[3];
    const uint32_t tid = threadIdx.x;
    const uint32_t* verdict = reinterpret_cast<const uint32_t*>(A.ws + A.L.pmeta);
    uint64_t total = 0;
    const uint32_t st_a = check_stream(A.a, A.a_bytes, A, total);
    auto frame_verdict = [&](uint32_t frame, uint32_t& kind) -> uint32_t {
        const uint64_t f0 = (uint64_t)frame * A.chunk;
        const uint32_t nf = (uint32_t)((A.n - f0 < A.chunk) ? (A.n - f0) : A.chunk);
        uint32_t st = 0;
        for (uint32_t db = 0; db < A.dbpf && db * A.dblk < nf; db++) {
            const uint32_t v = verdict[(size_t)frame * A.dbpf + db];
            st = (v & 0xFFu) > st ? (v & 0xFFu) : st;
            if (db == 0) kind = v >> 8;
        }
        return st;
    };
    if (st_a == ST_OK) {
        for (uint32_t frame = blockIdx.x; frame < A.n_frames; frame += gridDim.x) {
            uint32_t kind;
            if (frame_verdict(frame, kind) == ST_OK) continue;
            const uint64_t f0 = (uint64_t)frame * A.chunk;
            const uint32_t nf = (uint32_t)((A.n - f0 < A.chunk) ? (A.n - f0) : A.chunk);
            for (uint32_t i = tid; i < nf; i += 256) A.out[f0 + i] = 0.0f;
        }
    }
    if (blockIdx.x != 0) return;
    if (tid == 0) { s_status = st_a; s_cnt[0] = 0; s_cnt[1] = 0; s_cnt[2] = 0; }
    __syncthreads();
    if (st_a == ST_OK) {
        uint32_t worst = 0, c[3] = { 0, 0, 0 };
        for (uint32_t frame = tid; frame < A.n_frames; frame += 256) {
            uint32_t kind = KIND_ZERO;
            const uint32_t st = frame_verdict(frame, kind);
            worst = st > worst ? st : worst;
            if (st == ST_OK && kind < 3u) c[kind]++;
        }
        if (worst) atomicMax(&s_status, worst);
        for (int k = 0; k < 3; k++) if (c[k]) atomicAdd(&s_cnt[k], c[k]);
    }
    __syncthreads();
    if (tid == 0) {
        ResultRec* res = reinterpret_cast<ResultRec*>(A.res);
        res->bytes = (st_a == ST_OK) ? total : 0ull;
        res->status = s_status; res->n_frames = A.n_frames;
        res->n_raw = s_cnt[KIND_RAW]; res->n_fixed = s_cnt[KIND_FIXED]; res->n_huff = s_cnt[KIND_HUFF]; res->reserved = 0;
    }
}

hipError_t launch_decode_finish(const DecodeArgs& A, hipStream_t st) {
    DecodeArgs D = A;
    D.dblk = dec_threads(A) * kSeg;
    D.dbpf = (A.chunk + D.dblk - 1) / D.dblk;
    const uint32_t grid = A.n_frames < 1024u ? A.n_frames : 1024u;
    hipLaunchKernelGGL(k_decode_finish, dim3(grid), dim3(256), 0, st, D);
    return hipGetLastError();
}

hipError_t launch_decode(const DecodeArgs& A, int pass, hipStream_t st) {
    if (A.K > kPairAlphabet) return launch_decode_wide(A, pass, st);
    DecodeArgs D = A;
    if (A.pred) launch_decode_t<1>(D, pass, st); else launch_decode_t<0>(D, pass, st);
    return hipGetLastError();
}

}  // namespace nz
