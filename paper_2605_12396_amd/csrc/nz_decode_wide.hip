// nz_decode_wide.hip -- the decoder for alphabets of more than kPairAlphabet symbols, whose codes take two bytes.  Kernels of their own, chosen by
// the alphabet at launch, so that neither kind pays for the other's second store, tables or code.
#include "nz_decode.hpp"

namespace nz {

hipError_t launch_decode_wide(const DecodeArgs& A, int pass, hipStream_t st) {
    DecodeArgs D = A;
    if (A.pred) launch_decode_t<3>(D, pass, st); else launch_decode_t<2>(D, pass, st);
    return hipGetLastError();
}

}  // namespace nz
