// Backward fragment decode instantiated for the MLP shape (16, 32, 2).
#include "decode_bwd_impl.hpp"

namespace soup {

void launch_decode_bwd_k16_32_2(const DecodeArgs& a, hipStream_t s) {
    launch_decode_bwd_s<MlpShape<16, 32, 2>>(a, s);
}

size_t decode_bwd_lds_k16_32_2(int G) { return decode_bwd_lds_s<MlpShape<16, 32, 2>>(G); }

}  // namespace soup
