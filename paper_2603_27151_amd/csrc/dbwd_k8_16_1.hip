// Backward fragment decode instantiated for the MLP shape (8, 16, 1).
#include "decode_bwd_impl.hpp"

namespace soup {

void launch_decode_bwd_k8_16_1(const DecodeArgs& a, hipStream_t s) {
    launch_decode_bwd_s<MlpShape<8, 16, 1>>(a, s);
}

size_t decode_bwd_lds_k8_16_1(int G) { return decode_bwd_lds_s<MlpShape<8, 16, 1>>(G); }

}  // namespace soup
