#include "wave_fwd.hpp"

namespace mdl {

WaveKernel fwd_kernel_bf16_h64(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<64, 1, bf16_t, 2, 1>(ck);
        case 2: return fwd_kernel<64, 2, bf16_t, 4, 2>(ck);
        case 3: return fwd_kernel<64, 3, bf16_t, 2, 1>(ck);
        case 4: return fwd_kernel<64, 4, bf16_t, 2, 1>(ck);
        default: return {};
    }
}

}  // namespace mdl
