#include "wave_bwd.hpp"

namespace mdl {

WaveKernel bwd_kernel_bf16_h32(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<32, 1, bf16_t, 2, 1>();
        case 2: return bwd_kernel<32, 2, bf16_t, 2, 2>();
        case 3: return bwd_kernel<32, 3, bf16_t, 2, 1>();
        case 4: return bwd_kernel<32, 4, bf16_t, 2, 2>();
        default: return {};
    }
}

}  // namespace mdl
