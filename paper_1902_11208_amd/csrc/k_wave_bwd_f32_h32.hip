#include "wave_bwd.hpp"

namespace mdl {

WaveKernel bwd_kernel_f32_h32(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<32, 1, float, 2, 1>();
        case 2: return bwd_kernel<32, 2, float, 2, 2>();
        case 3: return bwd_kernel<32, 3, float, 2, 1>();
        case 4: return bwd_kernel<32, 4, float, 2, 2>();
        default: return {};
    }
}

}  // namespace mdl
