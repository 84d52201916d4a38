#include "wave_bwd.hpp"

namespace mdl {

WaveKernel bwd_kernel_f32_h64(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<64, 1, float, 2, 1>();
        case 2: return bwd_kernel<64, 2, float, 2, 1>();
        case 3: return bwd_kernel<64, 3, float, 2, 1>();
        case 4: return bwd_kernel<64, 4, float, 2, 1>();
        default: return {};
    }
}

}  // namespace mdl
