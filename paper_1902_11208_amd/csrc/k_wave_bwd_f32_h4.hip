#include "wave_bwd.hpp"

namespace mdl {

WaveKernel bwd_kernel_f32_h4(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<4, 1, float, 1, 1>();
        case 2: return bwd_kernel<4, 2, float, 1, 1>();
        case 3: return bwd_kernel<4, 3, float, 1, 1>();
        case 4: return bwd_kernel<4, 4, float, 1, 1>();
        default: return {};
    }
}

}  // namespace mdl
