#include "wave_bwd.hpp"

namespace mdl {

WaveKernel bwd_kernel_f32_h8(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<8, 1, float, 1, 1>();
        case 2: return bwd_kernel<8, 2, float, 1, 1>();
        case 3: return bwd_kernel<8, 3, float, 1, 1>();
        case 4: return bwd_kernel<8, 4, float, 1, 1>();
        default: return {};
    }
}

}  // namespace mdl
