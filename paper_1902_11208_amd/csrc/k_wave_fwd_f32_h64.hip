#include "wave_fwd.hpp"

namespace mdl {

WaveKernel fwd_kernel_f32_h64(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<64, 1, float, 4, 1>(ck);
        case 2: return fwd_kernel<64, 2, float, 4, 1>(ck);
        case 3: return fwd_kernel<64, 3, float, 4, 1>(ck);
        case 4: return fwd_kernel<64, 4, float, 4, 1>(ck);
        default: return {};
    }
}

}  // namespace mdl
