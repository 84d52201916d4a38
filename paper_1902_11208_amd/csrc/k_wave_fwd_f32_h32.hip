#include "wave_fwd.hpp"

namespace mdl {

WaveKernel fwd_kernel_f32_h32(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<32, 1, float, 2, 1>(ck);
        case 2: return fwd_kernel<32, 2, float, 2, 2>(ck);
        case 3: return fwd_kernel<32, 3, float, 2, 1>(ck);
        case 4: return fwd_kernel<32, 4, float, 2, 2>(ck);
        default: return {};
    }
}

}  // namespace mdl
