#include "wave_fwd.hpp"

namespace mdl {

WaveKernel fwd_kernel_f32_h4(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<4, 1, float, 1, 1>(ck);
        case 2: return fwd_kernel<4, 2, float, 1, 2>(ck);
        case 3: return fwd_kernel<4, 3, float, 1, 3>(ck);
        case 4: return fwd_kernel<4, 4, float, 1, 4>(ck);
        default: return {};
    }
}

}  // namespace mdl
