#include "wave_fwd.hpp"

namespace mdl {

WaveKernel fwd_kernel_bf16_h32(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<32, 1, bf16_t, 2, 1>(ck);
        case 2: return fwd_kernel<32, 2, bf16_t, 2, 2>(ck);
        case 3: return fwd_kernel<32, 3, bf16_t, 2, 3>(ck);
        case 4: return fwd_kernel<32, 4, bf16_t, 2, 4>(ck);
        default: return {};
    }
}

}  // namespace mdl
