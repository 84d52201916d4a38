#include "wave_bwd.hpp"
#include "wave_fwd.hpp"

namespace mdl {

WaveKernel fwd_kernel_mem_h32(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<32, 1, float, 1, 1, true>(ck);
        case 2: return fwd_kernel<32, 2, float, 1, 1, true>(ck);
        case 3: return fwd_kernel<32, 3, float, 1, 1, true>(ck);
        case 4: return fwd_kernel<32, 4, float, 1, 1, true>(ck);
        default: return {};
    }
}

WaveKernel bwd_kernel_mem_h32(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<32, 1, float, 1, 1, true>();
        case 2: return bwd_kernel<32, 2, float, 1, 1, true>();
        case 3: return bwd_kernel<32, 3, float, 1, 1, true>();
        case 4: return bwd_kernel<32, 4, float, 1, 1, true>();
        default: return {};
    }
}

}  // namespace mdl
