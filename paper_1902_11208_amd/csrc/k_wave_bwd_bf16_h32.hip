#include "wave_bwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken
// (backward with its gradients):
// 1 tile: 1,1 342/669, *2,1 334/648, 4,1 416/645; 2: 2,1 590/1304, *2,2 566/1282, 4,2 627/1301,
// 4,1 782/1345; 3: 2,1 880/1980, *2,3 793/1972, 4,3 886/1980; 4: *2,2 1070/2597, 2,4 1120/2559,
// 2,1 1179/2601, 4,2 1275/2696.
WaveKernel bwd_kernel_bf16_h32(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<32, 1, bf16_t, 2, 1>();
        case 2: return bwd_kernel<32, 2, bf16_t, 2, 2>();
        case 3: return bwd_kernel<32, 3, bf16_t, 2, 3>();
        case 4: return bwd_kernel<32, 4, bf16_t, 2, 2>();
        default: return {};
    }
}

}  // namespace mdl
