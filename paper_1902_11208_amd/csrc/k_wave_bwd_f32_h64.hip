#include "wave_bwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken
// (backward with its gradients):
// 1 tile: 4,1 1434/2154, *2,1 1259/2087; 2: 2,1 3634/4985, 4,2 4673/6494, *4,1 2918/4412,
// 2,2 5927/7106; 3: 4,3 9831/13985, 4,1 6051/8560, *2,1 5579/7794; 4: 4,2 12193/16368,
// 4,4 14999/24905, 2,2 15112/19091, *2,1 9166/13126.
WaveKernel bwd_kernel_f32_h64(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<64, 1, float, 2, 1>();
        case 2: return bwd_kernel<64, 2, float, 4, 1>();
        case 3: return bwd_kernel<64, 3, float, 2, 1>();
        case 4: return bwd_kernel<64, 4, float, 2, 1>();
        default: return {};
    }
}

}  // namespace mdl
