#include "wave_bwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken
// (backward with its gradients):
// 1 tile: 4,1 456/674, *2,1 417/690; 2: 2,2 898/1308, 4,2 764/1237, *2,1 777/1256; 3: 4,3 2112/2905,
// 4,1 2917/3366, *2,1 1241/1750; 4: 2,2 2283/3266, 4,4 4152/5456, 4,2 1801/2779, *2,1 1760/2505.
WaveKernel bwd_kernel_bf16_h64(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<64, 1, bf16_t, 2, 1>();
        case 2: return bwd_kernel<64, 2, bf16_t, 2, 1>();
        case 3: return bwd_kernel<64, 3, bf16_t, 2, 1>();
        case 4: return bwd_kernel<64, 4, bf16_t, 2, 1>();
        default: return {};
    }
}

}  // namespace mdl
