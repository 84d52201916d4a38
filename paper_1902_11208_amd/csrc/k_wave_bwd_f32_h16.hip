#include "wave_bwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken
// (backward with its gradients):
// 2 tiles: 1,1 1024/2224, *1,2 971/2217, 2,1 1170/2337, 2,2 987/2256; 3: 1,1 1499/3416,
// 1,3 1453/3407, 2,1 1798/3573, *2,3 1390/3420; 4: 1,2 1963/4539, *1,4 1902/4535, 1,1 2058/4604,
// 2,2 1946/4496.
WaveKernel bwd_kernel_f32_h16(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<16, 1, float, 1, 1>();
        case 2: return bwd_kernel<16, 2, float, 1, 2>();
        case 3: return bwd_kernel<16, 3, float, 2, 3>();
        case 4: return bwd_kernel<16, 4, float, 1, 4>();
        default: return {};
    }
}

}  // namespace mdl
