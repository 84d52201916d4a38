#include "wave_bwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken
// (backward with its gradients):
// 1 tile: 1,1 500/767, *2,1 481/731, 4,1 695/823; 2: 2,1 954/1337, *2,2 891/1318, 1,1 1011/1456,
// 4,2 935/1360; 3: 2,1 1585/2149, *2,3 1288/2000, 1,1 1496/2206, 4,3 2126/3015; 4: 2,2 3010/3957,
// 2,1 3129/4138, 2,4 3449/4395, *4,4 2065/3047.
WaveKernel bwd_kernel_f32_h32(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<32, 1, float, 2, 1>();
        case 2: return bwd_kernel<32, 2, float, 2, 2>();
        case 3: return bwd_kernel<32, 3, float, 2, 3>();
        case 4: return bwd_kernel<32, 4, float, 4, 4>();
        default: return {};
    }
}

}  // namespace mdl
