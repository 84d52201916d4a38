#include "wave_bwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken
// (backward with its gradients):
// 2 tiles: 1,1 913/1976, *1,2 804/1954, 2,1 1042/2007, 2,2 890/1969; 3: 1,1 1326/2970,
// *1,3 1134/2903, 2,1 1604/3038, 2,3 1180/2951; 4: 1,1 1773/4031, 1,2 1542/3937, *1,4 1453/3861,
// 2,2 1682/3970.
WaveKernel bwd_kernel_f32_h8(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<8, 1, float, 1, 1>();
        case 2: return bwd_kernel<8, 2, float, 1, 2>();
        case 3: return bwd_kernel<8, 3, float, 1, 3>();
        case 4: return bwd_kernel<8, 4, float, 1, 4>();
        default: return {};
    }
}

}  // namespace mdl
