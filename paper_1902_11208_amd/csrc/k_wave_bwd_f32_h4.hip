#include "wave_bwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken
// (backward with its gradients):
// 2 tiles: 1,1 889/1862, *1,2 785/1828; 3: 1,1 1290/2803, *1,3 1088/2743;
// 4: 1,1 1708/3729, 1,2 1512/3639, *1,4 1398/3611.
WaveKernel bwd_kernel_f32_h4(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<4, 1, float, 1, 1>();
        case 2: return bwd_kernel<4, 2, float, 1, 2>();
        case 3: return bwd_kernel<4, 3, float, 1, 3>();
        case 4: return bwd_kernel<4, 4, float, 1, 4>();
        default: return {};
    }
}

}  // namespace mdl
