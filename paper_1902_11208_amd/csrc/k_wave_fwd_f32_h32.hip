#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 1 tile: 1,1 323/335, *2,1 333/300, 4,1 572/387; 2: 2,1 705/718, *2,2 511/618, 1,1 638/733,
// 4,2 727/736; 3: 1,1 1045/1170, *2,1 1080/1130, 2,3 1803/2381, 4,3 2047/3103;
// 4: 2,4 3863/4855, 1,1 1506/1695, 2,1 1563/1685, *2,2 1206/1451.
WaveKernel fwd_kernel_f32_h32(int nt, int ck, bool one_step) {
    switch (nt) {
        case 1: return fwd_kernel<32, 1, float, 2, 1>(ck, one_step);
        case 2: return fwd_kernel<32, 2, float, 2, 2>(ck, one_step);
        case 3: return fwd_kernel<32, 3, float, 2, 1>(ck, one_step);
        case 4: return fwd_kernel<32, 4, float, 2, 2>(ck, one_step);
        default: return {};
    }
}

}  // namespace mdl
