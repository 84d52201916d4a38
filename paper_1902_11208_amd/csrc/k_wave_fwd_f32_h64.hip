#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 1 tile: 2,1 1115/1275, *4,1 887/1032; 2: 4,2 4361/5446, 2,1 2705/3454, 2,2 6505/6947,
// *4,1 1870/2210; 3: 4,3 7966/9508, 2,1 3950/4740, *4,1 2705/3436; 4: 4,2 8551/10963,
// 2,1 6342/7988, 4,4 13885/20880, *4,1 3511/4697.
WaveKernel fwd_kernel_f32_h64(int nt, int ck, bool one_step) {
    switch (nt) {
        case 1: return fwd_kernel<64, 1, float, 4, 1>(ck, one_step);
        case 2: return fwd_kernel<64, 2, float, 4, 1>(ck, one_step);
        case 3: return fwd_kernel<64, 3, float, 4, 1>(ck, one_step);
        case 4: return fwd_kernel<64, 4, float, 4, 1>(ck, one_step);
        default: return {};
    }
}

}  // namespace mdl
