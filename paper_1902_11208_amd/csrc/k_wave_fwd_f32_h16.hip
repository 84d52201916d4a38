#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 2 tiles: 1,1 410/360, *1,2 316/356, 2,2 366/329, 2,1 551/398; 3: 1,1 610/658, *1,3 410/538,
// 2,3 462/549, 2,1 845/817; 4: 1,1 810/920, 1,2 600/867, 1,4 648/935, *2,4 513/749.
WaveKernel fwd_kernel_f32_h16(int nt, int ck, bool one_step) {
    switch (nt) {
        case 1: return fwd_kernel<16, 1, float, 1, 1>(ck, one_step);
        case 2: return fwd_kernel<16, 2, float, 1, 2>(ck, one_step);
        case 3: return fwd_kernel<16, 3, float, 1, 3>(ck, one_step);
        case 4: return fwd_kernel<16, 4, float, 2, 4>(ck, one_step);
        default: return {};
    }
}

}  // namespace mdl
