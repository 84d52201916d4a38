#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 2 tiles: 1,1 414/411, *1,2 284/382; 3: 1,1 642/628, *1,3 341/567;
// 4: 1,1 921/893, 1,2 596/813, *1,4 414/772.
WaveKernel fwd_kernel_f32_h4(int nt, int ck, bool one_step) {
    switch (nt) {
        case 1: return fwd_kernel<4, 1, float, 1, 1>(ck, one_step);
        case 2: return fwd_kernel<4, 2, float, 1, 2>(ck, one_step);
        case 3: return fwd_kernel<4, 3, float, 1, 3>(ck, one_step);
        case 4: return fwd_kernel<4, 4, float, 1, 4>(ck, one_step);
        default: return {};
    }
}

}  // namespace mdl
