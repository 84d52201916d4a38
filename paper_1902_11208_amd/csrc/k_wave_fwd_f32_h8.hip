#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 2 tiles: 1,1 381/430, *1,2 262/398, 2,2 340/414; 3: 1,1 566/638, *1,3 322/563, 2,3 381/602;
// 4: 1,1 766/903, 1,2 508/792, *1,4 353/769, 2,4 432/758.
WaveKernel fwd_kernel_f32_h8(int nt, int ck, bool one_step) {
    switch (nt) {
        case 1: return fwd_kernel<8, 1, float, 1, 1>(ck, one_step);
        case 2: return fwd_kernel<8, 2, float, 1, 2>(ck, one_step);
        case 3: return fwd_kernel<8, 3, float, 1, 3>(ck, one_step);
        case 4: return fwd_kernel<8, 4, float, 1, 4>(ck, one_step);
        default: return {};
    }
}

}  // namespace mdl
