#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 1 tile: 1,1 199/188, *2,1 199/170, 4,1 264/222; 2: 2,1 346/311, *2,2 296/305, 4,2 358/310;
// 3: 2,1 506/485, *2,3 389/445, 4,3 497/487; 4: 2,1 692/697, 2,2 589/655, *2,4 519/626, 4,4 542/618.
WaveKernel fwd_kernel_bf16_h32(int nt, int ck, bool one_step) {
    switch (nt) {
        case 1: return fwd_kernel<32, 1, bf16_t, 2, 1>(ck, one_step);
        case 2: return fwd_kernel<32, 2, bf16_t, 2, 2>(ck, one_step);
        case 3: return fwd_kernel<32, 3, bf16_t, 2, 3>(ck, one_step);
        case 4: return fwd_kernel<32, 4, bf16_t, 2, 4>(ck, one_step);
        default: return {};
    }
}

}  // namespace mdl
