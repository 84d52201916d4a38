#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 1 tile: 4,1 310/271, *2,1 297/290, 1,1 344/345; 2: 2,1 559/590, *4,2 524/548, 4,1 612/598,
// 2,2 904/925; 3: 4,3 2045/2321, 4,1 923/952, *2,1 849/937; 4: 4,2 1235/1322, 4,1 1326/1381,
// 2,2 1803/2147, *2,1 1250/1334.
WaveKernel fwd_kernel_bf16_h64(int nt, int ck, bool one_step) {
    switch (nt) {
        case 1: return fwd_kernel<64, 1, bf16_t, 2, 1>(ck, one_step);
        case 2: return fwd_kernel<64, 2, bf16_t, 4, 2>(ck, one_step);
        case 3: return fwd_kernel<64, 3, bf16_t, 2, 1>(ck, one_step);
        case 4: return fwd_kernel<64, 4, bf16_t, 2, 1>(ck, one_step);
        default: return {};
    }
}

}  // namespace mdl
