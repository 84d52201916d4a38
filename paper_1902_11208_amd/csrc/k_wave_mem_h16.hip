#include "wave_bwd.hpp"
#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 1 tile: 2,1 413/287, *1,1 297/224; 2: 1,1 622/440, *1,2 420/447, 2,2 525/398; 3: 1,1 936/881,
// *1,3 556/667, 2,3 689/732, 2,1 1411/1304; 4: 1,4 1212/1504, 1,1 1263/1285, 2,2 1076/1102, *1,2 840/992.
WaveKernel fwd_kernel_mem_h16(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<16, 1, float, 1, 1, true>(ck);
        case 2: return fwd_kernel<16, 2, float, 1, 2, true>(ck);
        case 3: return fwd_kernel<16, 3, float, 1, 3, true>(ck);
        case 4: return fwd_kernel<16, 4, float, 1, 2, true>(ck);
        default: return {};
    }
}

// Backward with its gradients: 2,1 667/1218, 1318/2492, 1969/3737, 2682/5117;
// *1,1 573/1177, 1046/2270, 1568/3466, 2134/4697.
WaveKernel bwd_kernel_mem_h16(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<16, 1, float, 1, 1, true>();
        case 2: return bwd_kernel<16, 2, float, 1, 1, true>();
        case 3: return bwd_kernel<16, 3, float, 1, 1, true>();
        case 4: return bwd_kernel<16, 4, float, 1, 1, true>();
        default: return {};
    }
}

}  // namespace mdl
