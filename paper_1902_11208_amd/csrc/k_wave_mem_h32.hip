#include "wave_bwd.hpp"
#include "wave_fwd.hpp"

namespace mdl {

// (units per lane, tile groups) by tiles. Call times in us, 16 images of 100-300
// columns / 128 of 50-150, rows = 16 tiles, 32 channels; * the one taken:
// 1 tile: 2,1 683/508, *1,1 453/469; 2: 2,2 1032/1036, 2,1 1119/1026, *1,1 930/951; 3: 2,1 1775/1698,
// 2,3 3255/3864, *1,1 1477/1569; 4: 1,1 2690/4203, 1,2 5802/7046, 2,2 2603/3161, *2,1 2294/2639.
WaveKernel fwd_kernel_mem_h32(int nt, int ck) {
    switch (nt) {
        case 1: return fwd_kernel<32, 1, float, 1, 1, true>(ck);
        case 2: return fwd_kernel<32, 2, float, 1, 1, true>(ck);
        case 3: return fwd_kernel<32, 3, float, 1, 1, true>(ck);
        case 4: return fwd_kernel<32, 4, float, 2, 1, true>(ck);
        default: return {};
    }
}

// Backward with its gradients: 2,1 679/1098, 1399/2205, 2154/3487, 5785/7694;
// *1,1 608/1103, 1205/2199, 1851/3340, 5457/7537.
WaveKernel bwd_kernel_mem_h32(int nt) {
    switch (nt) {
        case 1: return bwd_kernel<32, 1, float, 1, 1, true>();
        case 2: return bwd_kernel<32, 2, float, 1, 1, true>();
        case 3: return bwd_kernel<32, 3, float, 1, 1, true>();
        case 4: return bwd_kernel<32, 4, float, 1, 1, true>();
        default: return {};
    }
}

}  // namespace mdl
