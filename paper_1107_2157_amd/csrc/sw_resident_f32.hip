// The resident time loop's instances: FP32, paper's scheme (one file each: they build in parallel).
#include "sw_resident_kernel.h"

hipError_t sw_res_launch_f32(const SwResArgs &a, int rows, bool exact, int nw, int nwg, hipStream_t s) {
    return launch_rows<float, false>(a, rows, exact, nw, nwg, s);
}
