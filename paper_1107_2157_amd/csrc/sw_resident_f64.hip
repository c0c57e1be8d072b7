// The resident time loop's instances: FP64, paper's scheme (one file each: they build in parallel).
#include "sw_resident_kernel.h"

hipError_t sw_res_launch_f64(const SwResArgs &a, int rows, bool exact, int nw, int nwg, hipStream_t s) {
    return launch_rows<double, false>(a, rows, exact, nw, nwg, s);
}
