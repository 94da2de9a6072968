// fused_int.hip -- the fused kernel for batches without string atoms (the smallest
// instantiation, no spills), and the launch of the instantiation a batch
// needs.
#include "fused.h"

namespace dpf {

size_t fused_wave_area_bytes(bool str, bool pend) { return wave_area_bytes(str, pend); }

hipError_t launch_fused(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s) {
    if (waves != 4 && waves != 8 && waves != 16) return hipErrorInvalidValue;
    return a.str_stage == 2 ? launch_fused_fsst(a, waves, grid, lds_bytes, s)
           : a.str_stage    ? launch_fused_str(a, waves, grid, lds_bytes, s)
                            : launch_fused_mode<0>(a, waves, grid, lds_bytes, s);
}

}  // namespace dpf
