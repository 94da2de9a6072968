// fused_fsst.hip -- the fused kernel for batches with a string atom on an FSST column
// (VARLEN atoms still run): only they carry the FSST walk.
#include "fused.h"

namespace dpf {

hipError_t launch_fused_fsst(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s) {
    return launch_fused_mode<2>(a, waves, grid, lds_bytes, s);
}

}  // namespace dpf
