// fused_str.hip -- the fused kernel for batches with string atoms on VARLEN columns.
// Only they carry the string stage's code and registers (its segment buffers
// and record queue).
#include "fused.h"

namespace dpf {

hipError_t launch_fused_str(const BatchArgs& a, int waves, int grid, size_t lds_bytes, hipStream_t s) {
    return launch_fused_mode<1>(a, waves, grid, lds_bytes, s);
}

}  // namespace dpf
