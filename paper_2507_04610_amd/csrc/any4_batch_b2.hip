// The 2-bit variants of the kernel for a few dozen rows of x (a translation unit per code width keeps the
// build parallel).
#include "any4_batch.h"

namespace any4 {

hipError_t launch_batch_bits2(const batch::Params& p, int mt, int blocks_m, bool f16, bool fine, hipStream_t stream) {
    return batch::launch_bits<2>(p, mt, blocks_m, f16, fine, stream);
}

}  // namespace any4
