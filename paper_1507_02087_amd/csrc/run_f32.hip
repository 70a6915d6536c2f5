// Resident run kernels of one precision: every tile edge, with and without
// McWeeny's two products.
#include "run_impl.h"

namespace sp2 {

const void* run_kernel_f32(int mb, bool mw) {
  switch (mb) {
    case 2: return run_fn<RunCfg<1, 2, 4>>(mw);
    case 3: return run_fn<RunCfg<1, 3, 4>>(mw);
    case 4: return run_fn<RunCfg<1, 4, 4>>(mw);
    case 5: return run_fn<RunCfg<1, 5, 4>>(mw);
    default: return nullptr;
  }
}

}  // namespace sp2
