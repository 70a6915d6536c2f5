// Resident run kernels of one precision: every tile edge, with and without
// McWeeny's two products. Single runs and batches have the same kernels.
#include "run_impl.h"

namespace sp2 {

const void* run_kernel_b3(int mb, bool mw, RunKind) {
  switch (mb) {
    case 2: return run_fn<RunCfg<2, 2, 4, false>>(mw);
    case 4: return run_fn<RunCfg<2, 4, 4, false>>(mw);
    default: return nullptr;
  }
}

}  // namespace sp2
