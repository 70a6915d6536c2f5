// Resident run kernels of one precision: every tile edge, with and without
// McWeeny's two products. Single runs and batches have the same kernels, but
// for the short chains (48-tiles reach the launch sequence's errors without).
#include "run_impl.h"

namespace sp2 {

const void* run_kernel_f64(int mb, bool mw, RunKind kind) {
  switch (mb) {
    case 2:
      return kind == kRunBrief ? run_fn<RunCfg<0, 2, 4, false, true>>(mw)
                               : run_fn<RunCfg<0, 2, 4, false>>(mw);
    case 3: return run_fn<RunCfg<0, 3, 4, false>>(mw);
    case 4: return run_fn<RunCfg<0, 4, 4, false>>(mw);
    default: return nullptr;
  }
}

}  // namespace sp2
