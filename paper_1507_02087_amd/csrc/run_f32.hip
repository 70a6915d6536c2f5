// Resident run kernels of one precision: every tile edge, with and without
// McWeeny's two products, for small single runs (short chains), single runs
// and batches.
#include "run_impl.h"

namespace sp2 {

const void* run_kernel_f32(int mb, bool mw, RunKind kind) {
  const bool solo = (kind != kRunBatch);
  switch (mb) {
    case 2:
      return kind == kRunBrief ? run_fn<RunCfg<1, 2, 4, false, true>>(mw)
                               : run_fn<RunCfg<1, 2, 4, false>>(mw);
    case 3:
      return kind == kRunBrief ? run_fn<RunCfg<1, 3, 4, false, true>>(mw)
                               : run_fn<RunCfg<1, 3, 4, false>>(mw);
    case 4: return solo ? run_fn<RunCfg<1, 4, 4, true>>(mw) : run_fn<RunCfg<1, 4, 4, false>>(mw);
    case 5: return solo ? run_fn<RunCfg<1, 5, 4, true>>(mw) : nullptr;
    default: return nullptr;
  }
}

}  // namespace sp2
