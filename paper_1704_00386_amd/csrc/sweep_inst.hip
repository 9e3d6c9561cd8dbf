// sweep_inst.hip -- the sweep kernels of one k and one type of tau, the
// one-graph ones and (16 and 32 bits) the batches'; built once per pair, with
// ND_SWEEP_K, ND_SWEEP_T and ND_SWEEP_BATCH set on the command line, so that
// the pairs compile side by side.
#include "batch_kernels.h"

namespace nd {

template void sweep_kind<ND_SWEEP_K, ND_SWEEP_T>(const KindState &,
                                                 const SweepArgs &, bool,
                                                 hipStream_t);
#if ND_SWEEP_BATCH
template const void *batch_kernel<ND_SWEEP_K, ND_SWEEP_T>(bool, bool);
#endif

}  // namespace nd
