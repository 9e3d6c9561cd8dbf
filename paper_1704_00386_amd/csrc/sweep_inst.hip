// sweep_inst.hip -- the sweep kernels of one k and one type of tau; built
// once per pair, with ND_SWEEP_K and ND_SWEEP_T set on the command line, so
// that the pairs compile side by side.
#include "sweep_kernels.h"

namespace nd {

template void sweep_kind<ND_SWEEP_K, ND_SWEEP_T>(const KindState &,
                                                 const SweepArgs &, bool,
                                                 hipStream_t);

}  // namespace nd
