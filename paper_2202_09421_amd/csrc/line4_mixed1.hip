// Line passes of both directions in one launch, FP32 plans.
#include "line4_mixed.h"

namespace rte {

hipError_t lines4_mixed(const Lines4Args<float>& a, int nq, bool adj, hipStream_t s) { return mixed(a, nq, adj, s); }

}  // namespace rte
