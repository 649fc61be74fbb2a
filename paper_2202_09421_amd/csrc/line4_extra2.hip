// Line passes for extended lengths 50, 75, 81, 150, 180, 256, 270, 375,
// 400, 480, 576.
#include "line4_impl.h"

namespace rte {

template <typename T>
static hipError_t extra(const Lines4Args<T>& a, int Np, int nq, bool adj, hipStream_t s) {
  switch (Np) {
    case 50: return adj ? go_one<T, true, 5, 10>(a, nq, s) : go_one<T, false, 5, 10>(a, nq, s);
    case 75: return adj ? go_one<T, true, 3, 25>(a, nq, s) : go_one<T, false, 3, 25>(a, nq, s);
    case 81: return adj ? go_one<T, true, 9, 9>(a, nq, s) : go_one<T, false, 9, 9>(a, nq, s);
    case 150: return adj ? go_one<T, true, 10, 15>(a, nq, s) : go_one<T, false, 10, 15>(a, nq, s);
    case 180: return adj ? go_one<T, true, 12, 15>(a, nq, s) : go_one<T, false, 12, 15>(a, nq, s);
    case 256: return adj ? go_one<T, true, 16, 16>(a, nq, s) : go_one<T, false, 16, 16>(a, nq, s);
    case 270: return adj ? go_one<T, true, 3, 90>(a, nq, s) : go_one<T, false, 3, 90>(a, nq, s);
    case 375: return adj ? go_one<T, true, 15, 25>(a, nq, s) : go_one<T, false, 15, 25>(a, nq, s);
    case 400: return adj ? go_one<T, true, 8, 50>(a, nq, s) : go_one<T, false, 8, 50>(a, nq, s);
    case 480: return adj ? go_one<T, true, 8, 60>(a, nq, s) : go_one<T, false, 8, 60>(a, nq, s);
    case 576: return adj ? go_one<T, true, 24, 24>(a, nq, s) : go_one<T, false, 24, 24>(a, nq, s);
    default: return hipErrorNotSupported;
  }
}

hipError_t lines4_extra2(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }
hipError_t lines4_extra2(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }

}  // namespace rte
