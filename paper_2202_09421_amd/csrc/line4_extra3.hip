// Line passes for extended lengths 54, 96, 100, 144, 216, 225, 250, 324,
// 432, 486, 500.
#include "line4_impl.h"

namespace rte {

template <typename T>
static hipError_t extra(const Lines4Args<T>& a, int Np, int nq, bool adj, hipStream_t s) {
  switch (Np) {
    case 54: return adj ? go_one<T, true, 6, 9>(a, nq, s) : go_one<T, false, 6, 9>(a, nq, s);
    case 96: return adj ? go_one<T, true, 3, 32>(a, nq, s) : go_one<T, false, 3, 32>(a, nq, s);
    case 100: return adj ? go_one<T, true, 4, 25>(a, nq, s) : go_one<T, false, 4, 25>(a, nq, s);
    case 144: return adj ? go_one<T, true, 12, 12>(a, nq, s) : go_one<T, false, 12, 12>(a, nq, s);
    case 216: return adj ? go_one<T, true, 8, 27>(a, nq, s) : go_one<T, false, 8, 27>(a, nq, s);
    case 225: return adj ? go_one<T, true, 15, 15>(a, nq, s) : go_one<T, false, 15, 15>(a, nq, s);
    case 250: return adj ? go_one<T, true, 10, 25>(a, nq, s) : go_one<T, false, 10, 25>(a, nq, s);
    case 324: return adj ? go_one<T, true, 6, 54>(a, nq, s) : go_one<T, false, 6, 54>(a, nq, s);
    case 432: return adj ? go_one<T, true, 8, 54>(a, nq, s) : go_one<T, false, 8, 54>(a, nq, s);
    case 486: return adj ? go_one<T, true, 9, 54>(a, nq, s) : go_one<T, false, 9, 54>(a, nq, s);
    case 500: return adj ? go_one<T, true, 10, 50>(a, nq, s) : go_one<T, false, 10, 50>(a, nq, s);
    default: return hipErrorNotSupported;
  }
}

hipError_t lines4_extra3(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }
hipError_t lines4_extra3(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }

}  // namespace rte
