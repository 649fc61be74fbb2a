// Line passes for extended lengths 900, 960, 972, 1000, 1024, 1080, 1152, 1200,
// 1125.
#include "line4_impl.h"

namespace rte {

template <typename T>
static hipError_t longs(const Lines4Args<T>& a, int Np, int nq, bool adj, hipStream_t s) {
  switch (Np) {
    case 900: return adj ? go_one<T, true, 4, 225>(a, nq, s) : go_one<T, false, 4, 225>(a, nq, s);
    case 960: return adj ? go_one<T, true, 15, 64>(a, nq, s) : go_one<T, false, 15, 64>(a, nq, s);
    case 972: return adj ? go_one<T, true, 18, 54>(a, nq, s) : go_one<T, false, 18, 54>(a, nq, s);
    case 1000: return adj ? go_one<T, true, 10, 100>(a, nq, s) : go_one<T, false, 10, 100>(a, nq, s);
    case 1024: return adj ? go_one<T, true, 16, 64>(a, nq, s) : go_one<T, false, 16, 64>(a, nq, s);
    case 1080: return adj ? go_one<T, true, 10, 108>(a, nq, s) : go_one<T, false, 10, 108>(a, nq, s);
    case 1152: return adj ? go_one<T, true, 18, 64>(a, nq, s) : go_one<T, false, 18, 64>(a, nq, s);
    case 1200: return adj ? go_one<T, true, 8, 150>(a, nq, s) : go_one<T, false, 8, 150>(a, nq, s);
    case 1125: return adj ? go_one<T, true, 15, 75>(a, nq, s) : go_one<T, false, 15, 75>(a, nq, s);
    default: return hipErrorNotSupported;
  }
}

hipError_t lines4_long1(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s) { return longs(a, Np, nq, adj, s); }
hipError_t lines4_long1(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s) { return longs(a, Np, nq, adj, s); }

}  // namespace rte
