// Line passes for extended lengths 625, 640, 648, 675, 720, 729, 750, 768,
// 800, 810, 864.
#include "line4_impl.h"

namespace rte {

template <typename T>
static hipError_t longs(const Lines4Args<T>& a, int Np, int nq, bool adj, hipStream_t s) {
  switch (Np) {
    case 625: return adj ? go_one<T, true, 25, 25>(a, nq, s) : go_one<T, false, 25, 25>(a, nq, s);
    case 640: return adj ? go_one<T, true, 10, 64>(a, nq, s) : go_one<T, false, 10, 64>(a, nq, s);
    case 648: return adj ? go_one<T, true, 12, 54>(a, nq, s) : go_one<T, false, 12, 54>(a, nq, s);
    case 675: return adj ? go_one<T, true, 15, 45>(a, nq, s) : go_one<T, false, 15, 45>(a, nq, s);
    case 720: return adj ? go_one<T, true, 5, 144>(a, nq, s) : go_one<T, false, 5, 144>(a, nq, s);
    case 729: return adj ? go_one<T, true, 27, 27>(a, nq, s) : go_one<T, false, 27, 27>(a, nq, s);
    case 750: return adj ? go_one<T, true, 10, 75>(a, nq, s) : go_one<T, false, 10, 75>(a, nq, s);
    case 768: return adj ? go_one<T, true, 12, 64>(a, nq, s) : go_one<T, false, 12, 64>(a, nq, s);
    case 800: return adj ? go_one<T, true, 32, 25>(a, nq, s) : go_one<T, false, 32, 25>(a, nq, s);
    case 810: return adj ? go_one<T, true, 18, 45>(a, nq, s) : go_one<T, false, 18, 45>(a, nq, s);
    case 864: return adj ? go_one<T, true, 6, 144>(a, nq, s) : go_one<T, false, 6, 144>(a, nq, s);
    default: return hipErrorNotSupported;
  }
}

hipError_t lines4_long0(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s) { return longs(a, Np, nq, adj, s); }
hipError_t lines4_long0(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s) { return longs(a, Np, nq, adj, s); }

}  // namespace rte
