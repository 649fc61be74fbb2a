// Line passes for extended lengths 48, 64, 80, 108, 125, 128, 162, 240,
// 243, 320, 450, 512.
#include "line4_impl.h"

namespace rte {

template <typename T>
static hipError_t extra(const Lines4Args<T>& a, int Np, int nq, bool adj, hipStream_t s) {
  switch (Np) {
    case 48: return adj ? go_one<T, true, 3, 16>(a, nq, s) : go_one<T, false, 3, 16>(a, nq, s);
    case 64: return adj ? go_one<T, true, 4, 16>(a, nq, s) : go_one<T, false, 4, 16>(a, nq, s);
    case 80: return adj ? go_one<T, true, 8, 10>(a, nq, s) : go_one<T, false, 8, 10>(a, nq, s);
    case 108: return adj ? go_one<T, true, 9, 12>(a, nq, s) : go_one<T, false, 9, 12>(a, nq, s);
    case 125: return adj ? go_one<T, true, 5, 25>(a, nq, s) : go_one<T, false, 5, 25>(a, nq, s);
    case 128: return adj ? go_one<T, true, 4, 32>(a, nq, s) : go_one<T, false, 4, 32>(a, nq, s);
    case 162: return adj ? go_one<T, true, 3, 54>(a, nq, s) : go_one<T, false, 3, 54>(a, nq, s);
    case 240: return adj ? go_one<T, true, 16, 15>(a, nq, s) : go_one<T, false, 16, 15>(a, nq, s);
    case 243: return adj ? go_one<T, true, 3, 81>(a, nq, s) : go_one<T, false, 3, 81>(a, nq, s);
    case 320: return adj ? go_one<T, true, 5, 64>(a, nq, s) : go_one<T, false, 5, 64>(a, nq, s);
    case 450: return adj ? go_one<T, true, 5, 90>(a, nq, s) : go_one<T, false, 5, 90>(a, nq, s);
    case 512: return adj ? go_one<T, true, 8, 64>(a, nq, s) : go_one<T, false, 8, 64>(a, nq, s);
    default: return hipErrorNotSupported;
  }
}

hipError_t lines4_extra0(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }
hipError_t lines4_extra0(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }

}  // namespace rte
