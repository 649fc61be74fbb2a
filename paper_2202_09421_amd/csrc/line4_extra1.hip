// Line passes for extended lengths 45, 60, 72, 120, 135, 192, 200, 300,
// 360, 384, 405, 600.
#include "line4_impl.h"

namespace rte {

template <typename T>
static hipError_t extra(const Lines4Args<T>& a, int Np, int nq, bool adj, hipStream_t s) {
  switch (Np) {
    case 45: return adj ? go_one<T, true, 5, 9>(a, nq, s) : go_one<T, false, 5, 9>(a, nq, s);
    case 60: return adj ? go_one<T, true, 6, 10>(a, nq, s) : go_one<T, false, 6, 10>(a, nq, s);
    case 72: return adj ? go_one<T, true, 6, 12>(a, nq, s) : go_one<T, false, 6, 12>(a, nq, s);
    case 120: return adj ? go_one<T, true, 10, 12>(a, nq, s) : go_one<T, false, 10, 12>(a, nq, s);
    case 135: return adj ? go_one<T, true, 9, 15>(a, nq, s) : go_one<T, false, 9, 15>(a, nq, s);
    case 192: return adj ? go_one<T, true, 12, 16>(a, nq, s) : go_one<T, false, 12, 16>(a, nq, s);
    case 200: return adj ? go_one<T, true, 20, 10>(a, nq, s) : go_one<T, false, 20, 10>(a, nq, s);
    case 300: return adj ? go_one<T, true, 6, 50>(a, nq, s) : go_one<T, false, 6, 50>(a, nq, s);
    case 360: return adj ? go_one<T, true, 8, 45>(a, nq, s) : go_one<T, false, 8, 45>(a, nq, s);
    case 384: return adj ? go_one<T, true, 6, 64>(a, nq, s) : go_one<T, false, 6, 64>(a, nq, s);
    case 405: return adj ? go_one<T, true, 5, 81>(a, nq, s) : go_one<T, false, 5, 81>(a, nq, s);
    case 600: return adj ? go_one<T, true, 12, 50>(a, nq, s) : go_one<T, false, 12, 50>(a, nq, s);
    default: return hipErrorNotSupported;
  }
}

hipError_t lines4_extra1(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }
hipError_t lines4_extra1(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s) { return extra(a, Np, nq, adj, s); }

}  // namespace rte
