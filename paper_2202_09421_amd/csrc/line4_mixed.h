// Both directions in one launch on grids whose extended lengths differ.
//
// On a small grid a line pass is launch and memory latency, and a second launch
// costs as much as the first.  This kernel holds the units of all lengths up to
// 256 and a block takes the one of its direction.  Forward / transposed pass,
// us, two launches and one (FP64): 25 x 21 x 8 7.6 / 9.2 and 4.3 / 5.1,
// 60 x 40 x 16 8.3 / 10.2 and 4.6 / 5.4, 120 x 80 x 32 10.9 / 12.2 and
// 6.8 / 7.1, 200 x 150 x 32 with two sources 21.5 / 22.3 and 17.3 / 16.6.  It
// needs the registers of its largest length (160, three waves per SIMD)
// and the waves of the longer line, so larger grids keep two launches; and with
// the lengths up to 600 in it, grids of those got slower (301 x 190 x 20, two
// sources: 25.9 / 29.2 and 32.1 / 37.0).
#pragma once
#include <algorithm>

#include "line4_impl.h"

namespace rte {

// lengths and splits as in fourstep_split
#define RTE_MIXED_SIZES(X)                                                                                          \
  X(45, 5, 9) X(48, 3, 16) X(50, 5, 10) X(54, 6, 9) X(60, 6, 10) X(64, 4, 16) X(72, 6, 12) X(75, 3, 25)             \
  X(80, 8, 10) X(81, 9, 9) X(90, 3, 30) X(96, 3, 32) X(100, 4, 25) X(108, 9, 12) X(120, 10, 12) X(125, 5, 25)       \
  X(128, 4, 32) X(135, 9, 15) X(144, 12, 12) X(150, 10, 15) X(160, 10, 16) X(162, 3, 54) X(180, 12, 15)             \
  X(192, 12, 16) X(200, 20, 10) X(216, 8, 27) X(225, 15, 15) X(240, 16, 15) X(243, 3, 81) X(250, 10, 25)            \
  X(256, 16, 16)

// a.dir[dirn], member by member (indexed at run time over this many uses, the
// arguments would be copied to scratch memory)
template <typename T>
__device__ __forceinline__ Lines4Dir pick_dir(const Lines4Args<T>& a, bool y) {
  const Lines4Dir &u = a.dir[0], &v = a.dir[1];
  Lines4Dir D;
  D.coef = y ? v.coef : u.coef;
  D.mu = y ? v.mu : u.mu;
  D.Mx = y ? v.Mx : u.Mx;
  D.MxT = y ? v.MxT : u.MxT;
  D.tw = y ? v.tw : u.tw;
  D.n = y ? v.n : u.n;
  D.CE = y ? v.CE : u.CE;
  D.Np = y ? v.Np : u.Np;
  D.nlines = y ? v.nlines : u.nlines;
  D.npe = y ? v.npe : u.npe;
  D.along_x = y ? v.along_x : u.along_x;
#pragma unroll
  for (int k = 0; k < kMaxFcD; ++k) {
    D.pr[k] = y ? v.pr[k] : u.pr[k];
    D.pl[k] = y ? v.pl[k] : u.pl[k];
  }
  return D;
}

template <typename T, bool ADJ>
__global__ __launch_bounds__(256) void lines4_mixed_kernel(Lines4Args<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int u = remap_unit16((int)blockIdx.x);
  if (u >= a.nunits) return;
  const bool second = u >= a.units_first, y = second != (a.first == 1);
  const Lines4Dir D = pick_dir(a, y);
  T* dout = y ? a.out[1] : a.out[0];
  const int line0 = 2 * (second ? u - a.units_first : u);
  if (line0 >= D.nlines) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  switch (D.Np) {
#define RTE_CASE(n, n1, m)                                                                      \
  case n:                                                                                       \
    lines4_unit<T, ADJ, n1, m>(a, D, dout, line0, smem_raw, wave < Geo<n1, m>::NW);             \
    break;
    RTE_MIXED_SIZES(RTE_CASE)
#undef RTE_CASE
  }
}

struct MixedSize {
  int np, n1, threads;
  size_t bytes;
  void (*positions)(Lines4Dir&, int);
};

inline const MixedSize* mixed_size(int np) {
#define RTE_ROW(n, n1, m) {n, n1, Geo<n1, m>::NTH, Geo<n1, m>::bytes, set_positions<n1, m>},
  static const MixedSize rows[] = {RTE_MIXED_SIZES(RTE_ROW)};
#undef RTE_ROW
  int n1 = 0, m = 0;
  for (const MixedSize& r : rows)
    if (r.np == np && fourstep_split(np, &n1, &m) && n1 == r.n1) return &r;
  return nullptr;
}

template <typename T>
inline hipError_t mixed(Lines4Args<T> a, int nq, bool adj, hipStream_t s) {
  const MixedSize* x = mixed_size(a.dir[0].Np);
  const MixedSize* y = mixed_size(a.dir[1].Np);
  if (!x || !y) return hipErrorNotSupported;
  // faster at every size tried up to 4096 blocks (4608: 20 against 26 us at
  // 140 x 130 x 64 with two sources) where both lengths use as many waves; with
  // idle ones in the shorter lines' blocks up to 2048 (1792: 11.3 / 13.5 us
  // against 13.7 / 14.9 at 180 x 40 x 64; 3584: 17.4 / 22.0 against 18.2 / 19.2)
  const unsigned gx = (unsigned)(((a.nunits + 15) / 16) * 16);
  if ((int64_t)gx * a.G * nq > (x->threads == y->threads ? 4096 : 2048)) return hipErrorNotSupported;
  x->positions(a.dir[0], a.d);
  y->positions(a.dir[1], a.d);
  const dim3 grid(gx, (unsigned)a.G, (unsigned)nq), block((unsigned)std::max(x->threads, y->threads));
  const size_t bytes = std::max(x->bytes, y->bytes);
  if (adj) hipLaunchKernelGGL((lines4_mixed_kernel<T, true>), grid, block, bytes, s, a);
  else hipLaunchKernelGGL((lines4_mixed_kernel<T, false>), grid, block, bytes, s, a);
  return hipGetLastError();
}

}  // namespace rte
