// Line passes for extended lengths with a register-codelet split (included by
// the translation units that instantiate them).
#pragma once
// FC-Gram continuation + filtered spectral derivative along x lines (rows)
// and y lines (columns) of one state, or the exact transpose (Sec. 4.3).
//
// The DFT of length N = N1 x M is formed in stages that each hold their
// transforms in registers: A over the N1 index, and M = N2 x N3 either as one
// stage (N3 = 1) or as two (B over the N2 index, C over the N3 index).  The
// last forward stage multiplies by the derivative factor i mu_k and starts the
// inverse, which runs the stages backwards.  Where the two factors of a split
// are coprime the index maps of the prime-factor algorithm (Good 1958) are
// used, n -> (n mod N1, n mod M) with k = M k1 + N1 k2 mod N, and the split
// needs no twiddles at all; otherwise n = n1 M + m with twiddles w^(m k1).
//
// Work unit: two neighbouring lines of one ordinate group, four complex
// lines: complex line r holds slot r of the first line in its real part and
// slot r of the second in its imaginary part (the operator is real-linear, so
// both are differentiated by one complex transform).  Pairing one ordinate of
// two neighbouring lines keeps the rounding of each relative to values of
// similar size; pairing two ordinates of one line (a bright and a dim one,
// near a beam) makes the dim one's derivative inherit the bright one's
// rounding, which grew the gradient maps' error 4x at 513 x 513 x 64.
//
// A workgroup loads and stores its unit together (one 16-byte piece of a
// point's slots per lane, so that an instruction covers whole 32- or 64-byte
// runs of a row), and in between each wave transforms its own LPW complex
// lines: the stages of a wave are ordered by its own in-order LDS accesses,
// so a unit has two workgroup barriers in all.
//
// What bounds it (513 x 513 x 64, N = 540).  FP64, four sources: the streams,
// 2.2 GB a launch at 4.7 TB/s (462 / 465 us forward / transpose; 594 / 603 us
// with a barrier after each stage, two ordinates' values exchanged between
// lanes to form complex entries, twiddles at every step and each stage's 80
// to 108 jobs on a two-wave workgroup); with whole planes per group in memory
// it ran at 5.0 TB/s, the columns of a banded state cost that (rows 213 us,
// columns 247 us on 513 x 440).  FP32: vector and LDS issue, each busy for 57 %
// of the cycles (364 / 375 us; 540 / 571 us before).  At 257 x 257 x 32 a CU
// has eight units, one round: 18.9 / 20.7 us in FP64 (24.6 / 25.9 us before),
// 12 us of it the transforms.

#include "line4_stages.h"
#include "rte_internal.h"

namespace rte {

struct Lines4Dir {
  const double* coef;      // xi or eta in slot order
  const double* mu;        // multipliers in the order of the last stage (line4_orders)
  const double* Mx;        // (C + E) x 2d continuation matrix [MR | ML]
  const double* MxT;       // its transpose [side][kMaxFcD][C + E], zero rows beyond d
  const double2* tw;       // twiddle powers in job order (line4_orders)
  int n, CE, Np;           // nodes per line, extension points, their sum
  int pr[kMaxFcD], pl[kMaxFcD];  // LDS positions of the matching values n - d + k and d - 1 - k (k < d; else 0)
  int nlines, npe;         // lines, line pairs rounded up to even
  bool along_x;            // lines are rows (else columns)
};

template <typename T>
struct Lines4Args {
  const T* in;
  T* out[2];
  Lines4Dir dir[2];
  RowMap rows;
  int64_t grp_stride, inst_stride;
  int G, d;
  int first, units_first;  // direction of units [0, units_first) of a (source, group)
  int nunits;              // units per (source, group)
  int nt_out;              // non-temporal stores: bit 0 rows, bit 1 columns
};

// LDS accesses of one wave are executed in order; this keeps the compiler's order
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 16 bytes of one (point, line): 2 FP64 or 4 FP32 slots
typedef double d2v __attribute__((ext_vector_type(2)));
typedef float f4v16 __attribute__((ext_vector_type(4)));
template <typename T>
struct Vec16;
template <>
struct Vec16<double> { typedef d2v type; };
template <>
struct Vec16<float> { typedef f4v16 type; };

// Workgroup b runs on XCD b % 8, so units 2x and 2x + 1 of each chunk of 16
// (the two column pairs of one 128-byte row segment) go to workgroups b and
// b + 8 of that chunk, i.e. to one XCD and its L2.
__device__ __forceinline__ int remap_unit16(int b) {
  const int chunk = b >> 4, x = b & 7, h = (b >> 3) & 1;
  return chunk * 16 + 2 * x + h;
}

// Sum over the 4 lanes of a quad (DPP quad permutations)
__device__ __forceinline__ double quad_sum(double x) {
  auto dpp = [](double v, auto sel) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(u & 0xffffffffLL), decltype(sel)::value, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), decltype(sel)::value, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
  };
  x += dpp(x, std::integral_constant<int, 0xB1>());   // lane ^ 1
  x += dpp(x, std::integral_constant<int, 0x4E>());   // lane ^ 2
  return x;
}

// Row p of the continuation matrix: coefficients of the right and the left
// matching values (MxT: lanes read consecutive rows).  The first kFcD5 values
// are read without a test (the rows beyond d are zero), the others only when
// d > kFcD5.
constexpr int kFcD5 = 5;
struct MxRow {
  double r[kMaxFcD], l[kMaxFcD];
  __device__ __forceinline__ void load(const Lines4Dir& D, int dd, int p) {
    const int pc = min(p, D.CE - 1);
#pragma unroll
    for (int k = 0; k < kFcD5; ++k) {
      r[k] = D.MxT[k * D.CE + pc];
      l[k] = D.MxT[(kMaxFcD + k) * D.CE + pc];
    }
    if (dd > kFcD5) {
#pragma unroll
      for (int k = kFcD5; k < kMaxFcD; ++k) {
        r[k] = D.MxT[k * D.CE + pc];
        l[k] = D.MxT[(kMaxFcD + k) * D.CE + pc];
      }
    }
  }
  // extension value of line L
  __device__ __forceinline__ cx<double> apply(const Lines4Dir& D, int dd, const cx<double>* L) const {
    double sr = 0.0, si = 0.0;
    auto add = [&](int k) {
      const cx<double> gr = L[D.pr[k]], gl = L[D.pl[k]];
      sr += r[k] * gr.re + l[k] * gl.re;
      si += r[k] * gr.im + l[k] * gl.im;
    };
#pragma unroll
    for (int k = 0; k < kFcD5; ++k) add(k);
    if (dd > kFcD5) {
#pragma unroll
      for (int k = kFcD5; k < kMaxFcD; ++k) add(k);
    }
    return {sr, si};
  }
};

// byte offset of point i of a line (columns: the terms of RowMap)
struct PtMap {
  uint32_t inv, ps, skip, most;
  __device__ __forceinline__ uint32_t operator()(int i) const {
    return (uint32_t)i * ps + min(__umulhi((uint32_t)i, inv) * skip, most);
  }
};

// Stores of one lane: its piece of every PT-th point.  NT: non-temporal, for
// plans that stream their state arrays.
template <class G, typename T, bool NT>
__device__ __forceinline__ void store_unit(char* out, const double* src, uint32_t lout, PtMap pt, int i0, int n) {
  constexpr int SL = 16 / sizeof(T), PT = G::NTH / (8 / SL), TMAX = (G::N - 1 + PT - 1) / PT;
  typedef typename Vec16<T>::type V16;
#pragma unroll
  for (int t = 0; t < TMAX; ++t) {
    const int i = i0 + PT * t;
    if (i < n) {
      const double* q = src + 2 * G::pos(i);
      V16 o;
#pragma unroll
      for (int r = 0; r < SL; ++r) o[r] = T(q[2 * r * G::LSZ]);
      V16* dst = reinterpret_cast<V16*>(out + (lout + pt(i)));
      if constexpr (NT) __builtin_nontemporal_store(o, dst);
      else *dst = o;
    }
  }
}

// Lines line0 and line0 + 1 of direction D of the block's (source, group), by
// the first G::NTH threads.  All waves of the block call this, those beyond with
// active = false (the same for a whole wave): they share the barriers and do
// nothing else.
template <typename T, bool ADJ, int N1, int M>
__device__ __forceinline__ void lines4_unit(const Lines4Args<T>& a, const Lines4Dir& D, T* dout, int line0, unsigned char* smem_raw,
                                            bool active) {
  typedef Geo<N1, M> G;
  constexpr int N = G::N, NTH = G::NTH, LPW = G::LPW;
  cx<double>* buf = reinterpret_cast<cx<double>*>(smem_raw);
  double* bufd = reinterpret_cast<double*>(smem_raw);
  const bool has1 = line0 + 1 < D.nlines;
  const int g = (int)blockIdx.y, s0 = g * kGroup;
  const uint32_t l0 = D.along_x ? a.rows(line0, g) : (uint32_t)line0 * kGroup;
  const int64_t base = (int64_t)blockIdx.z * a.inst_stride + (int64_t)g * a.grp_stride + l0;
  const int n = D.n, CE = D.CE, dd = a.d;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // lane = (point, line, 16-byte piece of its 4 slots): neighbouring lanes
  // cover a point's 32 (x lines) or 64 (y lines) contiguous bytes
  constexpr int SL = 16 / sizeof(T), PC = 4 / SL;   // slots per lane, pieces per (point, line)
  typedef typename Vec16<T>::type V16;
  const int pc = tid % PC, it = tid / PC & 1, i0 = tid / (2 * PC);
  constexpr int PT = NTH / (2 * PC);                // points per load slot
  constexpr int TMAX = (N - 1 + PT - 1) / PT;       // n < N

  // byte offsets from the unit's base fit 32 bits (one source's state is below 4 GiB)
  const char* in = reinterpret_cast<const char*>(a.in + base);
  const uint32_t ls = ((D.along_x ? a.rows(line0 + 1, g) : (uint32_t)(line0 + 1) * kGroup) - l0) * (uint32_t)sizeof(T);
  const PtMap pt{a.rows.inv, (D.along_x ? (uint32_t)kGroup : a.rows.row) * (uint32_t)sizeof(T),
                 D.along_x ? 0u : a.rows.skip * (uint32_t)sizeof(T),
                 (a.rows.most - (uint32_t)g * a.rows.cut) * (uint32_t)sizeof(T)};
  const uint32_t lin = ((it && has1) ? ls : 0u) + 16u * pc;
  constexpr int CH = TMAX < 20 ? TMAX : (TMAX + 1) / 2;
  // the lane's row of the continuation matrix (first job of the extension)
  MxRow row;
  const double2* __restrict__ tw = D.tw;
  if (active) {
    if constexpr (!ADJ) row.load(D, dd, lane / LPW);
#pragma unroll
    for (int c0 = 0; c0 < TMAX; c0 += CH) {
      V16 v[CH];
#pragma unroll
      for (int t = 0; t < CH; ++t) {
        const int i = i0 + PT * (c0 + t);
        if (c0 + t < TMAX) v[t] = *reinterpret_cast<const V16*>(in + (lin + pt(min(i, n - 1))));
      }
      if (!has1 && it) {
#pragma unroll
        for (int t = 0; t < CH; ++t) v[t] = V16(T(0));
      }
#pragma unroll
      for (int t = 0; t < CH; ++t) {
        const int i = i0 + PT * (c0 + t);
        if (c0 + t < TMAX && i < n) {
          double* q = bufd + 2 * (G::pos(i) + pc * SL * G::LSZ) + it;
#pragma unroll
          for (int r = 0; r < SL; ++r) q[2 * r * G::LSZ] = (double)v[t][r];
        }
      }
    }
  }
  __syncthreads();

  if (active) {
    // ---- the wave's own complex lines
    cx<double>* L = buf + wave * LPW * G::LSZ;
    if constexpr (ADJ) {
      for (int e = lane; e < LPW * CE; e += 64) L[(e % LPW) * G::LSZ + G::pos(n + e / LPW)] = {0.0, 0.0};
    } else {
      // extension values (Sec. 4.3 steps 1-4 as one linear map of the 2d
      // matching values): job (row p, line l)
      for (int e = lane; e < LPW * CE; e += 64) {
        const int l = e % LPW, p = e / LPW;
        if (e >= 64) row.load(D, dd, p);
        L[l * G::LSZ + G::pos(n + p)] = row.apply(D, dd, L + l * G::LSZ);
      }
    }
    wave_order();
    stage_a<G, -1>(L, lane, tw);
    wave_order();
    if constexpr (G::THREE) {
      stage_b<G, -1>(L, lane, tw);
      wave_order();
    }
    stage_c<G>(L, lane, D.mu, D.coef + s0 + wave * LPW);
    wave_order();
    if constexpr (G::THREE) {
      stage_b<G, 1>(L, lane, tw);
      wave_order();
    }
    // fold of the extension region onto the 2d matching points (transpose of the
    // continuation): quad c sums column c over the extension rows.  From 128 to
    // 600 points its first 8 coefficients are read before the last stage (N = 540:
    // 437 us against 451, N = 160: 8.9 against 9.3; N = 90 and 1080 lose 4 and 1 %).
    const int c = lane >> 2, part = lane & 3;
    const bool on = c < 2 * dd;
    constexpr int kFold = N >= 128 && N <= 600 ? 8 : 0;
    double mf[kFold + 1];
    if constexpr (ADJ) {
#pragma unroll
      for (int j = 0; j < kFold; ++j) mf[j] = D.Mx[min(part + 4 * j, CE - 1) * 2 * dd + min(c, 2 * dd - 1)];
    }
    stage_a<G, 1>(L, lane, tw);
    wave_order();
    if constexpr (ADJ) {
      double sr[LPW] = {}, si[LPW] = {};
      auto add = [&](int p, double mv) {
        const cx<double>* y = L + G::pos(n + p);
#pragma unroll
        for (int l = 0; l < LPW; ++l) {
          sr[l] += mv * y[l * G::LSZ].re;
          si[l] += mv * y[l * G::LSZ].im;
        }
      };
      if (on) {
#pragma unroll
        for (int j = 0; j < kFold; ++j)
          if (part + 4 * j < CE) add(part + 4 * j, mf[j]);
        for (int p = part + 4 * kFold; p < CE; p += 4) add(p, D.Mx[p * 2 * dd + c]);
      }
      cx<double>* q = L + (on ? G::pos(c < dd ? n - dd + c : 2 * dd - 1 - c) : 0);
#pragma unroll
      for (int l = 0; l < LPW; ++l) {
        const double fr = quad_sum(sr[l]), fi = quad_sum(si[l]);
        if (on && part == 0) {
          q[l * G::LSZ].re += fr;
          q[l * G::LSZ].im += fi;
        }
      }
    }
  }
  __syncthreads();

  if (!active || (it && !has1)) return;
  const uint32_t lout = (it ? ls : 0u) + 16u * pc;
  char* out = reinterpret_cast<char*>(dout + base);
  const double* src = bufd + 2 * (pc * SL * G::LSZ) + it;
  if (a.nt_out & (D.along_x ? 1 : 2)) store_unit<G, T, true>(out, src, lout, pt, i0, n);
  else store_unit<G, T, false>(out, src, lout, pt, i0, n);
}

template <typename T, bool ADJ, int N1, int M>
__global__ __launch_bounds__((Geo<N1, M>::NTH)) void lines4_kernel(Lines4Args<T> a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int u = remap_unit16((int)blockIdx.x);
  if (u >= a.nunits) return;
  const bool second = u >= a.units_first;
  const int dirn = second ? 1 - a.first : a.first;
  const int line0 = 2 * (second ? u - a.units_first : u);
  if (line0 >= a.dir[dirn].nlines) return;
  lines4_unit<T, ADJ, N1, M>(a, a.dir[dirn], a.out[dirn], line0, smem_raw, true);
}

constexpr size_t kLines4MaxLds = 160 * 1024;

// LDS positions of the matching values
template <int N1, int M>
inline void set_positions(Lines4Dir& D, int d) {
  typedef Geo<N1, M> G;
  for (int k = 0; k < kMaxFcD; ++k) {
    D.pr[k] = k < d ? G::pos(D.n - d + k) : 0;
    D.pl[k] = k < d ? G::pos(d - 1 - k) : 0;
  }
}

template <typename T, bool ADJ, int N1, int M>
inline hipError_t go_one(Lines4Args<T> a, int nq, hipStream_t s) {
  typedef Geo<N1, M> G;
  for (Lines4Dir& D : a.dir) set_positions<N1, M>(D, a.d);
  static_assert(G::bytes <= kLines4MaxLds, "line buffer exceeds the LDS of a CU");
  if (a.nunits == 0) return hipSuccess;
  const unsigned gx = (unsigned)(((a.nunits + 15) / 16) * 16);
  hipLaunchKernelGGL((lines4_kernel<T, ADJ, N1, M>), dim3(gx, (unsigned)a.G, (unsigned)nq), dim3(G::NTH), G::bytes, s, a);
  return hipGetLastError();
}

// both directions of unequal lengths in one launch; hipErrorNotSupported where
// that is not built or not faster
hipError_t lines4_mixed(const Lines4Args<double>& a, int nq, bool adj, hipStream_t s);
hipError_t lines4_mixed(const Lines4Args<float>& a, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra0(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra0(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra1(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra1(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra2(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra2(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra3(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_extra3(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_long0(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_long0(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_long1(const Lines4Args<double>& a, int Np, int nq, bool adj, hipStream_t s);
hipError_t lines4_long1(const Lines4Args<float>& a, int Np, int nq, bool adj, hipStream_t s);

}  // namespace rte
