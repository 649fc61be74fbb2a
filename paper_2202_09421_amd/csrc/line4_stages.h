// The transform stages of the line passes, on lines in LDS (line4_impl.h runs
// them; a host build runs the same code on ordinary memory).  Split, LDS
// positions, twiddle and multiplier orders, and the stages themselves.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

#include "fft_codelets.h"

namespace rte {

constexpr int kLP = 4;  // complex lines per unit (slot r of both lines, r = 0..3)

constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v / 2); }
constexpr int tw_powers(int K) { return ilog2c(K - 1) + 1; }   // 2^0 .. 2^j <= K - 1
constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }

// First factor N2 of the second factor m of a split n1 x m (m / N2 = N3; m
// itself: one stage).  The splits of all lengths are the fastest of those with
// the lowest instruction and LDS counts, forward plus transposed pass on an
// (N - 25)-node square grid with 32 ordinates.  That is three stages from 270
// on but for five lengths: with two, most need radices up to 32 (over 200
// registers, two waves per SIMD) and fill the lanes worse (20 x 27 at N = 540:
// 27 and 20 jobs a line for 64 lanes).  375 = 15 x 25, 576 = 24 x 24, 625 = 25 x
// 25, 729 = 27 x 27 and 800 = 32 x 25 measured faster in two all the same, and
// twelve shorter lengths (48, 64, 75, 90, 96, 100, 125, 128, 162, 216, 243, 250)
// in three.
constexpr int inner_n2(int n1, int m) {
  switch (n1 * m) {
    case 216: case 675: case 810: return 3;
    case 48: case 64: case 96: case 128: case 640: case 768: case 960: case 1024: case 1152: return 4;
    case 75: case 100: case 125: case 250: case 750: case 1125: return 5;
    case 90: case 162: case 288: case 324: case 432: case 486: case 648: case 972: case 1080: return 6;
    case 320: case 384: case 512: return 8;
    case 243: case 360: case 405: case 540: return 9;
    case 270: case 300: case 400: case 450: case 500: case 600: case 1200: return 10;
    case 480: case 720: return 12;
    case 900: return 15;
    case 864: return 16;
    case 1000: return 20;
    default: return m;
  }
}

// Complex lines per wave (1, 2 or 4; 4 / this = waves per unit).  Short lines:
// all four on one wave (fewest instructions, no workgroup barrier between
// waves; N = 160, FP64: 8.8 us against 9.8 / 10.1 us with two / one, 129 x 129
// x 32 forward pass).  Long lines: one per wave, whose smaller radices leave
// four waves per SIMD (N = 288: 20.1 us against 21.6 / 26.7 us with two / four,
// 257 x 257 x 32; N = 540: 93 us against 102 / 146 us, 513 x 513 x 64).  In
// between, and at the five long lengths of two stages, whichever measured faster.
constexpr int lines_per_wave(int n1, int m) {
  const int N = n1 * m;
  switch (N) {
    case 45: case 48: case 50: case 54: case 60: case 64: case 72: case 75: case 80: case 81: case 108:
    case 120: case 135: case 144: case 150: case 160: case 180: case 192: case 200: case 225: case 240:
    case 256: return 4;
    case 90: case 96: case 100: case 125: case 128: case 162: case 216: case 243: case 250: case 270: case 300:
    case 375: case 576: case 625: case 729: case 800: return 2;
    default: return 1;
  }
}

// LDS positions.  Line = [N1][block], block = [N2][S3] (three factors) or [M].
// S3 is odd, so the last stage's lanes (rows S3 apart) fall in distinct banks
// (16-byte entries, 16 per bank row); the block pitch S1 is padded by the
// amount that leaves the fewest bank conflicts over the stages without
// lowering the units that fit a CU.
template <int N1_, int M_>
struct Geo {
  static constexpr int N1 = N1_, M = M_, N = N1 * M;
  static constexpr int N2 = inner_n2(N1, M), N3 = M / N2;
  static constexpr bool THREE = N3 > 1;
  static constexpr bool PF1 = gcd_c(N1, M) == 1, PF2 = THREE && gcd_c(N2, N3) == 1;
  static constexpr int LPW = lines_per_wave(N1, M), NW = kLP / LPW, NTH = 64 * NW;
  static constexpr int S3 = THREE ? (N3 | 1) : 1;
  static constexpr int BLK = THREE ? N2 * S3 : M;

  // largest number of a 16-lane group's entries on one bank column, summed over the groups of one access
  static constexpr int conflicts(int s1, int stage) {
    int cost = 0;
    for (int g = 0; g < 4; ++g) {
      int cnt[16] = {};
      int worst = 0;
      for (int l = 0; l < 16; ++l) {
        const int job = 16 * g + l;
        int e = 0;
        if (stage == 0) {         // staging and stores: consecutive points
          const int n1 = PF1 ? job % N1 : job / M, m = job % M;
          e = n1 * s1 + (!THREE ? m : (PF2 ? (m % N2) * S3 + m % N3 : (m / N3) * S3 + m % N3));
        } else if (stage == 1) {  // A
          if (job >= M) break;
          e = THREE ? (job / N3) * S3 + job % N3 : job;
        } else if (stage == 2) {  // B
          if (!THREE || job >= N1 * N3) break;
          e = (job / N3) * s1 + job % N3;
        } else {                  // last stage
          if (THREE) {
            if (job >= N1 * N2) break;
            e = (job / N2) * s1 + (job % N2) * S3;
          } else {
            if (job >= N1) break;
            e = job * s1;
          }
        }
        const int c = ++cnt[e % 16];
        if (c > worst) worst = c;
      }
      cost += worst;
    }
    return cost;
  }
  static constexpr int total(int s1) {
    return 2 * conflicts(s1, 0) + 4 * conflicts(s1, 1) + 4 * conflicts(s1, 2) + 2 * conflicts(s1, 3);
  }
  static constexpr int lsz(int s1) { return N1 * s1 + (12 - N1 * s1 % 8) % 8; }
  static constexpr int fit(int s1) { return 163840 / (16 * kLP * lsz(s1)); }
  static constexpr int pick() {
    int best = BLK, cost = total(BLK);
    for (int s = BLK + 1; s <= BLK + 16; ++s) {
      if (fit(s) < fit(BLK) && fit(BLK) <= 8) continue;
      const int c = total(s);
      if (c < cost) {
        cost = c;
        best = s;
      }
    }
    return best;
  }
  static constexpr int S1 = pick();
  static constexpr int LSZ = lsz(S1);
  static constexpr size_t bytes = sizeof(double) * 2 * kLP * LSZ;

  // position of point n of a line
  static RTE_HD int pos(int n) {
    const int n1 = PF1 ? n % N1 : n / M, m = n % M;
    return n1 * S1 + (!THREE ? m : (PF2 ? (m % N2) * S3 + m % N3 : jpos(m)));
  }
  // position inside a block of stage-A job j
  static RTE_HD int jpos(int j) { return (!THREE || S3 == N3) ? j : (j / N3) * S3 + j % N3; }
  // entries of the stage-A twiddle table (stage B's follow)
  static constexpr int TWA = PF1 ? 0 : tw_powers(N1) * M;
};

// Twiddles w^k, k = 1 .. K - 1, of one job: only the table values w^(2^j) are
// loaded, and every other power is one complex product of an earlier power
// and one of them, at most log2 K products deep (relative error a few units
// in the last place).  The table holds w^(2^j) of every job in job order
// (split_orders), so a wave's load is one run.  TW: pair of doubles x, y.

template <int K>
struct TwPow {
  static constexpr int NB = tw_powers(K);
  cx<double> P[NB];
  cx<double> w[K];
  // job's entries of a table of J jobs
  template <int J, typename TW>
  RTE_HD void load(const TW* __restrict__ t, int job) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const TW v = t[j * J + job];
      P[j] = {v.x, v.y};
    }
  }
  template <int k>
  RTE_HD cx<double> get() {
    constexpr int lb = k & -k;
    constexpr int j = ilog2c(lb);
    static_assert(j < NB, "power table too short");
    if constexpr (k == lb) {
      w[k] = P[j];
    } else {
      const cx<double> a = w[k - lb], p = P[j];
      w[k] = {a.re * p.re - a.im * p.im, a.re * p.im + a.im * p.re};
    }
    return w[k];
  }
};

// x[k] *= w^(S k) for k = k0 .. K - 1 (S = +-1 conjugates)
template <int K, int k, int S>
struct TwApply {
  static RTE_HD void run(TwPow<K>& tp, cx<double>* x) {
    const cx<double> w = tp.template get<k>();
    x[k] = cx_rot(x[k], w.re, S * w.im);
    TwApply<K, k + 1, S>::run(tp, x);
  }
};
template <int K, int S>
struct TwApply<K, K, S> {
  static RTE_HD void run(TwPow<K>&, cx<double>*) {}
};

// R entries of a line, STRIDE apart
template <int R, int STRIDE>
RTE_HD void ld(const cx<double>* p, cx<double>* x) {
#pragma unroll
  for (int i = 0; i < R; ++i) x[i] = p[i * STRIDE];
}
template <int R, int STRIDE>
RTE_HD void st(cx<double>* p, const cx<double>* x) {
#pragma unroll
  for (int i = 0; i < R; ++i) p[i * STRIDE] = x[i];
}

// S = -1: forward stage A of the wave's lines (transforms over the N1 index,
// then the twiddles); S = +1: its inverse.  Job j: position j of every block.
template <class G, int S, typename TW>
RTE_HD void stage_a(cx<double>* L, int lane, const TW* __restrict__ tw) {
  constexpr int J = G::LPW * G::M;
#pragma unroll
  for (int t = 0; t < (J + 63) / 64; ++t) {
    const int job = lane + 64 * t;
    if (J % 64 == 0 || 64 * (t + 1) <= J || job < J) {
      const int l = G::LPW == 1 ? 0 : job / G::M, j = G::LPW == 1 ? job : job % G::M;
      cx<double>* p = L + l * G::LSZ + G::jpos(j);
      cx<double> x[G::N1];
      ld<G::N1, G::S1>(p, x);
      if constexpr (S < 0) Dft<G::N1, -1, double>::run(x);
      if constexpr (!G::PF1) {
        TwPow<G::N1> tp;
        tp.template load<G::M>(tw, j);
        TwApply<G::N1, 1, -S>::run(tp, x);
      }
      if constexpr (S > 0) Dft<G::N1, 1, double>::run(x);
      st<G::N1, G::S1>(p, x);
    }
  }
}

// the same over the N2 index inside each block; job (k1, b)
template <class G, int S, typename TW>
RTE_HD void stage_b(cx<double>* L, int lane, const TW* __restrict__ tw) {
  constexpr int JL = G::N1 * G::N3, J = G::LPW * JL;
#pragma unroll
  for (int t = 0; t < (J + 63) / 64; ++t) {
    const int job = lane + 64 * t;
    if (J % 64 == 0 || 64 * (t + 1) <= J || job < J) {
      const int l = G::LPW == 1 ? 0 : job / JL, r = G::LPW == 1 ? job : job % JL;
      const int k1 = r / G::N3, b = r % G::N3;
      cx<double>* p = L + l * G::LSZ + k1 * G::S1 + b;
      cx<double> x[G::N2];
      ld<G::N2, G::S3>(p, x);
      if constexpr (S < 0) Dft<G::N2, -1, double>::run(x);
      if constexpr (!G::PF2) {
        TwPow<G::N2> tp;
        tp.template load<G::N3>(tw + G::TWA, b);
        TwApply<G::N2, 1, -S>::run(tp, x);
      }
      if constexpr (S > 0) Dft<G::N2, 1, double>::run(x);
      st<G::N2, G::S3>(p, x);
    }
  }
}

// last stage: forward transforms, the line's factor i mu cf (cf = xi or eta of
// its ordinate; -i mu cf for both passes, the forward one being -xi D and the
// transpose conjugating i), inverse transforms
template <class G>
RTE_HD void stage_c(cx<double>* L, int lane, const double* __restrict__ mu,
                                        const double* __restrict__ coef) {
  constexpr int R = G::THREE ? G::N3 : G::N2, JL = G::N / R, J = G::LPW * JL;
#pragma unroll
  for (int t = 0; t < (J + 63) / 64; ++t) {
    const int job = lane + 64 * t;
    if (J % 64 == 0 || 64 * (t + 1) <= J || job < J) {
      const int l = G::LPW == 1 ? 0 : job / JL, r = G::LPW == 1 ? job : job % JL;
      cx<double>* p = L + l * G::LSZ + (G::THREE ? (r / G::N2) * G::S1 + (r % G::N2) * G::S3 : r * G::S1);
      const double cf = coef[l];
      cx<double> x[R];
      double m[R];
#pragma unroll
      for (int i = 0; i < R; ++i) m[i] = mu[i * JL + r];
      ld<R, 1>(p, x);
      Dft<R, -1, double>::run(x);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const cx<double> X = x[i];
        const double mc = m[i] * cf;
        x[i] = {mc * X.im, -mc * X.re};
      }
      Dft<R, 1, double>::run(x);
      st<R, 1>(p, x);
    }
  }
}

// Table orders of the split n1 x m: entry e of its multipliers is that of
// frequency mu[e], entry e of its twiddles is exp(-2 pi i tw[e] / (n1 m))
inline void split_orders(int n1, int m, std::vector<int>& mu, std::vector<int>& tw) {
  const int Np = n1 * m;
  const int n2 = inner_n2(n1, m), n3 = m / n2;
  const bool three = n3 > 1, pf1 = gcd_c(n1, m) == 1, pf2 = three && gcd_c(n2, n3) == 1;
  const int last = three ? n3 : n2, jobs = Np / last;
  mu.assign(Np, 0);
  for (int i = 0; i < last; ++i)
    for (int r = 0; r < jobs; ++r) {
      const int k1 = three ? r / n2 : r, k2 = three ? r % n2 : 0;
      const int km = !three ? i : (pf2 ? (n3 * k2 + n2 * i) % m : k2 + n2 * i);
      mu[i * jobs + r] = pf1 ? (m * k1 + n1 * km) % Np : k1 + n1 * km;
    }
  // stage-A job j holds the block index jm with (jm mod n2, jm mod n3) = (j / n3, j % n3)
  // in a coprime inner split, else jm = j
  if (!pf1)
    for (int p = 0; p < tw_powers(n1); ++p)
      for (int j = 0; j < m; ++j) {
        int jm = j;
        if (pf2) {
          jm = j % n3;
          while (jm % n2 != j / n3) jm += n3;
        }
        tw.push_back((int)(((int64_t)jm << p) % Np));
      }
  if (three && !pf2)
    for (int p = 0; p < tw_powers(n2); ++p)
      for (int b = 0; b < n3; ++b) tw.push_back((int)(((int64_t)n1 * b << p) % Np));
}

}  // namespace rte
