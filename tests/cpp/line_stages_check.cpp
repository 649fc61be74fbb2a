// CPU check of the line kernels' transform stages (line4_stages.h): for every
// split, the code that a wave runs on its lines in LDS, lane by lane, with the
// kernel's positions, table orders and twiddle powers, against
//   y = IDFT(-i mu c DFT(x))
// by brute force in long double (mu: a random multiplier per frequency, c: the
// line's coefficient).  Every position of a line has to be its own and inside
// the line.  Built with g++ and AddressSanitizer / UndefinedBehaviorSanitizer;
// the splits come from a generated file (line_splits.inc).
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <set>
#include <vector>

#include "line4_stages.h"

using namespace rte;
typedef std::complex<long double> cld;

struct Tw {
  double x, y;
};

static int g_fail = 0;
static double g_worst = 0.0;

static std::vector<cld> roots(int N) {
  std::vector<cld> w(N);
  for (int e = 0; e < N; ++e) {
    const long double a = -2.0L * 3.141592653589793238462643383279502884L * e / N;
    w[e] = cld(std::cos(a), std::sin(a));
  }
  return w;
}

static std::vector<cld> dft(const std::vector<cld>& x, const std::vector<cld>& w, bool inverse) {
  const long N = (long)x.size();
  std::vector<cld> y(N);
  for (long k = 0; k < N; ++k)
    for (long n = 0; n < N; ++n) y[k] += x[n] * (inverse ? std::conj(w[n * k % N]) : w[n * k % N]);
  return y;
}

template <int N1, int M>
static void check() {
  typedef Geo<N1, M> G;
  constexpr int N = G::N;
  std::mt19937_64 rng(N);
  std::uniform_real_distribution<double> u(-1, 1);
  const std::vector<cld> w = roots(N);
  // tables as the plan builds them
  std::vector<int> mu_order, tw_order;
  split_orders(N1, M, mu_order, tw_order);
  std::vector<double> mu(N), mup;
  for (double& m : mu) m = u(rng);
  for (int k : mu_order) mup.push_back(mu.at(k));
  std::vector<Tw> tw;
  for (int e : tw_order) tw.push_back({(double)w.at(e).real(), (double)w.at(e).imag()});
  std::set<int> pos;
  for (int n = 0; n < N; ++n) pos.insert(G::pos(n));
  bool ok = (int)pos.size() == N && *pos.begin() >= 0 && *pos.rbegin() < G::LSZ && (int)mup.size() == N;
  // one wave: LPW lines
  std::vector<cx<double>> lds((size_t)G::LPW * G::LSZ);
  std::vector<double> coef(G::LPW);
  std::vector<std::vector<cld>> x(G::LPW, std::vector<cld>(N));
  for (int l = 0; l < G::LPW; ++l) {
    coef[l] = u(rng);
    for (int n = 0; n < N; ++n) {
      const cx<double> v = {u(rng), u(rng)};
      x[l][n] = cld(v.re, v.im);
      lds.at((size_t)l * G::LSZ + G::pos(n)) = v;
    }
  }
  cx<double>* L = lds.data();
  for (int lane = 0; lane < 64; ++lane) stage_a<G, -1>(L, lane, tw.data());
  if constexpr (G::THREE)
    for (int lane = 0; lane < 64; ++lane) stage_b<G, -1>(L, lane, tw.data());
  for (int lane = 0; lane < 64; ++lane) stage_c<G>(L, lane, mup.data(), coef.data());
  if constexpr (G::THREE)
    for (int lane = 0; lane < 64; ++lane) stage_b<G, 1>(L, lane, tw.data());
  for (int lane = 0; lane < 64; ++lane) stage_a<G, 1>(L, lane, tw.data());
  double err = 0.0;
  for (int l = 0; l < G::LPW; ++l) {
    std::vector<cld> X = dft(x[l], w, false);
    for (int k = 0; k < N; ++k) X[k] *= cld(0, -(long double)mu[k] * coef[l]);
    const std::vector<cld> y = dft(X, w, true);
    long double num = 0, den = 0;
    for (int n = 0; n < N; ++n) {
      const cx<double> v = lds[(size_t)l * G::LSZ + G::pos(n)];
      num += std::norm(cld(v.re, v.im) - y[n]);
      den += std::norm(y[n]);
    }
    err = std::max(err, (double)std::sqrt(num / den));
  }
  // two transforms at the codelets' 4e-16 (1 + log2 N), and four twiddle steps
  // whose powers are up to log2 of the factor products deep at 2.5e-16 each
  const double lg = std::log2((double)N), tol = 8e-16 * (1 + lg) + 5e-16 * (2 + lg);
  g_worst = std::max(g_worst, err);
  if (!ok || !(err <= tol)) {
    std::printf("FAIL N=%d = %d x %d (%d x %d) positions %d err %.3e tol %.1e\n", N, N1, M, G::N2, G::N3, (int)ok, err, tol);
    ++g_fail;
  }
}

int main() {
  int ncase = 0;
#define SPLIT(N1, M) check<N1, M>(), ++ncase;
#include "line_splits.inc"
  std::printf("cases %d failures %d worst %.3e\n", ncase, g_fail, g_worst);
  return g_fail ? 1 : 0;
}
