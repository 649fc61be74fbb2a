// Line passes with register codelets: split table, table orders and launch
// code for all extended lengths (instantiated here and in line4_extra*.hip,
// line4_long*.hip, which compile in parallel).
#include "line4_impl.h"

namespace rte {

// N_p = N1 x M; M is one or two stages (inner_n2)
bool fourstep_split(int Np, int* n1, int* n2) {
  switch (Np) {
    case 45: *n1 = 5; *n2 = 9; return true;
    case 48: *n1 = 3; *n2 = 16; return true;
    case 50: *n1 = 5; *n2 = 10; return true;
    case 54: *n1 = 6; *n2 = 9; return true;
    case 60: *n1 = 6; *n2 = 10; return true;
    case 64: *n1 = 4; *n2 = 16; return true;
    case 72: *n1 = 6; *n2 = 12; return true;
    case 75: *n1 = 3; *n2 = 25; return true;
    case 80: *n1 = 8; *n2 = 10; return true;
    case 81: *n1 = 9; *n2 = 9; return true;
    case 90: *n1 = 3; *n2 = 30; return true;
    case 96: *n1 = 3; *n2 = 32; return true;
    case 100: *n1 = 4; *n2 = 25; return true;
    case 108: *n1 = 9; *n2 = 12; return true;
    case 120: *n1 = 10; *n2 = 12; return true;
    case 125: *n1 = 5; *n2 = 25; return true;
    case 128: *n1 = 4; *n2 = 32; return true;
    case 135: *n1 = 9; *n2 = 15; return true;
    case 144: *n1 = 12; *n2 = 12; return true;
    case 150: *n1 = 10; *n2 = 15; return true;
    case 160: *n1 = 10; *n2 = 16; return true;
    case 162: *n1 = 3; *n2 = 54; return true;
    case 180: *n1 = 12; *n2 = 15; return true;
    case 192: *n1 = 12; *n2 = 16; return true;
    case 200: *n1 = 20; *n2 = 10; return true;
    case 216: *n1 = 8; *n2 = 27; return true;
    case 225: *n1 = 15; *n2 = 15; return true;
    case 240: *n1 = 16; *n2 = 15; return true;
    case 243: *n1 = 3; *n2 = 81; return true;
    case 250: *n1 = 10; *n2 = 25; return true;
    case 256: *n1 = 16; *n2 = 16; return true;
    case 270: *n1 = 3; *n2 = 90; return true;
    case 288: *n1 = 6; *n2 = 48; return true;
    case 300: *n1 = 6; *n2 = 50; return true;
    case 320: *n1 = 5; *n2 = 64; return true;
    case 324: *n1 = 6; *n2 = 54; return true;
    case 360: *n1 = 8; *n2 = 45; return true;
    case 375: *n1 = 15; *n2 = 25; return true;
    case 384: *n1 = 6; *n2 = 64; return true;
    case 400: *n1 = 8; *n2 = 50; return true;
    case 405: *n1 = 5; *n2 = 81; return true;
    case 432: *n1 = 8; *n2 = 54; return true;
    case 450: *n1 = 5; *n2 = 90; return true;
    case 480: *n1 = 8; *n2 = 60; return true;
    case 486: *n1 = 9; *n2 = 54; return true;
    case 500: *n1 = 10; *n2 = 50; return true;
    case 512: *n1 = 8; *n2 = 64; return true;
    case 540: *n1 = 5; *n2 = 108; return true;
    case 576: *n1 = 24; *n2 = 24; return true;
    case 600: *n1 = 12; *n2 = 50; return true;
    case 625: *n1 = 25; *n2 = 25; return true;
    case 640: *n1 = 10; *n2 = 64; return true;
    case 648: *n1 = 12; *n2 = 54; return true;
    case 675: *n1 = 15; *n2 = 45; return true;
    case 720: *n1 = 5; *n2 = 144; return true;
    case 729: *n1 = 27; *n2 = 27; return true;
    case 750: *n1 = 10; *n2 = 75; return true;
    case 768: *n1 = 12; *n2 = 64; return true;
    case 800: *n1 = 32; *n2 = 25; return true;
    case 810: *n1 = 18; *n2 = 45; return true;
    case 864: *n1 = 6; *n2 = 144; return true;
    case 900: *n1 = 4; *n2 = 225; return true;
    case 960: *n1 = 15; *n2 = 64; return true;
    case 972: *n1 = 18; *n2 = 54; return true;
    case 1000: *n1 = 10; *n2 = 100; return true;
    case 1024: *n1 = 16; *n2 = 64; return true;
    case 1080: *n1 = 10; *n2 = 108; return true;
    case 1125: *n1 = 15; *n2 = 75; return true;
    case 1152: *n1 = 18; *n2 = 64; return true;
    case 1200: *n1 = 8; *n2 = 150; return true;
    default: return false;
  }
}

void line4_orders(int Np, std::vector<int>& mu, std::vector<int>& tw) {
  int n1 = 0, m = 0;
  mu.clear();
  tw.clear();
  if (fourstep_split(Np, &n1, &m)) split_orders(n1, m, mu, tw);
}

template <typename T, bool ADJ>
static hipError_t by_size(const Lines4Args<T>& a, int Np, int nq, hipStream_t s) {
  switch (Np) {
    case 90: return go_one<T, ADJ, 3, 30>(a, nq, s);
    case 160: return go_one<T, ADJ, 10, 16>(a, nq, s);
    case 288: return go_one<T, ADJ, 6, 48>(a, nq, s);
    case 540: return go_one<T, ADJ, 5, 108>(a, nq, s);
    default: {
      hipError_t e = lines4_extra0(a, Np, nq, ADJ, s);
      if (e == hipErrorNotSupported) e = lines4_extra1(a, Np, nq, ADJ, s);
      if (e == hipErrorNotSupported) e = lines4_extra2(a, Np, nq, ADJ, s);
      if (e == hipErrorNotSupported) e = lines4_extra3(a, Np, nq, ADJ, s);
      if (e == hipErrorNotSupported) e = lines4_long0(a, Np, nq, ADJ, s);
      if (e == hipErrorNotSupported) e = lines4_long1(a, Np, nq, ADJ, s);
      return e;
    }
  }
}

template <typename T>
static hipError_t launch4_t(const Plan& p, const LineLaunch& L, hipStream_t s) {
  Lines4Args<T> a;
  a.in = static_cast<const T*>(L.in);
  a.out[0] = static_cast<T*>(L.out_x);
  a.out[1] = static_cast<T*>(L.out_y);
  for (int k = 0; k < 2; ++k) {
    const FcPlanDev& fc = k ? p.fcy : p.fcx;
    Lines4Dir& D = a.dir[k];
    D.coef = k ? p.dev.eta : p.dev.xi;
    D.mu = fc.mup;
    D.Mx = fc.Mx;
    D.MxT = fc.MxT;
    D.tw = reinterpret_cast<const double2*>(fc.tw4);
    D.Np = fc.Np;
    D.n = fc.n;
    D.CE = fc.C + fc.E;
    D.nlines = (int)(k ? p.nx : p.ny);
    const int np = (D.nlines + 1) / 2;
    D.npe = np + (np & 1);
    D.along_x = k == 0;
  }
  const bool dx = (L.dirs & 1) != 0, dy = (L.dirs & 2) != 0;
  const FcPlanDev& fc = dx ? p.fcx : p.fcy;
  a.d = fc.d;
  a.rows = p.rows;
  a.grp_stride = p.grp_stride;
  a.inst_stride = p.inst_stride;
  a.G = (int)p.G;
  // FP32 columns leave in 32-byte pieces per point, which a large plan's passes
  // rather let the L2 merge with the neighbouring pair's: at more than 64 MiB a
  // source, plain stores give 640 x 640 x 64 160 us a pass against 175,
  // 1025 x 1025 x 64 448 against 493; below (385 x 385 x 64, four sources 234
  // against 221) and in FP64 (700 x 700 x 64 240 against 207) the hint is better
  const bool merge_y = p.dtype == RTE_F32 && p.inst_stride * (int64_t)sizeof(float) > kStreamNtBytes;
  a.nt_out = p.line_nt ? (merge_y ? 1 : 3) : 0;
  a.first = dx ? 0 : 1;
  a.units_first = a.dir[a.first].npe;
  a.nunits = a.units_first + ((dx && dy) ? a.dir[1].npe : 0);
  if (dx && dy && p.fcx.Np != p.fcy.Np) return lines4_mixed(a, (int)p.cnq, L.mode == LINE_ADJ, s);
  return L.mode == LINE_ADJ ? by_size<T, true>(a, fc.Np, (int)p.cnq, s) : by_size<T, false>(a, fc.Np, (int)p.cnq, s);
}

hipError_t launch_lines4(const Plan& p, const LineLaunch& L, hipStream_t s) {
  if (p.dtype == RTE_F64) return launch4_t<double>(p, L, s);
  return launch4_t<float>(p, L, s);
}

}  // namespace rte
