// Host generation of every dense matrix the box code applies (built once per process).
//
// Near tables (the volume quadrature of adjacent leaves, Sec. 4.2 eq. (vbulk) restricted to a
// pair of touching leaves) in target half-widths:
//     T_r[m,k] = -(1/2pi) [ ln(rho_r) W_k + I_k((xi_m - d_r)/rho_r) ],
//     I_k(x0)  = int_{[-1,1]^2} ln|y - x0| l_k(y) dy,
// computed here independently of any other code path:
//   * x0 inside the square (self relation): four triangles with apex x0 in Duffy coordinates
//     y = x0 + u (P0 - x0 + v (P1 - P0)); ln|y - x0| = ln u + ln|E(v)|. The u integral of
//     u (ln u + c) poly(u) (degree <= 31) is exact with 32 Gauss-Legendre nodes and
//     product-integration weights for ln u (Legendre moments int_0^1 ln(u) P*_n(u) du =
//     (-1)^(n+1)/(n(n+1))); the v integral uses Gauss panels refined until the complex
//     singularity of ln|E(v)| lies outside the Bernstein ellipse of parameter 4.
//   * x0 outside (all other relations): a tensor mesh graded geometrically towards the
//     nearest boundary point p, breakpoints p +- h 2^(k-1) (h = |x0 - p|), 24-point Gauss in
//     each direction, applied as Lx diag(w G) Ly^T.
// D4 symmetry: only the 7 relation classes are integrated; the other 26 tables are the same
// numbers with rows and columns permuted alike.
//
// Far-field matrices follow the Greengard-Rokhlin expansions in scaled form (multipole
// phi(z) = a_0 ln(z-c) + sum a_n (s/(z-c))^n, local psi(z) = sum b_l ((z-c)/s)^l, complex
// z = x + iy, G = -(1/2pi) Re ln z), converted to real matrices on interleaved (Re, Im).
#include <algorithm>
#include <atomic>
#include <stdexcept>
#include <cmath>
#include <complex>
#include <map>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <mutex>
#include <string>
#include <thread>

#include "plan.hpp"
#include "moments.hpp"

namespace vp {

using cd = std::complex<double>;
static const double kInv2Pi = 1.0 / (2.0 * M_PI);

// ---------------------------------------------------------------- 1D rules and basis
static void gauss_legendre(int n, std::vector<double>& x, std::vector<double>& w) {
  x.assign(n, 0.0);
  w.assign(n, 0.0);
  for (int i = 0; i < n; ++i) {
    double z = std::cos(M_PI * (i + 0.75) / (n + 0.5)), dp = 1.0;
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = z;
      for (int k = 2; k <= n; ++k) {
        double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      dp = n * (z * p1 - p0) / (z * z - 1.0);
      double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-17) break;
    }
    double p0 = 1.0, p1 = z;
    for (int k = 2; k <= n; ++k) {
      double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    dp = n * (z * p1 - p0) / (z * z - 1.0);
    x[n - 1 - i] = z;
    w[n - 1 - i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

struct Basis {
  double t[kP], lam[kP], w[kP], W[kNP];
  Basis() {
    for (int i = 0; i < kP; ++i) t[i] = -std::cos((2.0 * i + 1.0) * M_PI / (2.0 * kP));
    for (int i = 0; i < kP; ++i) {
      double v = 1.0;
      for (int j = 0; j < kP; ++j)
        if (j != i) v *= (t[i] - t[j]);
      lam[i] = 1.0 / v;
    }
    // Fejer first-rule weights (interpolatory weights of these points)
    for (int i = 0; i < kP; ++i) {
      double th = std::acos(t[i]), s = 0.0;
      for (int j = 1; j <= kP / 2; ++j) s += std::cos(2.0 * j * th) / (4.0 * j * j - 1.0);
      w[i] = (2.0 / kP) * (1.0 - 2.0 * s);
    }
    for (int j = 0; j < kP; ++j)
      for (int i = 0; i < kP; ++i) W[j * kP + i] = w[i] * w[j];
  }
  void lagrange(double x, double* L) const {
    for (int i = 0; i < kP; ++i)
      if (x == t[i]) {
        for (int j = 0; j < kP; ++j) L[j] = (i == j) ? 1.0 : 0.0;
        return;
      }
    double s = 0.0;
    for (int i = 0; i < kP; ++i) {
      L[i] = lam[i] / (x - t[i]);
      s += L[i];
    }
    for (int i = 0; i < kP; ++i) L[i] /= s;
  }
};
static const Basis& basis() { static const Basis b; return b; }

// ---------------------------------------------------------------- near: x0 inside
struct LogRule {
  std::vector<double> u, w, wl;  // 32 GL nodes on [0,1], weights, ln-product weights
  LogRule() {
    std::vector<double> x, ww;
    gauss_legendre(32, x, ww);
    u.resize(32); w.resize(32); wl.resize(32);
    for (int j = 0; j < 32; ++j) { u[j] = 0.5 * (x[j] + 1.0); w[j] = 0.5 * ww[j]; }
    for (int j = 0; j < 32; ++j) {
      // shifted Legendre P*_n(u) = P_n(2u - 1)
      double z = 2.0 * u[j] - 1.0, p0 = 1.0, p1 = z, s = -1.0;  // n = 0 term: (2*0+1) P0 M0 = -1
      s += 3.0 * p1 * 0.5;  // n = 1: M1 = +1/2
      for (int n = 2; n < 32; ++n) {
        double p2 = ((2.0 * n - 1.0) * z * p1 - (n - 1.0) * p0) / n;
        p0 = p1;
        p1 = p2;
        double Mn = ((n + 1) % 2 == 0 ? 1.0 : -1.0) / (double(n) * (n + 1));
        s += (2.0 * n + 1.0) * p1 * Mn;
      }
      wl[j] = w[j] * s;
    }
  }
};

static double bernstein_rho(cd z, double c, double hl) {
  cd w = (z - c) / hl;
  cd s = std::sqrt(w - 1.0) * std::sqrt(w + 1.0);
  return std::max(std::abs(w + s), std::abs(w - s));
}

static void accumulate_point(const Basis& B, double y1, double y2, double wt, double* I) {
  double Lx[kP], Ly[kP];
  B.lagrange(y1, Lx);
  B.lagrange(y2, Ly);
  for (int j = 0; j < kP; ++j) {
    double a = wt * Ly[j];
    double* row = I + j * kP;
    for (int i = 0; i < kP; ++i) row[i] += a * Lx[i];
  }
}

static void inside_triangle(const Basis& B, const LogRule& R, const std::vector<double>& gx,
                            const std::vector<double>& gw, double x0, double y0, double p0x, double p0y,
                            double p1x, double p1y, double* I) {
  double e0x = p0x - x0, e0y = p0y - y0, dx = p1x - p0x, dy = p1y - p0y;
  double twoA = std::fabs(e0x * dy - e0y * dx);
  if (twoA < 1e-300) return;
  double L2 = dx * dx + dy * dy, L = std::sqrt(L2);
  double vf = -(e0x * dx + e0y * dy) / L2, hv = twoA / L / L;  // singularities at vf +- i hv
  cd zs(vf, hv);
  std::vector<std::pair<double, double>> stack{{0.0, 1.0}}, panels;
  while (!stack.empty()) {
    auto pr = stack.back();
    stack.pop_back();
    double c = 0.5 * (pr.first + pr.second), hl = 0.5 * (pr.second - pr.first);
    if (bernstein_rho(zs, c, hl) >= 4.0 || hl < 1e-12) panels.push_back(pr);
    else { stack.push_back({pr.first, c}); stack.push_back({c, pr.second}); }
  }
  for (auto& pr : panels) {
    double c = 0.5 * (pr.first + pr.second), hl = 0.5 * (pr.second - pr.first);
    for (size_t q = 0; q < gx.size(); ++q) {
      double v = c + hl * gx[q], wv = hl * gw[q];
      double ex = e0x + v * dx, ey = e0y + v * dy;
      double lnE = 0.5 * std::log(ex * ex + ey * ey);
      for (int j = 0; j < 32; ++j) {
        double u = R.u[j];
        double wt = twoA * wv * u * (R.wl[j] + lnE * R.w[j]);
        accumulate_point(B, x0 + u * ex, y0 + u * ey, wt, I);
      }
    }
  }
}

// ---------------------------------------------------------------- near: x0 outside
static std::vector<double> graded_breaks(double p, double h) {
  std::vector<double> b{-1.0, 1.0};
  for (double d = 0.5 * h; d < 2.0; d *= 2.0) {
    if (p - d > -1.0) b.push_back(p - d);
    if (p + d < 1.0) b.push_back(p + d);
  }
  std::sort(b.begin(), b.end());
  b.erase(std::unique(b.begin(), b.end(), [](double a, double c) { return std::fabs(a - c) < 1e-15; }), b.end());
  return b;
}

static void outside_graded(const Basis& B, double x0, double y0, double* I) {
  double px = std::min(1.0, std::max(-1.0, x0)), py = std::min(1.0, std::max(-1.0, y0));
  double h = std::hypot(x0 - px, y0 - py);
  std::vector<double> bx = graded_breaks(px, h), by = graded_breaks(py, h);
  static thread_local std::vector<double> gx, gw;
  if (gx.empty()) gauss_legendre(24, gx, gw);
  const int n = 24;
  double Lx[24][kP], Ly[24][kP], G[24][24], C[kP][24];
  for (size_t a = 0; a + 1 < bx.size(); ++a) {
    double cx = 0.5 * (bx[a] + bx[a + 1]), hx = 0.5 * (bx[a + 1] - bx[a]);
    for (int q = 0; q < n; ++q) B.lagrange(cx + hx * gx[q], Lx[q]);
    for (size_t b = 0; b + 1 < by.size(); ++b) {
      double cy = 0.5 * (by[b] + by[b + 1]), hy = 0.5 * (by[b + 1] - by[b]);
      for (int q = 0; q < n; ++q) B.lagrange(cy + hy * gx[q], Ly[q]);
      for (int qa = 0; qa < n; ++qa) {
        double ddx = cx + hx * gx[qa] - x0;
        for (int qb = 0; qb < n; ++qb) {
          double ddy = cy + hy * gx[qb] - y0;
          G[qa][qb] = 0.5 * std::log(ddx * ddx + ddy * ddy) * gw[qa] * gw[qb] * hx * hy;
        }
      }
      for (int i = 0; i < kP; ++i)
        for (int qb = 0; qb < n; ++qb) {
          double s = 0.0;
          for (int qa = 0; qa < n; ++qa) s += Lx[qa][i] * G[qa][qb];
          C[i][qb] = s;
        }
      for (int j = 0; j < kP; ++j)
        for (int i = 0; i < kP; ++i) {
          double s = 0.0;
          for (int qb = 0; qb < n; ++qb) s += C[i][qb] * Ly[qb][j];
          I[j * kP + i] += s;
        }
    }
  }
}

static void logint(double x0, double y0, double* I) {
  const Basis& B = basis();
  std::memset(I, 0, sizeof(double) * kNP);
  if (std::fabs(x0) < 1.0 && std::fabs(y0) < 1.0) {
    static const LogRule R;
    static thread_local std::vector<double> gx, gw;
    if (gx.empty()) gauss_legendre(32, gx, gw);
    const double P[5][2] = {{-1, -1}, {1, -1}, {1, 1}, {-1, 1}, {-1, -1}};
    for (int e = 0; e < 4; ++e) inside_triangle(B, R, gx, gw, x0, y0, P[e][0], P[e][1], P[e + 1][0], P[e + 1][1], I);
  } else {
    outside_graded(B, x0, y0, I);
  }
}

// ---------------------------------------------------------------- moments at an arbitrary point
// For xi = (x0, y0) anywhere: I_k = int log|xi - eta| l_k(eta) d eta and (Ix_k, Iy_k) =
// int (xi - eta) / |xi - eta|^2 l_k(eta) d eta over the reference square (the gradient of I in
// xi). The square is refined towards xi as a quadtree: a square at distance >= its side from
// xi takes a 24 x 24 tensor Gauss rule (the kernels are analytic there); a square of
// half-width <= 1/32 whose closure holds xi takes four
// polar-Duffy triangles with apex xi (a 16-point log-product rule in the radial variable, exact
// to degree 15, which on so small a square leaves terms of relative size 32^-16; adaptive
// 12-point panels along the far edge, as for the tables). The gradient kernel times the Duffy
// Jacobian u is smooth in u and takes the plain Gauss weights.
struct LogRule16 {
  double u[16], w[16], wl[16];
  LogRule16() {
    std::vector<double> x, ww;
    gauss_legendre(16, x, ww);
    for (int j = 0; j < 16; ++j) { u[j] = 0.5 * (x[j] + 1.0); w[j] = 0.5 * ww[j]; }
    for (int j = 0; j < 16; ++j) {  // interpolatory weights of int_0^1 ln(u) p(u) du (shifted Legendre moments)
      double z = 2.0 * u[j] - 1.0, p0 = 1.0, p1 = z, sum = -1.0 + 3.0 * p1 * 0.5;
      for (int n = 2; n < 16; ++n) {
        double p2 = ((2.0 * n - 1.0) * z * p1 - (n - 1.0) * p0) / n;
        p0 = p1;
        p1 = p2;
        sum += (2.0 * n + 1.0) * p1 * (((n + 1) % 2 == 0 ? 1.0 : -1.0) / (double(n) * (n + 1)));
      }
      wl[j] = w[j] * sum;
    }
  }
};

constexpr int kNT = 24;  // tensor rule of the accepted squares
struct PointRules {
  std::vector<double> gtx, gtw, g12x, g12w;
  LogRule16 R;
  PointRules() {
    gauss_legendre(kNT, gtx, gtw);
    gauss_legendre(12, g12x, g12w);
  }
};


void moment_rules(MomentRules* R) {
  static const PointRules Q;
  const Basis& B = basis();
  for (int i = 0; i < kP; ++i) { R->t[i] = B.t[i]; R->lam[i] = B.lam[i]; R->w[i] = B.w[i]; }
  for (int a = 0; a < kNT; ++a) { R->gx[a] = Q.gtx[size_t(a)]; R->gw[a] = Q.gtw[size_t(a)]; }
  for (int a = 0; a < 12; ++a) { R->px[a] = Q.g12x[size_t(a)]; R->pw[a] = Q.g12w[size_t(a)]; }
  for (int j = 0; j < 16; ++j) { R->u[j] = Q.R.u[j]; R->uw[j] = Q.R.w[j]; R->ul[j] = Q.R.wl[j]; }
}

// D4 element g: (x, y) -> (sx * (swap ? y : x), sy * (swap ? x : y))
struct D4 { int sx, sy, swap; };
static void apply_d4(const D4& g, double x, double y, double& ox, double& oy) {
  double a = g.swap ? y : x, b = g.swap ? x : y;
  ox = g.sx * a;
  oy = g.sy * b;
}
static int node_map(const D4& g, int m) {
  int i = m % kP, j = m / kP;
  int a = g.swap ? j : i, b = g.swap ? i : j;
  int ni = g.sx > 0 ? a : kP - 1 - a, nj = g.sy > 0 ? b : kP - 1 - b;
  return nj * kP + ni;
}

static std::vector<std::vector<double>> near_tables_compute() {
  const auto& NO = near_offsets();
  const Basis& B = basis();
  const int reps[7][3] = {{0, 0, 2}, {4, 0, 2}, {4, 4, 2}, {3, 1, 1}, {3, 3, 1}, {6, 2, 4}, {6, 6, 4}};  // (2dx, 2dy, 2rho)
  std::vector<std::vector<double>> rep(7, std::vector<double>(kNP * kNP));
  std::vector<std::pair<int, int>> jobs;
  for (int r = 0; r < 7; ++r)
    for (int m = 0; m < kNP; ++m) jobs.push_back({r, m});
  unsigned nth = std::max(1u, std::min(32u, std::thread::hardware_concurrency()));
  std::vector<std::thread> th;
  std::atomic<size_t> next{0};
  for (unsigned t = 0; t < nth; ++t)
    th.emplace_back([&]() {
      double I[kNP];
      for (;;) {
        size_t id = next.fetch_add(1);
        if (id >= jobs.size()) break;
        int r = jobs[id].first, m = jobs[id].second;
        double dx = 0.5 * reps[r][0], dy = 0.5 * reps[r][1], rho = 0.5 * reps[r][2];
        double xm = B.t[m % kP], ym = B.t[m / kP];
        logint((xm - dx) / rho, (ym - dy) / rho, I);
        double lr = std::log(rho);
        for (int k = 0; k < kNP; ++k) rep[r][size_t(m) * kNP + k] = -kInv2Pi * (lr * B.W[k] + I[k]);
      }
    });
  for (auto& t : th) t.join();
  std::vector<std::vector<double>> out(NO.size());
  const D4 G[8] = {{1, 1, 0}, {-1, 1, 0}, {1, -1, 0}, {-1, -1, 0}, {1, 1, 1}, {-1, 1, 1}, {1, -1, 1}, {-1, -1, 1}};
  for (size_t r = 0; r < NO.size(); ++r) {
    bool done = false;
    for (int q = 0; q < 7 && !done; ++q) {
      double rdx = 0.5 * reps[q][0], rdy = 0.5 * reps[q][1], rrho = 0.5 * reps[q][2];
      if (std::fabs(rrho - NO[r].rho) > 1e-12) continue;
      for (const D4& g : G) {
        double ox, oy;
        apply_d4(g, rdx, rdy, ox, oy);
        if (std::fabs(ox - NO[r].dx) < 1e-12 && std::fabs(oy - NO[r].dy) < 1e-12) {
          out[r].assign(kNP * kNP, 0.0);
          for (int m = 0; m < kNP; ++m)
            for (int k = 0; k < kNP; ++k) out[r][size_t(node_map(g, m)) * kNP + node_map(g, k)] = rep[q][size_t(m) * kNP + k];
          done = true;
          break;
        }
      }
    }
    if (!done) throw std::runtime_error("no D4 representative for a near relation");
  }
  return out;
}

// ---------------------------------------------------------------- cache
static std::string g_cache_dir;
static std::mutex g_cache_mu;
void set_table_cache_dir(const char* dir) {
  std::lock_guard<std::mutex> lk(g_cache_mu);
  g_cache_dir = dir ? dir : "";
}

static uint64_t fnv1a(const double* d, size_t n) {
  uint64_t h = 1469598103934665603ull;
  const unsigned char* p = reinterpret_cast<const unsigned char*>(d);
  for (size_t i = 0; i < n * sizeof(double); ++i) { h ^= p[i]; h *= 1099511628211ull; }
  return h;
}

static const char kMagic[8] = {'V', 'P', 'N', 'E', 'A', 'R', '0', '1'};

static bool cache_load(const std::string& path, std::vector<std::vector<double>>& out) {
  std::ifstream f(path, std::ios::binary);
  if (!f) return false;
  char mg[8];
  int32_t hdr[4];
  uint64_t hash;
  f.read(mg, 8);
  f.read(reinterpret_cast<char*>(hdr), sizeof(hdr));
  f.read(reinterpret_cast<char*>(&hash), 8);
  if (!f || std::memcmp(mg, kMagic, 8) != 0 || hdr[0] != kP || hdr[1] != 33 || hdr[2] != kNP) return false;
  std::vector<double> all(size_t(33) * kNP * kNP);
  f.read(reinterpret_cast<char*>(all.data()), all.size() * sizeof(double));
  if (!f || fnv1a(all.data(), all.size()) != hash) return false;
  out.assign(33, std::vector<double>());
  for (int r = 0; r < 33; ++r) out[r].assign(all.begin() + size_t(r) * kNP * kNP, all.begin() + size_t(r + 1) * kNP * kNP);
  return true;
}

static void cache_store(const std::string& path, const std::vector<std::vector<double>>& t) {
  std::vector<double> all;
  for (auto& v : t) all.insert(all.end(), v.begin(), v.end());
  int32_t hdr[4] = {kP, 33, kNP, 0};
  uint64_t hash = fnv1a(all.data(), all.size());
  std::string tmp = path + ".tmp";
  std::ofstream f(tmp, std::ios::binary);
  if (!f) return;
  f.write(kMagic, 8);
  f.write(reinterpret_cast<const char*>(hdr), sizeof(hdr));
  f.write(reinterpret_cast<const char*>(&hash), 8);
  f.write(reinterpret_cast<const char*>(all.data()), all.size() * sizeof(double));
  f.close();
  if (f) std::rename(tmp.c_str(), path.c_str());
}

// ---------------------------------------------------------------- far-field matrices
static void real_from_linear(const std::vector<cd>& K, int rows, int cols, std::vector<double>& R) {
  // complex-linear map on interleaved (Re, Im)
  R.assign(size_t(2 * rows) * (2 * cols), 0.0);
  for (int l = 0; l < rows; ++l)
    for (int k = 0; k < cols; ++k) {
      cd z = K[size_t(l) * cols + k];
      R[size_t(2 * l) * (2 * cols) + 2 * k] = z.real();
      R[size_t(2 * l) * (2 * cols) + 2 * k + 1] = -z.imag();
      R[size_t(2 * l + 1) * (2 * cols) + 2 * k] = z.imag();
      R[size_t(2 * l + 1) * (2 * cols) + 2 * k + 1] = z.real();
    }
}
static void real_from_realin(const std::vector<cd>& S, int rows, int cols, std::vector<double>& R) {
  // real input (cols) -> complex output (rows)
  R.assign(size_t(2 * rows) * cols, 0.0);
  for (int l = 0; l < rows; ++l)
    for (int k = 0; k < cols; ++k) {
      R[size_t(2 * l) * cols + k] = S[size_t(l) * cols + k].real();
      R[size_t(2 * l + 1) * cols + k] = S[size_t(l) * cols + k].imag();
    }
}
static void real_from_realout(const std::vector<cd>& L, int rows, int cols, std::vector<double>& R) {
  // complex input (cols) -> real output Re(L x) (rows)
  R.assign(size_t(rows) * (2 * cols), 0.0);
  for (int m = 0; m < rows; ++m)
    for (int l = 0; l < cols; ++l) {
      R[size_t(m) * (2 * cols) + 2 * l] = L[size_t(m) * cols + l].real();
      R[size_t(m) * (2 * cols) + 2 * l + 1] = -L[size_t(m) * cols + l].imag();
    }
}
static double binom(int n, int k) {
  if (k < 0 || k > n) return 0.0;
  return std::exp(std::lgamma(n + 1.0) - std::lgamma(k + 1.0) - std::lgamma(n - k + 1.0));
}
static double binom_exact(int n, int k) {
  // Pascal recursion in double: exact below 2^53, correctly rounded-ish above
  static std::vector<std::vector<double>> T;
  if (T.empty()) {
    T.assign(2 * kTerms + 2, std::vector<double>(2 * kTerms + 2, 0.0));
    for (int a = 0; a < int(T.size()); ++a) {
      T[a][0] = 1.0;
      for (int b = 1; b <= a; ++b) T[a][b] = T[a - 1][b - 1] + (b <= a - 1 ? T[a - 1][b] : 0.0);
    }
  }
  if (k < 0 || k > n || n >= int(T.size())) return binom(n, k);
  return T[n][k];
}

// integrals over the reference square of l_k(eta) g(eta) with a tensor Gauss rule of n points
template <class F>
static std::vector<cd> quad_basis(int n, int nfun, F g) {
  std::vector<double> x, w;
  gauss_legendre(n, x, w);
  const Basis& B = basis();
  std::vector<std::vector<double>> L(n, std::vector<double>(kP));
  for (int a = 0; a < n; ++a) B.lagrange(x[a], L[a].data());
  std::vector<cd> out(size_t(nfun) * kNP, cd(0.0));
  std::vector<cd> G(size_t(n) * n);
  for (int f = 0; f < nfun; ++f) {
    for (int a = 0; a < n; ++a)
      for (int b = 0; b < n; ++b) G[size_t(a) * n + b] = w[a] * w[b] * g(f, cd(x[a], x[b]));
    for (int i = 0; i < kP; ++i) {
      std::vector<cd> Cb(n, cd(0.0));
      for (int b = 0; b < n; ++b)
        for (int a = 0; a < n; ++a) Cb[b] += L[a][i] * G[size_t(a) * n + b];
      for (int j = 0; j < kP; ++j) {
        cd s(0.0);
        for (int b = 0; b < n; ++b) s += Cb[b] * L[b][j];
        out[size_t(f) * kNP + j * kP + i] = s;
      }
    }
  }
  return out;
}

// the near tables: the same for every expansion order, computed (or read from the cache) once
static const std::vector<std::vector<double>>& near_tables() {
  static std::once_flag once;
  static std::vector<std::vector<double>>* T = nullptr;
  std::call_once(once, []() {
    T = new std::vector<std::vector<double>>();
    std::string path;
    {
      std::lock_guard<std::mutex> lk(g_cache_mu);
      if (!g_cache_dir.empty()) path = g_cache_dir + "/volpot_near_p16_v1.bin";
    }
    if (path.empty() || !cache_load(path, *T)) {
      *T = near_tables_compute();
      if (!path.empty()) cache_store(path, *T);
    }
  });
  return *T;
}

// T (n x n, row-major) ~= Q R with Q (n x k, orthonormal columns) and R (k x n): Householder QR
// with column pivoting (the column of largest remaining norm first), stopped after k columns;
// R's columns are returned in T's original order. The discarded part is the trailing block
// R[k:, k:] of the pivoted factorization.
static void pivoted_qr(const std::vector<double>& T, int n, int k, std::vector<double>& Qk, std::vector<double>& Rk) {
  std::vector<double> A(T);
  std::vector<int> perm(static_cast<size_t>(n));
  for (int c = 0; c < n; ++c) perm[size_t(c)] = c;
  std::vector<std::vector<double>> V(static_cast<size_t>(k));
  std::vector<double> beta(static_cast<size_t>(k), 0.0);
  for (int j = 0; j < k; ++j) {
    int p = j;
    double best = -1.0;
    for (int c = j; c < n; ++c) {
      double sq = 0.0;
      for (int i = j; i < n; ++i) sq += A[size_t(i) * n + c] * A[size_t(i) * n + c];
      if (sq > best) { best = sq; p = c; }
    }
    if (p != j) {
      for (int i = 0; i < n; ++i) std::swap(A[size_t(i) * n + j], A[size_t(i) * n + p]);
      std::swap(perm[size_t(j)], perm[size_t(p)]);
    }
    std::vector<double>& v = V[size_t(j)];
    v.assign(size_t(n - j), 0.0);
    double nrm = 0.0;
    for (int i = j; i < n; ++i) { v[size_t(i - j)] = A[size_t(i) * n + j]; nrm += v[size_t(i - j)] * v[size_t(i - j)]; }
    nrm = std::sqrt(nrm);
    const double alpha = v[0] >= 0.0 ? -nrm : nrm;
    v[0] -= alpha;
    double vv = 0.0;
    for (double x : v) vv += x * x;
    beta[size_t(j)] = vv > 0.0 ? 2.0 / vv : 0.0;
    for (int c = j; c < n; ++c) {  // A[j:, c] -= beta v (v . A[j:, c])
      double d = 0.0;
      for (int i = j; i < n; ++i) d += v[size_t(i - j)] * A[size_t(i) * n + c];
      d *= beta[size_t(j)];
      for (int i = j; i < n; ++i) A[size_t(i) * n + c] -= d * v[size_t(i - j)];
    }
  }
  Rk.assign(size_t(k) * n, 0.0);
  for (int i = 0; i < k; ++i)
    for (int c = i; c < n; ++c) Rk[size_t(i) * n + perm[size_t(c)]] = A[size_t(i) * n + c];
  Qk.assign(size_t(n) * k, 0.0);  // H_0 H_1 ... H_{k-1} applied to the first k unit vectors
  for (int c = 0; c < k; ++c) Qk[size_t(c) * k + c] = 1.0;
  for (int j = k - 1; j >= 0; --j) {
    const std::vector<double>& v = V[size_t(j)];
    for (int c = 0; c < k; ++c) {
      double d = 0.0;
      for (int i = j; i < n; ++i) d += v[size_t(i - j)] * Qk[size_t(i) * k + c];
      d *= beta[size_t(j)];
      for (int i = j; i < n; ++i) Qk[size_t(i) * k + c] -= d * v[size_t(i - j)];
    }
  }
}

// The low-rank factors of the 32 adjacent-leaf tables other than the self table, computed once
// (the near tables are the same for every expansion order).
struct NearFactors {
  std::vector<std::vector<double>> U, V;  // 32 each: 256 x k_r and k_r x 256
  std::vector<int> rank;                  // k_r
};
// Truncating a relation's factors after kNearRankLow columns is kept when the discarded part
// is below this fraction of the self table (Frobenius norms). For the 32 relations the
// truncation error is either at rounding level (about 3e-15 of it) or above 1e-11: the
// threshold sits between the two groups.
constexpr double kNearRankLowTol = 1e-13;
static const NearFactors& near_factors() {
  static std::once_flag once;
  static NearFactors* F = nullptr;
  std::call_once(once, []() {
    F = new NearFactors();
    const std::vector<std::vector<double>>& T = near_tables();
    F->U.resize(32);
    F->V.resize(32);
    F->rank.assign(32, kNearRank);
    double self2 = 0.0;
    for (double x : T[0]) self2 += x * x;
    std::vector<std::thread> th;
    for (int r = 1; r <= 32; ++r)
      th.emplace_back([&, r, self2]() {
        std::vector<double>& U = F->U[size_t(r - 1)];
        std::vector<double>& V = F->V[size_t(r - 1)];
        pivoted_qr(T[size_t(r)], kNP, kNearRank, U, V);
        const int k = kNearRankLow;
        double e2 = 0.0;  // || T_r - U_r[:, :k] V_r[:k, :] ||_F^2
        for (int i = 0; i < kNP; ++i)
          for (int j = 0; j < kNP; ++j) {
            double s = T[size_t(r)][size_t(i) * kNP + j];
            for (int c = 0; c < k; ++c) s -= U[size_t(i) * kNearRank + c] * V[size_t(c) * kNP + j];
            e2 += s * s;
          }
        if (e2 > kNearRankLowTol * kNearRankLowTol * self2) return;
        std::vector<double> Uk(size_t(kNP) * k);
        for (int i = 0; i < kNP; ++i)
          for (int c = 0; c < k; ++c) Uk[size_t(i) * k + c] = U[size_t(i) * kNearRank + c];
        U.swap(Uk);
        V.resize(size_t(k) * kNP);  // the first k rows
        F->rank[size_t(r - 1)] = k;
      });
    for (auto& t : th) t.join();
  });
  return *F;
}

// ---------------------------------------------------------------- compressed leaf form
// Tables of the compressed near field, in the parity basis of a leaf's 16 x 16 nodal values:
// index p 64 + 8 j + i (j, i < 8), p = px + 2 py, holds half of v[j][i] +- v[j][15 - i] +-
// v[15 - j][i] +- v[15 - j][15 - i], the signs of the mirrored values negative where the part is
// odd in x (px) or y (py). The transform is orthonormal; it splits every table that commutes with
// the two reflections (a leaf with itself, S2M, L2T, E and the target bases below) into one block
// per part.
static void to_parity(const double* v, int64_t stride, double* out) {
  for (int j = 0; j < 8; ++j)
    for (int i = 0; i < 8; ++i) {
      const double a = v[stride * (16 * j + i)], b = v[stride * (16 * j + 15 - i)];
      const double c = v[stride * (16 * (15 - j) + i)], d = v[stride * (16 * (15 - j) + 15 - i)];
      const double ab = a + b, am = a - b, cd_ = c + d, cm = c - d;
      out[8 * j + i] = 0.5 * (ab + cd_);
      out[64 + 8 * j + i] = 0.5 * (am + cm);
      out[128 + 8 * j + i] = 0.5 * (ab - cd_);
      out[192 + 8 * j + i] = 0.5 * (am - cm);
    }
}
// rows of A (m x 256), then columns of A (256 x n), to the parity basis
static std::vector<double> parity_rows(const std::vector<double>& A, int m) {
  std::vector<double> R(A.size());
  for (int i = 0; i < m; ++i) to_parity(A.data() + size_t(i) * kNP, 1, R.data() + size_t(i) * kNP);
  return R;
}
static std::vector<double> parity_cols(const std::vector<double>& A, int n) {
  std::vector<double> R(A.size());
  double col[kNP];
  for (int c = 0; c < n; ++c) {
    to_parity(A.data() + c, n, col);
    for (int i = 0; i < kNP; ++i) R[size_t(i) * n + c] = col[i];
  }
  return R;
}

// E: the 28 outgoing values of each part of a leaf's data. The potential of polynomial data of
// degree 15 outside the leaf vanishes exactly when the data is the Laplacian of a polynomial with
// a double zero on the boundary, (1 - x^2)^2 (1 - y^2)^2 q with q of degree 11: 6 x 6 of each
// part. E is an orthonormal basis of the complement of these (64 - 36 = 28), so every functional
// of the leaf's exterior field (the tables to other leaves, S2M, S2L) is T E^T E without loss.
// The 36 are evaluated and orthogonalised in extended precision: in double the second derivatives
// would leave 3e-14 of the self table's norm.
static void outgoing_basis(std::vector<double>& E) {  // 4 x 28 x 64
  typedef long double ld;
  const Basis& B = basis();
  ld ph[12][8], p2[12][8];  // phi_a = (1 - x^2)^2 T_a(x) and its second derivative at the first 8 nodes
  for (int i = 0; i < 8; ++i) {
    const ld x = B.t[i];
    ld T[12], T1[12], T2[12];
    T[0] = 1; T1[0] = 0; T2[0] = 0;
    T[1] = x; T1[1] = 1; T2[1] = 0;
    for (int a = 2; a < 12; ++a) {
      T[a] = 2 * x * T[a - 1] - T[a - 2];
      T1[a] = 2 * T[a - 1] + 2 * x * T1[a - 1] - T1[a - 2];
      T2[a] = 4 * T1[a - 1] + 2 * x * T2[a - 1] - T2[a - 2];
    }
    const ld g = (1 - x * x) * (1 - x * x), g1 = -4 * x * (1 - x * x), g2 = 12 * x * x - 4;
    for (int a = 0; a < 12; ++a) {
      ph[a][i] = g * T[a];
      p2[a][i] = g2 * T[a] + 2 * g1 * T1[a] + g * T2[a];
    }
  }
  E.assign(size_t(4) * kOut * 64, 0.0);
  for (int p = 0; p < 4; ++p) {
    // Gram-Schmidt, each vector twice: the 36 first, then the unit vectors, largest remainder first
    std::vector<std::vector<ld>> q;
    auto residual = [&](std::vector<ld>& v) {
      for (int twice = 0; twice < 2; ++twice)
        for (auto& u : q) {
          ld d = 0;
          for (int k = 0; k < 64; ++k) d += u[size_t(k)] * v[size_t(k)];
          for (int k = 0; k < 64; ++k) v[size_t(k)] -= d * u[size_t(k)];
        }
      ld n = 0;
      for (ld x : v) n += x * x;
      return std::sqrt(n);
    };
    auto push = [&](std::vector<ld> v, ld n) {
      for (ld& x : v) x /= n;
      q.push_back(std::move(v));
    };
    for (int b = p >> 1; b < 12; b += 2)
      for (int a = p & 1; a < 12; a += 2) {
        std::vector<ld> v(64);
        ld n0 = 0;
        for (int j = 0; j < 8; ++j)
          for (int i = 0; i < 8; ++i) {
            v[size_t(8 * j + i)] = p2[a][i] * ph[b][j] + ph[a][i] * p2[b][j];
            n0 += v[size_t(8 * j + i)] * v[size_t(8 * j + i)];
          }
        for (ld& x : v) x /= std::sqrt(n0);
        const ld n = residual(v);
        push(v, n);
      }
    for (int r = 0; r < kOut; ++r) {
      ld best = -1;
      std::vector<ld> bv;
      for (int k = 0; k < 64; ++k) {
        std::vector<ld> v(64, 0);
        v[size_t(k)] = 1;
        const ld n = residual(v);
        if (n > best) { best = n; bv = v; }
      }
      push(bv, best);
      for (int k = 0; k < 64; ++k) E[(size_t(p) * kOut + r) * 64 + k] = double(q.back()[size_t(k)]);
    }
  }
}

// A (m x 256, parity basis) times E^T: m x 112, columns 28 p + r
static std::vector<double> times_et(const std::vector<double>& A, int m, const std::vector<double>& E) {
  std::vector<double> R(size_t(m) * kOutAll);
  for (int i = 0; i < m; ++i)
    for (int p = 0; p < 4; ++p)
      for (int r = 0; r < kOut; ++r) {
        double s = 0.0;
        for (int k = 0; k < 64; ++k) s += A[size_t(i) * kNP + 64 * p + k] * E[(size_t(p) * kOut + r) * 64 + k];
        R[size_t(i) * kOutAll + kOut * p + r] = s;
      }
  return R;
}

// Orthonormal basis (m x k) of the k leading left singular vectors of A (m x n, columns), by
// pivoted Gram-Schmidt on the columns to 64 vectors and one-sided Jacobi on what it leaves.
static std::vector<double> leading_basis(const std::vector<std::vector<double>>& cols, int m, int k) {
  const int n = int(cols.size()), kq = std::min(64, m);
  std::vector<std::vector<double>> res(cols), Q, R;
  double b0 = 0.0;
  for (int r = 0; r < kq; ++r) {
    int best = -1;
    double bn = -1.0;
    for (int c = 0; c < n; ++c) {
      double s = 0.0;
      for (double x : res[size_t(c)]) s += x * x;
      if (s > bn) { bn = s; best = c; }
    }
    if (r == 0) b0 = bn;
    if (!(bn > 1e-32 * b0)) break;  // nothing but rounding is left
    std::vector<double> v(res[size_t(best)]);
    for (int pass = 0; pass < 3; ++pass) {  // against the earlier vectors again, and to unit length
      if (pass > 0)
        for (auto& u : Q) {
          double d = 0.0;
          for (int i = 0; i < m; ++i) d += u[size_t(i)] * v[size_t(i)];
          for (int i = 0; i < m; ++i) v[size_t(i)] -= d * u[size_t(i)];
        }
      double nv = 0.0;
      for (double x : v) nv += x * x;
      nv = std::sqrt(nv);
      for (double& x : v) x /= nv;
    }
    // this vector's row of Q^T A, from what the earlier ones left of the columns: its small entries
    // keep their digits
    R.emplace_back(size_t(n), 0.0);
    for (int c = 0; c < n; ++c) {
      auto& w = res[size_t(c)];
      double d = 0.0;
      for (int i = 0; i < m; ++i) d += v[size_t(i)] * w[size_t(i)];
      for (int i = 0; i < m; ++i) w[size_t(i)] -= d * v[size_t(i)];
      R.back()[size_t(c)] = d;
    }
    Q.push_back(std::move(v));
  }
  const int q = int(Q.size());
  // Jacobi rotations of R's rows, the same rotations of Q's vectors
  for (int sweep = 0; sweep < 30; ++sweep) {
    double worst = 0.0;
    for (int a = 0; a + 1 < q; ++a)
      for (int b = a + 1; b < q; ++b) {
        double aa = 0, bb = 0, ab = 0;
        for (int c = 0; c < n; ++c) {
          aa += R[size_t(a)][size_t(c)] * R[size_t(a)][size_t(c)];
          bb += R[size_t(b)][size_t(c)] * R[size_t(b)][size_t(c)];
          ab += R[size_t(a)][size_t(c)] * R[size_t(b)][size_t(c)];
        }
        if (ab == 0.0) continue;
        worst = std::max(worst, std::fabs(ab) / std::sqrt(aa * bb));
        const double th = (bb - aa) / (2.0 * ab);
        const double t = (th >= 0.0 ? 1.0 : -1.0) / (std::fabs(th) + std::sqrt(1.0 + th * th));
        const double cs = 1.0 / std::sqrt(1.0 + t * t), sn = t * cs;
        auto rot = [&](std::vector<double>& x, std::vector<double>& y) {
          for (size_t c = 0; c < x.size(); ++c) {
            const double u = x[c], w = y[c];
            x[c] = cs * u - sn * w;
            y[c] = sn * u + cs * w;
          }
        };
        rot(R[size_t(a)], R[size_t(b)]);
        rot(Q[size_t(a)], Q[size_t(b)]);
      }
    if (worst < 1e-13) break;
  }
  std::vector<std::pair<double, int>> ord;
  for (int a = 0; a < q; ++a) {
    double s = 0.0;
    for (double x : R[size_t(a)]) s += x * x;
    ord.push_back({-s, a});
  }
  std::sort(ord.begin(), ord.end());
  // the rotations leave the vectors orthonormal to about 1e-14 only: Gram-Schmidt, each twice, in
  // extended precision
  std::vector<double> U(size_t(m) * k, 0.0);
  std::vector<std::vector<long double>> X;
  for (int c = 0; c < std::min(k, q); ++c) {
    const auto& src = Q[size_t(ord[size_t(c)].second)];
    std::vector<long double> v(src.begin(), src.end());
    for (int pass = 0; pass < 2; ++pass)
      for (auto& u : X) {
        long double d = 0;
        for (int i = 0; i < m; ++i) d += u[size_t(i)] * v[size_t(i)];
        for (int i = 0; i < m; ++i) v[size_t(i)] -= d * u[size_t(i)];
      }
    long double nv = 0;
    for (long double x : v) nv += x * x;
    nv = std::sqrt(nv);
    for (long double& x : v) x /= nv;
    for (int i = 0; i < m; ++i) U[size_t(i) * k + c] = double(v[size_t(i)]);
    X.push_back(std::move(v));
  }
  return U;
}

// M2T of W offset r for Q complex terms, 256 x 2Q
static std::vector<double> m2t_table(int r, int Q) {
  const Basis& B = basis();
  const Offset& o = w_offsets()[size_t(r)];
  const cd d(o.dx, o.dy);
  std::vector<cd> Mt(size_t(kNP) * Q);
  for (int m = 0; m < kNP; ++m) {
    const cd z = cd(B.t[m % kP], B.t[m / kP]) - d;
    Mt[size_t(m) * Q] = -kInv2Pi * std::log(std::abs(z));
    for (int k = 1; k < Q; ++k) Mt[size_t(m) * Q + k] = -kInv2Pi * std::pow(o.rho, k) * std::pow(z, -k);
  }
  std::vector<double> R;
  real_from_realout(Mt, kNP, Q, R);
  return R;
}
// S2M for Q complex terms (c_n int l_k eta^n, c_0 = 1, c_n = -1/n), 2Q x 256
static std::vector<double> s2m_table(int Q) {
  auto S = quad_basis(40, Q, [](int n, cd e) { return n == 0 ? cd(1.0) : -std::pow(e, n) / double(n); });
  std::vector<double> R;
  real_from_realin(S, Q, kNP, R);
  return R;
}

// Boxes on a diagonal are a corner's; the others are the edge's of their larger coordinate, also where they
// lie wholly to the side of it (W boxes at (1.5, 2.5) and its images).
int near_dir(double dx, double dy, double rho) {
  const double ax = std::fabs(dx), ay = std::fabs(dy);
  if (std::max(ax, ay) < 1.0 + rho - 1e-9) return -1;  // overlaps the target
  if (std::fabs(ax - ay) < 1e-9) return 4 + (dx < 0) + 2 * (dy < 0);
  if (ax > ay) return dx > 0 ? 0 : 1;
  return dy > 0 ? 2 : 3;
}

// The bases of what a leaf receives through each of its four edges and four corners, and the
// tables of the 32 adjacent relations between them and E.
//   H_E (256 x 96): the potentials in the leaf of everything across its right edge: the same-size
//   neighbour, the finer and the coarser ones, and the W-list boxes beyond. 48 vectors even in y
//   (on the parts py = 0) and 48 odd ones. The other edges are its images: W mirrors x (the sign
//   of the parts px = 1), N swaps x and y, S mirrors N.
//   H_NE (256 x 48): the same across the upper right corner; NW, SE, SW mirror it.
// The bases are fitted to the adjacent leaves' tables alone, on data of unit length. What they leave of
// those (Frobenius norm, in that of the self table) is 1.2e-15 to 1.7e-15 across edges and 4e-15 to 6e-15
// across corners; the rank-64/48 factors of the same tables leave 1.7e-15 to 8e-15. W-list boxes need no
// vectors of their own: a coarser neighbour fills the same region, and of the field of a point charge
// anywhere in one (a W box may be refined further, so its multipoles are not those of a leaf's
// polynomial) they leave 1.7e-15 at most, at every expansion order. That holds for the edge that near_dir
// names: H_NE leaves 4e-14 of a charge in the box at (1.5, 2.5), where H_N leaves 1.7e-15.
struct LeafForm {
  std::vector<double> E;               // 4 x 28 x 64
  std::vector<double> H[8];            // E, W, N, S (256 x 96), NE, NW, SE, SW (256 x 48)
  std::vector<std::vector<double>> C;  // near relations 1..32: H_d^T T_r E^T
};
// H^T A for A 256 x n
static std::vector<double> ht_times(const std::vector<double>& H, int k, const std::vector<double>& A, int n) {
  std::vector<double> R(size_t(k) * n, 0.0);
  for (int i = 0; i < kNP; ++i)
    for (int c = 0; c < k; ++c) {
      const double h = H[size_t(i) * k + c];
      if (h == 0.0) continue;
      for (int j = 0; j < n; ++j) R[size_t(c) * n + j] += h * A[size_t(i) * n + j];
    }
  return R;
}
static const LeafForm& leaf_form() {
  static std::once_flag once;
  static LeafForm* F = nullptr;
  std::call_once(once, []() {
    auto* f = new LeafForm();
    outgoing_basis(f->E);
    const auto& T = near_tables();
    const auto& NO = near_offsets();
    std::vector<std::vector<double>> TE(33);  // parity basis, times E^T: 256 x 112
    {
      std::vector<std::thread> th;
      for (int r = 1; r <= 32; ++r)
        th.emplace_back([&, r]() { TE[size_t(r)] = times_et(parity_rows(parity_cols(T[size_t(r)], kNP), kNP), kNP, f->E); });
      for (auto& t : th) t.join();
    }
    std::vector<std::vector<double>> even, odd, corner;
    for (int r = 1; r <= 32; ++r) {
      const int d = near_dir(NO[size_t(r)].dx, NO[size_t(r)].dy, NO[size_t(r)].rho);
      if (d != 0 && d != 4) continue;
      for (int c = 0; c < kOutAll; ++c) {
        std::vector<double> v(kNP);
        for (int i = 0; i < kNP; ++i) v[size_t(i)] = TE[size_t(r)][size_t(i) * kOutAll + c];
        if (d == 4) {
          corner.push_back(v);
        } else {
          even.emplace_back(v.begin(), v.begin() + 128);
          odd.emplace_back(v.begin() + 128, v.end());
        }
      }
    }
    std::vector<double> He, Ho, Hc;
    {
      std::thread a([&]() { He = leading_basis(even, 128, kEdge / 2); });
      std::thread b([&]() { Ho = leading_basis(odd, 128, kEdge / 2); });
      Hc = leading_basis(corner, kNP, kCorner);
      a.join();
      b.join();
    }
    f->H[0].assign(size_t(kNP) * kEdge, 0.0);
    for (int i = 0; i < 128; ++i)
      for (int c = 0; c < kEdge / 2; ++c) {
        f->H[0][size_t(i) * kEdge + c] = He[size_t(i) * (kEdge / 2) + c];
        f->H[0][size_t(128 + i) * kEdge + kEdge / 2 + c] = Ho[size_t(i) * (kEdge / 2) + c];
      }
    f->H[2].assign(size_t(kNP) * kEdge, 0.0);
    for (int p = 0; p < 4; ++p)
      for (int j = 0; j < 8; ++j)
        for (int i = 0; i < 8; ++i) {
          const int pt = (p >> 1) + 2 * (p & 1);
          for (int c = 0; c < kEdge; ++c)
            f->H[2][size_t(64 * p + 8 * j + i) * kEdge + c] = f->H[0][size_t(64 * pt + 8 * i + j) * kEdge + c];
        }
    f->H[4] = Hc;
    auto mirror = [&](const std::vector<double>& H, int k, int parts) {  // negative on the parts with a bit of `parts` odd
      std::vector<double> R(H);
      for (int p = 0; p < 4; ++p)
        if (__builtin_popcount(unsigned(p & parts)) & 1)
          for (int i = 0; i < 64 * k; ++i) R[size_t(p) * 64 * k + i] = -R[size_t(p) * 64 * k + i];
      return R;
    };
    f->H[1] = mirror(f->H[0], kEdge, 1);
    f->H[3] = mirror(f->H[2], kEdge, 2);
    f->H[5] = mirror(f->H[4], kCorner, 1);
    f->H[6] = mirror(f->H[4], kCorner, 2);
    f->H[7] = mirror(f->H[4], kCorner, 3);
    f->C.resize(33);
    std::vector<std::thread> th;
    for (int r = 1; r <= 32; ++r)
      th.emplace_back([&, r]() {
        const int d = near_dir(NO[size_t(r)].dx, NO[size_t(r)].dy, NO[size_t(r)].rho);
        f->C[size_t(r)] = ht_times(f->H[d], d < 4 ? kEdge : kCorner, TE[size_t(r)], kOutAll);
      });
    for (auto& t : th) t.join();
    F = f;
  });
  return *F;
}

// The relation tables of the compressed form for expansions of Q complex terms, from the others (B).
static void leaf_form_tables(Matrices& M, const Matrices& B, int Q) {
  const LeafForm& F = leaf_form();
  const int ne = 2 * Q, qh = Q / 2, qp = pad16(qh);
  auto set = [&](int id, int rows, int cols, std::vector<double>&& a) {
    M.M[id] = rows; M.K[id] = cols; M.a[id] = std::move(a);
  };
  for (int r = 1; r <= 32; ++r) {
    const Offset& o = near_offsets()[size_t(r)];
    set(kRelC + r - 1, near_dir(o.dx, o.dy, o.rho) < 4 ? kEdge : kCorner, kOutAll, std::vector<double>(F.C[size_t(r)]));
  }
  for (int r = 0; r < 20; ++r) {
    const Offset& w = w_offsets()[size_t(r)];
    const int d = near_dir(w.dx, w.dy, w.rho), k = d < 4 ? kEdge : kCorner;
    set(kRelCW + r, k, ne, ht_times(F.H[d], k, parity_cols(B.a[kRelM2T + r], ne), ne));
    set(kRelXE + r, ne, kOutAll, times_et(parity_rows(B.a[kRelS2L + r], ne), ne, F.E));
  }
  // real i of part p in an expansion of interleaved reals: the series' terms z^n have Re even in y
  // and Im odd in y, their parity in x that of n (Re) or n - 1 (Im)
  auto real_of = [](int p, int i) { return 4 * i + (p == 0 ? 0 : p == 1 ? 2 : p == 2 ? 3 : 1); };
  const std::vector<double> S = parity_rows(B.a[kRelS2M], ne), L = parity_cols(B.a[kRelL2T], ne);
  const std::vector<double> T0 = parity_rows(parity_cols(B.a[kRelNear], kNP), kNP);
  const int groups = kLinGroups + qp / 16;
  std::vector<double> li(size_t(kLinRows) * 64, 0.0), lia(size_t(groups) * 64 * 64, 0.0);
  std::vector<double> lo(size_t(kNP) * (kLoutCols + qp), 0.0), loa(size_t(kNP) * (kLoutAdjCols + qp), 0.0);
  // the kernels' parity sums leave out the factor 1/2, on the way in and on the way out: the
  // tables carry it
  for (int p = 0; p < 4; ++p) {
    for (int k = 0; k < 64; ++k) {
      for (int r = 0; r < kOut; ++r) li[size_t(48 * p + r) * 64 + k] = 0.5 * F.E[(size_t(p) * kOut + r) * 64 + k];
      for (int i = 0; i < qh; ++i) li[size_t(48 * p + kOut + i) * 64 + k] = 0.5 * S[size_t(real_of(p, i)) * kNP + 64 * p + k];
    }
    const int py = p >> 1, px = p & 1, h = kEdge / 2;
    for (int k = 0; k < 64; ++k) {  // node k of part p
      const size_t row = size_t(64 * p + k);
      double* o = lo.data() + row * (kLoutCols + qp);
      double* a = loa.data() + row * (kLoutAdjCols + qp);
      for (int c = 0; c < 64; ++c) {
        o[c] = 0.25 * T0[row * kNP + 64 * p + c];
        a[c] = 0.25 * T0[size_t(64 * p + c) * kNP + row];
      }
      for (int c = 0; c < h; ++c) {
        o[64 + c] = 0.5 * F.H[0][row * kEdge + h * py + c];
        o[64 + h + c] = 0.5 * F.H[2][row * kEdge + h * px + c];
      }
      for (int c = 0; c < kCorner; ++c) o[64 + kEdge + c] = 0.5 * F.H[4][row * kCorner + c];
      for (int i = 0; i < qh; ++i) o[kLoutCols + i] = 0.5 * L[row * ne + real_of(p, i)];
      for (int r = 0; r < kOut; ++r) a[64 + r] = 0.5 * F.E[(size_t(p) * kOut + r) * 64 + k];
      for (int i = 0; i < qh; ++i) a[kLoutAdjCols + i] = 0.5 * S[size_t(real_of(p, i)) * kNP + row];
      // the transpose of the incoming columns: row tile (4 g + p) holds rows 16 g .. of part p
      for (int c = 64; c < kLoutCols + qp; ++c) {
        const int g = (c - 64) / 16;
        lia[size_t((4 * g + p) * 16 + (c - 64) % 16) * 64 + k] = o[c];
      }
    }
  }
  set(kRelLI, kLinRows, 64, std::move(li));
  set(kRelLO, kNP, kLoutCols + qp, std::move(lo));
  set(kRelLI + kNumFwd, groups * 64, 64, std::move(lia));
  set(kRelLO + kNumFwd, kNP, kLoutAdjCols + qp, std::move(loa));
}

// Transposes of the tables of forward ids [id0, id1); non-zeros of every table present.
static void transpose_tables(Matrices& M, int id0, int id1) {
  for (int id = id0; id < id1; ++id) {
    const int r = M.M[id], c = M.K[id];
    std::vector<double> T(size_t(r) * c);
    for (int i = 0; i < r; ++i)
      for (int j = 0; j < c; ++j) T[size_t(j) * r + i] = M.a[id][size_t(i) * c + j];
    M.M[id + kNumFwd] = c; M.K[id + kNumFwd] = r; M.a[id + kNumFwd] = std::move(T);
  }
}
static void count_tables(Matrices& M) {
  for (int id = 0; id < kNumRel; ++id) {
    if (M.a[id].empty()) continue;
    double n = 0;
    for (double v : M.a[id]) n += (v != 0.0);
    M.nnz[id] = n;
  }
}

static Matrices build_matrices(const int Q) {
  const int kNE = 2 * Q;  // reals per expansion for this order
  Matrices M;
  M.M.assign(kNumRel, 0);
  M.K.assign(kNumRel, 0);
  M.a.assign(kNumRel, {});
  M.nnz.assign(kNumRel, 0.0);
  M.w_in.assign(kNumRel, {});
  M.w_out.assign(kNumRel, {});
  M.lnd.assign(kNumRel, 0.0);
  M.koff.assign(kNumRel, 0);
  const Basis& B = basis();
  std::vector<cd> xi(kNP);
  for (int m = 0; m < kNP; ++m) xi[m] = cd(B.t[m % kP], B.t[m / kP]);
  auto set = [&](int id, int rows, int cols, std::vector<double>&& a) {
    M.M[id] = rows; M.K[id] = cols; M.a[id] = std::move(a);
  };
  // S2M: c_n int l_k eta^n, c_0 = 1, c_n = -1/n
  set(kRelS2M, kNE, kNP, s2m_table(Q));
  // M2M_q and L2L_q
  for (int q = 0; q < 4; ++q) {
    cd z0((q & 1) ? 0.5 : -0.5, (q & 2) ? 0.5 : -0.5);
    std::vector<cd> Bm(size_t(Q) * Q, cd(0.0)), E(size_t(Q) * Q, cd(0.0));
    Bm[0] = 1.0;
    for (int l = 1; l < Q; ++l) {
      Bm[size_t(l) * Q] = -std::pow(z0, l) / double(l);
      for (int k = 1; k <= l; ++k) Bm[size_t(l) * Q + k] = std::ldexp(1.0, -k) * binom_exact(l - 1, k - 1) * std::pow(z0, l - k);
    }
    for (int l = 0; l < Q; ++l)
      for (int k = l; k < Q; ++k) E[size_t(l) * Q + k] = binom_exact(k, l) * std::pow(z0, k - l) * std::ldexp(1.0, -l);
    std::vector<double> R1, R2;
    real_from_linear(Bm, Q, Q, R1);
    real_from_linear(E, Q, Q, R2);
    set(kRelM2M + q, kNE, kNE, std::move(R1));
    set(kRelL2L + q, kNE, kNE, std::move(R2));
  }
  // two-level translations: M2M_qc M2M_qg (grandchild to box) and L2L_qg L2L_qc (box to grandchild)
  for (int qc = 0; qc < 4; ++qc)
    for (int qg = 0; qg < 4; ++qg) {
      std::vector<double> Pm(size_t(kNE) * kNE, 0.0), Pl(size_t(kNE) * kNE, 0.0);
      const std::vector<double>& Mc = M.a[kRelM2M + qc];
      const std::vector<double>& Mg = M.a[kRelM2M + qg];
      const std::vector<double>& Lc = M.a[kRelL2L + qc];
      const std::vector<double>& Lg = M.a[kRelL2L + qg];
      for (int i = 0; i < kNE; ++i)
        for (int k = 0; k < kNE; ++k) {
          const double mc = Mc[size_t(i) * kNE + k], lg = Lg[size_t(i) * kNE + k];
          for (int j = 0; j < kNE; ++j) {
            Pm[size_t(i) * kNE + j] += mc * Mg[size_t(k) * kNE + j];
            Pl[size_t(i) * kNE + j] += lg * Lc[size_t(k) * kNE + j];
          }
        }
      set(kRelM2M2 + 4 * qc + qg, kNE, kNE, std::move(Pm));
      set(kRelL2L2 + 4 * qc + qg, kNE, kNE, std::move(Pl));
    }
  // M2L_r: d = (source - target centre) / s
  const auto& VO = v_offsets();
  for (size_t r = 0; r < VO.size(); ++r) {
    cd d(VO[r].dx, VO[r].dy);
    std::vector<cd> K(size_t(Q) * Q, cd(0.0));
    K[0] = std::log(std::abs(d));
    for (int k = 1; k < Q; ++k) K[k] = ((k & 1) ? -1.0 : 1.0) * std::pow(d, -k);
    for (int l = 1; l < Q; ++l) {
      K[size_t(l) * Q] = -1.0 / (double(l) * std::pow(d, l));
      for (int k = 1; k < Q; ++k) K[size_t(l) * Q + k] = ((k & 1) ? -1.0 : 1.0) * binom_exact(k + l - 1, l) * std::pow(d, -(k + l));
    }
    std::vector<double> R;
    real_from_linear(K, Q, Q, R);
    set(kRelM2L + int(r), kNE, kNE, std::move(R));
    // the same map factored: w_out = d^-l, w_in = (-1)^k d^-k around the core kRelH; the
    // adjoint (the real transpose) conjugates both diagonals and swaps their roles
    const int id = kRelM2L + int(r), ia = id + kNumFwd, QP = pad16(Q);
    M.w_in[id].assign(size_t(2 * Q), 0.0);
    M.w_out[id].assign(size_t(2 * QP), 0.0);
    M.w_in[ia].assign(size_t(2 * Q), 0.0);
    M.w_out[ia].assign(size_t(2 * QP), 0.0);
    for (int k = 0; k < Q; ++k) {
      const cd dl = std::pow(d, -k), dr = ((k & 1) ? -1.0 : 1.0) * dl;
      M.w_out[id][size_t(2 * k)] = dl.real(); M.w_out[id][size_t(2 * k + 1)] = dl.imag();
      M.w_in[id][size_t(2 * k)] = dr.real(); M.w_in[id][size_t(2 * k + 1)] = dr.imag();
      M.w_in[ia][size_t(2 * k)] = dl.real(); M.w_in[ia][size_t(2 * k + 1)] = -dl.imag();
      M.w_out[ia][size_t(2 * k)] = dr.real(); M.w_out[ia][size_t(2 * k + 1)] = -dr.imag();
    }
    M.lnd[id] = M.lnd[ia] = std::log(std::abs(d));
  }
  {  // the offset-free core of the factored M2L, rows padded to a multiple of 16
    const int QP = pad16(Q);
    std::vector<double> H(size_t(QP) * Q, 0.0);
    for (int k = 1; k < Q; ++k) H[size_t(k)] = 1.0;
    for (int l = 1; l < Q; ++l) {
      H[size_t(l) * Q] = -1.0 / double(l);
      for (int k = 1; k < Q; ++k) H[size_t(l) * Q + k] = binom_exact(k + l - 1, l);
    }
    set(kRelH, QP, Q, std::move(H));
  }
  // S2L_r: source leaf (rho = 2) at d = (source - target centre) / s_target
  const auto& XO = x_offsets();
  for (size_t r = 0; r < XO.size(); ++r) {
    cd d(XO[r].dx, XO[r].dy);
    double rho = XO[r].rho;
    auto S = quad_basis(48, Q, [&](int l, cd e) {
      cd w = d + rho * e;
      return l == 0 ? cd(std::log(std::abs(w))) : -std::pow(w, -l) / double(l);
    });
    std::vector<double> R;
    real_from_realin(S, Q, kNP, R);
    set(kRelS2L + int(r), kNE, kNP, std::move(R));
  }
  // near tables
  {
    const std::vector<std::vector<double>>& T = near_tables();
    for (int r = 0; r < 33; ++r) set(kRelNear + r, kNP, kNP, std::vector<double>(T[size_t(r)]));
    // the low-rank form of relations 1..32 and the 64-column slices of the self table
    const NearFactors& F = near_factors();
    for (int r = 0; r < 32; ++r) {
      const int k = F.rank[size_t(r)];
      set(kRelNU + r, kNP, k, std::vector<double>(F.U[size_t(r)]));
      set(kRelNV + r, k, kNP, std::vector<double>(F.V[size_t(r)]));
    }
    const std::vector<double>& S = T[0];
    for (int q = 0; q < 4; ++q) {
      std::vector<double> fw(size_t(kNP) * 64), ad(size_t(kNP) * 64);
      for (int i = 0; i < kNP; ++i)
        for (int c = 0; c < 64; ++c) {
          fw[size_t(i) * 64 + c] = S[size_t(i) * kNP + 64 * q + c];  // T[i][64q + c]
          ad[size_t(i) * 64 + c] = S[size_t(64 * q + c) * kNP + i];  // (T[64q + c][i]): T^T's column block
        }
      set(kRelNSF + q, kNP, 64, std::move(fw));
      set(kRelNSA + q, kNP, 64, std::move(ad));
      M.koff[size_t(kRelNSF + q)] = M.koff[size_t(kRelNSA + q)] = 64 * q;
    }
  }
  // M2T_r: source box (rho = 1/2) at d = (source - target centre) / s_target
  for (int r = 0; r < int(w_offsets().size()); ++r) set(kRelM2T + r, kNP, kNE, m2t_table(r, Q));
  // L2T
  {
    std::vector<cd> Lt(size_t(kNP) * Q);
    for (int m = 0; m < kNP; ++m)
      for (int l = 0; l < Q; ++l) Lt[size_t(m) * Q + l] = -kInv2Pi * std::pow(xi[m], l);
    std::vector<double> R;
    real_from_realout(Lt, kNP, Q, R);
    set(kRelL2T, kNP, kNE, std::move(R));
  }
  transpose_tables(M, 0, kRelLeafForm);
  {  // the core's transpose keeps the padded shape: rows k (padded), columns l
    const int QP = pad16(Q);
    const std::vector<double>& H = M.a[kRelH];
    std::vector<double> T(size_t(QP) * Q, 0.0);
    for (int l = 0; l < Q; ++l)
      for (int k = 0; k < Q; ++k) T[size_t(k) * Q + l] = H[size_t(l) * Q + k];
    set(kRelH + kNumFwd, QP, Q, std::move(T));
  }
  count_tables(M);
  return M;
}

static Matrices build_leaf_matrices(const int Q) {
  const Matrices& B = matrices(Q);
  Matrices M;
  M.M = B.M; M.K = B.K; M.nnz = B.nnz; M.w_in = B.w_in; M.w_out = B.w_out; M.lnd = B.lnd; M.koff = B.koff;
  M.a.assign(kNumRel, {});
  leaf_form_tables(M, B, Q);
  // the leaf kernels' adjoint tables have their own layout and are set already
  transpose_tables(M, kRelLeafForm, kRelLI);
  count_tables(M);
  return M;
}

static const Matrices& build_once(int q, Matrices (*build)(int), std::mutex& mu, std::map<int, const Matrices*>& built) {
  std::lock_guard<std::mutex> lk(mu);
  auto it = built.find(q);
  if (it == built.end()) it = built.emplace(q, new Matrices(build(q))).first;
  return *it->second;
}
const Matrices& matrices(int q) {
  static std::mutex mu;
  static std::map<int, const Matrices*> built;
  return build_once(q, build_matrices, mu, built);
}
const Matrices& leaf_matrices(int q) {
  static std::mutex mu;
  static std::map<int, const Matrices*> built;
  return build_once(q, build_leaf_matrices, mu, built);
}

}  // namespace vp
