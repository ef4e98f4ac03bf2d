// Host side of libmsm: parameter validation, grid hierarchy, stencil and
// top-level tables (double precision on the host), workspace layout, and the
// C ABI declared in include/msm.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <utility>
#include <cmath>
#include <cstring>
#include <new>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "msm_plan.hpp"

namespace {
thread_local std::string g_last_error;
}  // namespace

msm_status fail(msm_status s, const std::string& msg) {
  g_last_error = msg;
  return s;
}

msm_status hip_fail(hipError_t e, const char* what) {
  g_last_error = std::string(what) + ": " + hipGetErrorString(e);
  return MSM_ERR_HIP;
}

// Create (once per owner) the auxiliary stream and fork/join events on the
// current device.  Streams keep the default priority.
hipError_t ensure_aux(AuxStreams& A) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (A.cc.shortr.stream && A.device == dev) return hipSuccess;
  destroy_aux(A);
  // the events only order work between streams of this device: no timing and
  // no system-scope fence (kernels end with a device-scope release already)
  const unsigned ev_flags = hipEventDisableTiming | hipEventDisableSystemFence;
  for (msm::SideStream* ss : {&A.cc.shortr, &A.cc.lattice0}) {
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&ss->stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ss->fork, ev_flags);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ss->join, ev_flags);
  }
  if (e != hipSuccess) {
    destroy_aux(A);
    return e;
  }
  A.device = dev;
  return hipSuccess;
}

void destroy_aux(AuxStreams& A) {
  for (msm::SideStream* ss : {&A.cc.shortr, &A.cc.lattice0}) {
    if (ss->stream) (void)hipStreamDestroy(ss->stream);
    if (ss->fork) (void)hipEventDestroy(ss->fork);
    if (ss->join) (void)hipEventDestroy(ss->join);
  }
  A.cc = msm::Concurrency{};
  A.device = -1;
}

namespace {

// Taylor smoothing (Sec. 2.3): gamma(rho) = sum_k c_k rho^{2k}, rho < 1, with c_k
// the coefficients of the degree-m Taylor polynomial of s^{-1/2} at s = 1,
// collected in powers of s.
void taylor_coeffs(int m, double* c) {
  for (int k = 0; k <= m; ++k) c[k] = 0.0;
  double tj = 1.0;                                   // binom(-1/2, j)
  for (int j = 0; j <= m; ++j) {
    if (j > 0) tj *= (-0.5 - (j - 1)) / j;
    double bjk = 1.0;                                // binom(j, k)
    for (int k = 0; k <= j; ++k) {
      if (k > 0) bjk = bjk * (j - k + 1) / k;
      c[k] += tj * bjk * (((j - k) % 2) ? -1.0 : 1.0);
    }
  }
}

double gamma_h(const double* c, int m, double rho) {
  if (rho >= 1.0) return 1.0 / rho;
  double s = rho * rho, v = c[m];
  for (int k = m - 1; k >= 0; --k) v = v * s + c[k];
  return v;
}


int floor_div2(int v) { return v >= 0 ? v / 2 : -((-v + 1) / 2); }
int ceil_div2(int v) { return -floor_div2(-v); }

// Top level of a periodic plan: K(d) = sum over images p of g^{l-1}(|h_t d + P p|)
// for every node offset d of the top grid (P = diag(box edges)).  g^{l-1}
// decays as 1/r, so the image sum is the Ewald one (conducting boundary,
// uniform neutralising background): K = Psi - sum over the images closer than
// A = 2^{l-1} a of (1/rho - g^{l-1}(rho)), with
//   Psi(r) = sum_p erfc(b |r + P p|) / |r + P p|
//          + (4 pi / V) sum_{k != 0} exp(-k^2 / 4b^2) cos(k.r) / k^2 - pi / (V b^2)
// and, at d = 0, the node's own term g^{l-1}(0) in place of the singular
// p = 0 Coulomb term (whose Ewald remainder is -2b/sqrt(pi)).  b = 3 / min(len);
// real-space images to 6 / b and wave vectors to k^2 = 156 b^2 leave terms
// below 1e-16.
void periodic_top_table(const double* c, int m, double A, double ht, const int nt[3], const double len[3],
                        std::vector<double>& K) {
  const double pi = 3.14159265358979323846;
  const double lmin = std::min({len[0], len[1], len[2]});
  const double b = 3.0 / lmin, V = len[0] * len[1] * len[2], rc = 6.0 / b, kc2 = 156.0 * b * b;
  struct Wave { double kx, ky, kz, w; };
  std::vector<Wave> waves;
  int kn[3], pn[3], an[3];
  for (int d = 0; d < 3; ++d) {
    kn[d] = (int)std::ceil(std::sqrt(kc2) * len[d] / (2.0 * pi));
    pn[d] = (int)std::ceil(rc / len[d]) + 1;
    an[d] = (int)std::ceil(A / len[d]) + 1;
  }
  for (int iz = -kn[2]; iz <= kn[2]; ++iz)
    for (int iy = -kn[1]; iy <= kn[1]; ++iy)
      for (int ix = -kn[0]; ix <= kn[0]; ++ix) {
        if (!ix && !iy && !iz) continue;
        const Wave v{2.0 * pi * ix / len[0], 2.0 * pi * iy / len[1], 2.0 * pi * iz / len[2], 0.0};
        const double k2 = v.kx * v.kx + v.ky * v.ky + v.kz * v.kz;
        if (k2 <= kc2) waves.push_back(Wave{v.kx, v.ky, v.kz, 4.0 * pi / V * std::exp(-k2 / (4.0 * b * b)) / k2});
      }
  K.assign((size_t)nt[0] * nt[1] * nt[2], 0.0);
  for (int dz = 0; dz < nt[2]; ++dz)
    for (int dy = 0; dy < nt[1]; ++dy)
      for (int dx = 0; dx < nt[0]; ++dx) {
        const double r[3] = {ht * dx, ht * dy, ht * dz};
        const bool self = !dx && !dy && !dz;
        double real = 0.0, corr = 0.0, recip = 0.0;
        // images within the Ewald real-space cutoff and within A, one pass each
        for (int pz = -std::max(pn[2], an[2]); pz <= std::max(pn[2], an[2]); ++pz)
          for (int py = -std::max(pn[1], an[1]); py <= std::max(pn[1], an[1]); ++py)
            for (int px = -std::max(pn[0], an[0]); px <= std::max(pn[0], an[0]); ++px) {
              if (self && !px && !py && !pz) continue;
              const double vx = r[0] + px * len[0], vy = r[1] + py * len[1], vz = r[2] + pz * len[2];
              const double rho = std::sqrt(vx * vx + vy * vy + vz * vz);
              if (rho < rc) real += std::erfc(b * rho) / rho;
              if (rho < A) corr += 1.0 / rho - gamma_h(c, m, rho / A) / A;
            }
        for (const Wave& v : waves) recip += v.w * std::cos(v.kx * r[0] + v.ky * r[1] + v.kz * r[2]);
        double k = real + recip - pi / (V * b * b) - corr;
        if (self) k += gamma_h(c, m, 0.0) / A - 2.0 * b / std::sqrt(pi);
        K[((size_t)dz * nt[1] + dy) * nt[0] + dx] = k;
      }
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

// The bfloat16 (8 significant bits) nearest to v, and its bits.
double bf16_nearest(double v) {
  int e = 0;
  (void)std::frexp(v, &e);                                 // |v| in [2^(e-1), 2^e)
  return std::ldexp(std::nearbyint(std::ldexp(v, 8 - e)), e - 8);
}

uint16_t bf16_bits(double nearest) {
  const float f = (float)nearest;
  uint32_t u;
  std::memcpy(&u, &f, sizeof u);
  return (uint16_t)(u >> 16);
}

// Weight fragments of the tiled lattice-cutoff kernel for the taps W(|n|),
// |n| < rad, n up to H per dimension; weight(n2) = W at |n|^2 = n2.  Lane l of a
// fragment holds output l & 15 and 8 inputs from first(l / 16), zero where there
// is no tap.  Fragments az (H + 1) + ay: the inputs within 8 of the outputs of
// row (ay, az).  Then (H > 8), (2 phase + p)(H + 1) + ay further on: the wings
// of the phase's planes 2p (lanes 0 - 31) and 2p + 1 (lanes 32 - 63).
template <class Weight>
void lattice_fragments(int H, double rad, Weight weight, msm::LatLaunch& lat, std::vector<uint16_t>& frags) {
  auto inside = [&](int n2) { return std::sqrt((double)n2) < rad; };
  for (int n2 = 0; n2 <= 3 * H * H; ++n2)
    if (inside(n2)) lat.n2max = n2;
  lat.phases = (2 * H + msm::kLatPlanes) / msm::kLatPlanes;
  const int words = msm::kLatFragBytes / 2, part = words / 3;
  const int n_main = (H + msm::kLatPlanes) * (H + 1), n_wing = H > 8 ? 2 * lat.phases * (H + 1) : 0;
  frags.assign((size_t)(n_main + n_wing) * words, 0);
  auto octet = [&](int id, int quad, int first, int ay, int az) {
    if (az > H) return;
    for (int l = 16 * quad; l < 16 * quad + 16; ++l)
      for (int i = 0; i < 8; ++i) {
        const int nx = first + i - (l & 15), n2 = nx * nx + ay * ay + az * az;
        if (std::abs(nx) > H || !inside(n2)) continue;
        double w = ay ? weight(n2) : 0.5 * weight(n2);     // (the pair +-0 counts its row twice)
        for (int p = 0; p < 3; ++p) {
          const double near = bf16_nearest(w);
          frags[(size_t)id * words + p * part + l * 8 + i] = bf16_bits(near);
          w -= near;
        }
      }
  };
  for (int az = 0; az <= H; ++az)                          // (the last phase's planes beyond H stay zero)
    for (int ay = 0; ay <= H; ++ay)
      for (int quad = 0; quad < 4; ++quad) octet(az * (H + 1) + ay, quad, 8 * quad - 8, ay, az);
  if (n_wing)
    for (int pp = 0; pp < 2 * lat.phases; ++pp)
      for (int ay = 0; ay <= H; ++ay)
        for (int quad = 0; quad < 4; ++quad)
          octet(n_main + pp * (H + 1) + ay, quad, quad & 1 ? 24 : -16, ay, std::abs(2 * pp + quad / 2 - H));
}

// Shares a phase's row pairs ny = +-ay among 4 waves with the least largest cost,
// which it returns (fragment products; a pair with wings counts for one and a
// half): in contiguous runs, or dealt in turn.  Half-width 9 has four pairs with
// wings of ten near the centre (3 in runs, 3.5 in turn), 11 eight of twelve (4.5
// and 4: 31 and 29 us at 24,000 atoms).
double share_rows(msm::LatLaunch& lat, int ph) {
  constexpr int waves = 4;
  const int nz0 = msm::kLatPlanes * ph - lat.H;
  const int az = nz0 > 0 ? nz0 : std::max(0, -(nz0 + msm::kLatPlanes - 1));
  std::vector<double> cost;
  double turn[waves] = {}, total = 0.0;
  for (int ay = 0; ay * ay + az * az <= lat.n2max; ++ay) {
    cost.push_back(lat.H > 8 && 81 + ay * ay + az * az <= lat.n2max ? 1.5 : 1.0);
    turn[ay % waves] += cost.back();
    total += cost.back();
  }
  const int n = (int)cost.size();
  unsigned char* share = lat.share[ph];
  auto runs = [&](double cap) {
    int w = 0;
    double acc = 0.0;
    std::fill(share, share + 2 * waves, (unsigned char)n);
    share[0] = 0;
    for (int i = 0; i < n; ++i) {
      if (acc + cost[i] > cap) {
        share[waves + w] = (unsigned char)i;
        if (++w == waves) return false;
        share[w] = (unsigned char)i;
        acc = 0.0;
      }
      acc += cost[i];
    }
    return true;
  };
  // costs are multiples of one half, the first the largest
  double cap = std::max(cost[0], 0.5 * std::ceil(2.0 * total / waves));
  while (!runs(cap)) cap += 0.5;
  lat.step[ph] = 1;
  const double most = *std::max_element(turn, turn + waves);
  if (most >= cap) return cap;
  for (int w = 0; w < waves; ++w) {
    share[w] = (unsigned char)w;
    share[waves + w] = (unsigned char)n;
  }
  lat.step[ph] = waves;
  return most;
}

// Tiles of the lattice-cutoff kernel: planes per block (force_b, or 6 where that
// makes 256 blocks of level 0 and 4 where not; two blocks fit a CU, so one
// stages its window while the other multiplies), the waves' shares of the
// phases' rows, and the split of each level's phases over blocks: more blocks
// fill the chip, fewer write and read back fewer partials.  The coarse levels'
// blocks come last and are split as far as they can be.  Level 0 by an estimate
// in cycles: a block starts and ends (9,000), each phase stages its window and
// runs its rows on the matrix pipe, 96 cycles a fragment and plane.  Blocks that
// all fit the chip take as long as the longest, sharing its pipes; of more, the
// work is spread over those that fit, and the longest block ends last.
// Stage time with 4, 6 and 8 planes: 1,000 charges 10.6, 12.6, 12.8 us; 9,000
// periodic (96 blocks with 6) 24.4, 28.2, 26.2; 4,096 ions (216) 15.8, 16.6; 24,000
// atoms (324) 27, 28, 34; 50,000 (315) 31, 28; 100,000 (864) 53, 57, 60; 1M (2880)
// 112, 109, 132; 1M periodic (1750) 58, 60, 66.  Level 0 in 1, 2, 3, 5, 6 blocks a
// tile: 24,000 atoms, 4 planes, 53, 32, 27, 28, 30 us; 100,000, 6 planes, 97, 57,
// 51, 51, 51 (61 with the coarse levels in 5 and 3 blocks); 1M, 6 planes, 1, 2, 3,
// 5 blocks: 109, 122, 115, 119.
void choose_lattice_tiles(const Geom& g, int H_, msm::LatLaunch& lat, int force_b = 0) {
  const int phases = lat.phases, n2max = lat.n2max;
  std::memset(&lat, 0, sizeof(lat));
  lat.H = H_;
  lat.phases = phases;
  lat.n2max = n2max;
  if (g.levels < 2 || H_ > msm::kLatMaxHalo) return;
  const int skip = g.periodic ? g.ghost : 0;
  auto tiles_of = [&](int k, int B, msm::LatTile& t) {
    // a periodic level's outputs: the nodes of one period, along x from the
    // multiple of 8 below its first
    const msm::Level& L = g.lv[k];
    t.ntx = ((g.periodic ? L.per[0] + (skip & 7) : L.n[0]) + 15) / 16;
    t.nty = (L.n[1] - 2 * skip + 15) / 16;
    t.ntz = (L.n[2] - 2 * skip + B - 1) / B;
    return (double)t.ntx * t.nty * t.ntz;
  };
  msm::LatTile probe{};
  const int B = force_b ? force_b : (tiles_of(0, 6, probe) * phases < 256.0 ? 4 : 6);
  lat.b = B;
  lat.n = g.levels - 1;
  lat.lds_bytes = msm::lat_lds(H_, B);
  std::vector<double> mat(phases);                         // fragment pairs of each phase's slowest wave
  for (int ph = 0; ph < phases; ++ph) mat[ph] = share_rows(lat, ph);
  // blocks on the chip at a time (two on a CU share its matrix pipes)
  const int slots = 256 * (B < 8 && 2 * (lat.lds_bytes + 2048) <= 160 * 1024 ? 2 : 1);
  // a block of phases [ph0, ph1): cycles beside the matrix pipe, and on it
  auto beside = [&](int ph0, int ph1) { return 9000.0 + (3000.0 + 500.0 * (B + 3)) * (ph1 - ph0); };
  auto matrix = [&](int ph0, int ph1) {
    double m = 0.0;
    for (int ph = ph0; ph < ph1; ++ph) m += mat[ph] * 96.0 * msm::kLatPlanes * B * 4 / msm::lat_waves(B);
    return m;
  };
  double coarse = 0.0, coarse_blocks = 0.0;                // cycles and blocks of the coarse levels
  for (int k = g.levels - 2; k >= 0; --k) {                // (level 0 takes the partials the others leave)
    const msm::Level& L = g.lv[k];
    msm::LatTile t{};
    t.level = k;
    t.groups = 1;
    const double tiles = tiles_of(k, B, t);
    double best = 1e300;
    for (int G = 1; G <= std::min(msm::kLatMaxGroups, phases); ++G) {
      if (G > 1 && lat.n_part + (double)G * L.count > (double)g.part_cap) break;
      if (k > 0) {
        t.groups = G;
        continue;
      }
      double sum = 0.0, side = 0.0, mm = 0.0;              // all blocks of a tile; its longest block
      for (int q = 0; q < G; ++q) {
        const int ph0 = phases * q / G, ph1 = phases * (q + 1) / G;
        sum += beside(ph0, ph1) + matrix(ph0, ph1);
        side = std::max(side, beside(ph0, ph1));
        mm = std::max(mm, matrix(ph0, ph1));
      }
      const double total = tiles * G + coarse_blocks;
      const double est = (total <= slots ? side + 1.05 * mm * std::ceil(total / 256.0) : (tiles * sum + coarse) / slots + side + mm) +
                         (G > 1 ? 0.013 * G * L.count : 0.0);
      if (est < best) {
        best = est;
        t.groups = G;
      }
    }
    if (k > 0) {
      coarse_blocks += tiles * t.groups;
      coarse += tiles * (9000.0 * (t.groups - 1) + beside(0, phases) + matrix(0, phases));
    }
    t.part0 = lat.n_part;
    if (t.groups > 1) lat.n_part += t.groups * L.count;
    lat.t[k] = t;
  }
  int blocks = 0;
  for (int k = 0; k < lat.n; ++k) {
    msm::LatTile& t = lat.t[k];
    t.block0 = blocks;
    blocks += t.ntx * t.nty * t.ntz * t.groups;
  }
}

// The plan's tiles, and the largest need of partials of any tuning.
void set_lattice_tiles(msm_plan* P, int H) {
  P->lat_part_max = 0;
  for (int b : {4, 6, 8}) {
    choose_lattice_tiles(P->g, H, P->lat, b);
    P->lat_part_max = std::max(P->lat_part_max, P->lat.n_part);
  }
  choose_lattice_tiles(P->g, H, P->lat);
}

// Least squares min |A c - b| over the columns of A (rows x cols, row-major)
// by Householder reflections; A and b are overwritten.
void householder_lsq(std::vector<double>& A, std::vector<double>& b, int rows, int cols, double* c) {
  for (int k = 0; k < cols; ++k) {
    double norm = 0.0;
    for (int i = k; i < rows; ++i) norm += A[i * cols + k] * A[i * cols + k];
    norm = std::sqrt(norm);
    const double alpha = A[k * cols + k] > 0 ? -norm : norm;
    std::vector<double> v(rows - k);
    for (int i = k; i < rows; ++i) v[i - k] = A[i * cols + k];
    v[0] -= alpha;
    double vv = 0.0;
    for (double e : v) vv += e * e;
    if (vv == 0.0) continue;
    for (int j = k; j < cols; ++j) {
      double s = 0.0;
      for (int i = k; i < rows; ++i) s += v[i - k] * A[i * cols + j];
      s *= 2.0 / vv;
      for (int i = k; i < rows; ++i) A[i * cols + j] -= s * v[i - k];
    }
    double s = 0.0;
    for (int i = k; i < rows; ++i) s += v[i - k] * b[i];
    s *= 2.0 / vv;
    for (int i = k; i < rows; ++i) b[i] -= s * v[i - k];
  }
  for (int k = cols - 1; k >= 0; --k) {
    double s = b[k];
    for (int j = k + 1; j < cols; ++j) s -= A[k * cols + j] * c[j];
    c[k] = A[k * cols + k] != 0.0 ? s / A[k * cols + k] : 0.0;
  }
}

// The Wolf pair function's erfc on the device: erfc(x) = exp(-x^2) R(x), with
// the smooth scaled function R(x) = erfc(x) exp(x^2) written as a polynomial
// in t = 1 / (1 + x/2) (the substitution of Hastings' approximations in
// Abramowitz and Stegun 7.1.25-28), fitted here in double over x in [0, x_hi]
// by least squares in relative error.  The coefficients are rounded to float
// one at a time from t^0 up, the later ones refitted after each rounding, so
// the rounded polynomial keeps the fit's accuracy (about 1e-9 relative for
// x_hi <= 6) instead of carrying a fixed float-rounding bias into every pair.
// Returns the fitted polynomial's largest relative error on a fine grid.
double fit_wolf_erfc(double x_hi, float* ec) {
  constexpr int m = msm::kWolfTerms, n = 12 * msm::kWolfTerms;
  const double tmin = 1.0 / (1.0 + 0.5 * x_hi);
  std::vector<double> t(n), w(n);
  for (int i = 0; i < n; ++i) {
    const double z = std::cos(M_PI * (i + 0.5) / n);
    t[i] = tmin + 0.5 * (z + 1.0) * (1.0 - tmin);
    const double x = 2.0 * (1.0 / t[i] - 1.0);
    w[i] = 1.0 / (std::erfc(x) * std::exp(x * x));
  }
  double fixed[m];
  for (int k = 0; k < m; ++k) {
    const int cols = m - k;
    std::vector<double> A(n * cols), b(n);
    for (int i = 0; i < n; ++i) {
      double tp = 1.0, rhs = 1.0;
      for (int j = 0; j < m; ++j, tp *= t[i]) {
        if (j < k) rhs -= fixed[j] * tp * w[i];
        else A[i * cols + (j - k)] = tp * w[i];
      }
      b[i] = rhs;
    }
    double c[m];
    householder_lsq(A, b, n, cols, c);
    fixed[k] = (double)(float)c[0];
  }
  double worst = 0.0;
  for (int i = 0; i <= 4000; ++i) {
    const double x = x_hi * i / 4000.0, tt = 1.0 / (1.0 + 0.5 * x);
    double p = 0.0;
    for (int k = m - 1; k >= 0; --k) p = p * tt + fixed[k];
    worst = std::max(worst, std::fabs(p / (std::erfc(x) * std::exp(x * x)) - 1.0));
  }
  for (int k = 0; k < m; ++k) ec[k] = (float)fixed[k];
  return worst;
}

}  // namespace

void refresh_launch(msm_plan* P) {
  const Geom& g = P->g;
  msm::DevPtrs keep = P->desc.d;
  std::memset(&P->desc, 0, sizeof(P->desc));
  P->desc.d = keep;
  P->desc.g = g;
  P->desc.lat = P->lat;
  P->desc.atom_off = 0;
  P->desc.index = 0;
  P->desc.n_partials = P->n_partials;
  P->desc.n_rows = (int)P->rows.size();
  const msm::SysBlocks sb = msm::system_blocks(g, P->lat, P->n_partials);
  msm::LaunchGeom& lg = P->lg;
  lg = msm::LaunchGeom{};
  lg.n_sys = 1;
  lg.order = g.order;
  lg.m = g.m;
  lg.pair = g.pair;
  lg.lat_b = P->lat.b;
  lg.lat_lds = P->lat.lds_bytes;
  lg.max_levels = g.levels;
  lg.short_after = P->short_after;
  lg.short_split = P->short_split;
  lg.zero.blocks = sb.zero;
  lg.atoms.blocks = sb.atoms;
  lg.bin.blocks = sb.bin;
  lg.binrow.blocks = sb.binrow;
  lg.binrow_lds = msm::bin_rows_lds(g);
  lg.bin4 = g.bin_blocks == 0 && g.bin_row_blocks == 0 && g.binr_blocks == 0;
  lg.rchunk.blocks = sb.rchunk;
  lg.binr_chunk = g.binr_chunk;
  lg.rscan.blocks = sb.rscan;
  lg.rsort.blocks = sb.rsort;
  lg.rsort_lds = msm::binr_sort_lds(g);
  lg.one.blocks = 1;
  lg.scan.blocks = sb.scan;
  lg.agather.blocks = sb.agather;
  lg.anterp_lds = msm::anterp_lds(g);
  // large grids: one prolongation launch per level instead of every block
  // rebuilding the coarser levels it reads (a level-0 tile of 8^3 nodes would
  // rebuild boxes of up to (2R + 3)^3 nodes on every coarser level)
  int tiles0 = 0;
  for (int k = 0; k + 1 < g.levels; ++k) {
    lg.prolong_level[k].blocks = sb.prolong_level[k];
    if (k == 0) tiles0 = sb.prolong_level[k];
  }
  lg.prolong_split = g.levels > 1 && (tiles0 >= msm::kProlongSplitTiles || g.periodic);
  lg.periodic = g.periodic && !g.pair;
  lg.short_periodic = g.periodic != 0;
  lg.shortr.blocks = sb.shortr;
  lg.short_parts = g.short_parts;
  lg.short_split_rows = g.short_parts > 1;
  lg.anterp.blocks = sb.anterp;
  lg.lattice0.blocks = sb.lattice0;
  lg.lattice0_tiles = msm::lattice0_tiles(P->lat);
  lg.lattice.blocks = sb.lattice;
  lg.lattice_all.blocks = sb.lattice_all;
  lg.top.blocks = sb.top;
  lg.energy.blocks = sb.energy;
  for (int k = 0; k + 1 < g.levels; ++k) {
    lg.restrict_[k].blocks = sb.restrict_[k];
  }
  lg.prolong.blocks = sb.prolong;
  lg.streams = lg.capture_streams = P->streams;
  if (!P->streams_set) default_streams(lg, g.periodic != 0);
}

// Neighbour cell rows (offsets oy, oz in [-reach, reach], row index
// (oz + reach) (2 reach + 1) + oy + reach) dealt to the 4 waves of a
// short-range block, largest expected x window first, each to the wave with
// the least work so far.  A row's expected window is the mean over atom
// positions (y, z) in a cell of 2 sqrt(a^2 - d^2), d the distance to the row.
// Free-space plans deal each row with its mirror (-oy, -oz) as one unit that
// a wave walks together: an atom near one face of its cell has a long window
// in the row beyond that face and a short one in the mirror row, so the sum
// of the two varies far less over the 64 atoms of a chunk than either.
void assign_short_rows(Geom& g) {
  const int R = g.reach, side = 2 * R + 1, nrows = side * side;
  const double a = g.a_win, cy = g.cs[1], cz = g.cs[2];
  std::vector<double> row_cost(nrows);
  for (int r = 0; r < nrows; ++r) {
    const int oy = r % side - R, oz = r / side - R;
    double sum = 0.0;
    const int K = 16;
    for (int iy = 0; iy < K; ++iy)
      for (int iz = 0; iz < K; ++iz) {
        const double y = (iy + 0.5) / K * cy, z = (iz + 0.5) / K * cz;
        auto gap = [](double v, int o, double c) {
          if (o > 0) return o * c - v;
          if (o < 0) return v - (o + 1) * c;
          return 0.0;
        };
        const double dy = gap(y, oy, cy), dz = gap(z, oz, cz), d2 = dy * dy + dz * dz;
        if (d2 < a * a) sum += 2.0 * std::sqrt(a * a - d2);
      }
    row_cost[r] = sum / (K * K) + 1.0;
  }
  // units: (cost, first row, second row or -1); the mirror of row r is nrows - 1 - r
  const bool pairs = !g.periodic;
  std::vector<std::tuple<double, int, int>> units;
  for (int r = 0; r < nrows; ++r) {
    const int m = nrows - 1 - r;
    if (pairs && m < r) continue;
    if (pairs && m > r) units.emplace_back(row_cost[r] + row_cost[m], r, m);
    else units.emplace_back(row_cost[r], r, -1);
  }
  std::sort(units.begin(), units.end(), [](const auto& x, const auto& y) {
    return std::get<0>(x) > std::get<0>(y) || (std::get<0>(x) == std::get<0>(y) && std::get<1>(x) < std::get<1>(y));
  });
  double load[msm::kShortWaves] = {};
  int count[msm::kShortWaves] = {};
  std::memset(g.short_rows, 0xff, sizeof(g.short_rows));
  std::memset(g.short_pair, 0xff, sizeof(g.short_pair));
  // a row r = (oz + R) side + oy + R is stored as its two offsets (R <= 4)
  auto code = [&](int r) { return (unsigned char)((r % side) | ((r / side) << 4)); };
  for (const auto& u : units) {
    int w = 0;
    for (int v = 1; v < msm::kShortWaves; ++v)
      if (count[v] < msm::kShortRowsPerWave && (count[w] >= msm::kShortRowsPerWave || load[v] < load[w])) w = v;
    g.short_rows[w][count[w]] = code(std::get<1>(u));
    if (std::get<2>(u) >= 0) g.short_pair[w][count[w]] = code(std::get<2>(u));
    ++count[w];
    load[w] += std::get<0>(u);
  }
}

// Short-range work items: each cell row's atoms are cut into 64-atom chunks;
// a row has row_items work items, item k taking chunks k, k + row_items, ...
// (sized for the row's expected atom count, so each item gets about
// item_chunks chunks; longer rows are still covered).
void set_row_items(Geom& g, int item_chunks, bool in_batch) {
  g.item_chunks = std::max(1, item_chunks);
  const double per_row = (double)g.n_atoms / ((double)g.nc[1] * g.nc[2]);
  const int chunks = std::max(1, (int)std::ceil(per_row / 64.0));
  g.row_items = std::max(1, (chunks + g.item_chunks - 1) / g.item_chunks);
  const int rows = g.nc[1] * g.nc[2];
  // a launch of at most one block per CU leaves the chip idle and lasts as long
  // as one wave's rows: 16 waves per item instead of 4, each wave's rows in
  // four parts (1,000 atoms in a cluster: k_short 45 -> 21 us, 9,000 periodic:
  // 70 -> 35; at 24,000 atoms and 400 items it still gains, 53 -> 33, but there
  // the grid stages beside it decide the time of an evaluation)
  g.short_parts = g.row_items * rows <= msm::kShortSmallItems ? msm::kShortParts : 1;
  // rows of an uneven cluster may be several times longer than the mean: a
  // small system on its own has blocks to spare for them
  if (g.short_parts > 1 && !in_batch) g.row_items = std::min(4 * g.row_items, std::max(g.row_items, msm::kShortSmallItems / rows));
}

void set_short_blocks(Geom& g, int cap) {
  const int items = g.row_items * g.nc[1] * g.nc[2];
  g.short_blocks = cap > 0 ? std::min(cap, items) : items;
}

// Link cells of edge >= a / reach along y and z (kXSub times finer along x;
// coarser if the cell count would exceed 8 n + 4096), the short-range row
// assignment and work items, and the binning path the cells allow: one kernel
// for small systems whose blocks own few enough cells (unless the plan prefers
// the two-kernel path, as in batches), else two kernels when the cell counts of
// every block fit (LDS, histogram size), else four by cell row when the rows
// fit, else four over the cells.
void set_cell_geometry(msm_plan* P, int reach) {
  Geom& g = P->g;
  const msm_params& p = P->p;
  const int n_atoms = g.n_atoms;
  const double amargin = p.cutoff * (1.0 + 1e-4);
  auto set_cells = [&](int r, double edge_min) {
    g.reach = r;
    long long tot = 1;
    for (int d = 0; d < 3; ++d) {
      int nc = (int)std::floor(p.box_len[d] / (d == 0 ? edge_min / msm::kXSub : edge_min));
      nc = std::max(1, std::min(nc, d == 0 ? 4096 : 1024));
      g.nc[d] = nc;
      g.inv_cs[d] = (float)(nc / p.box_len[d]);
      g.cs[d] = (float)(p.box_len[d] / nc);
      tot *= nc;
    }
    return tot;
  };
  const long long cap = 8LL * std::max(n_atoms, 1) + 4096;
  long long nct = set_cells(reach, amargin / reach);
  for (int r = reach - 1; r >= 1 && nct > cap; --r) nct = set_cells(r, amargin / r);
  if (nct > cap) {
    const double vol = p.box_len[0] * p.box_len[1] * p.box_len[2];
    nct = set_cells(1, std::max(amargin, std::cbrt(vol / (double)cap)));
  }
  g.n_cells = (int)nct;
  assign_short_rows(g);
  const int rows = g.nc[1] * g.nc[2];
  const int nbr = std::min(rows, msm::kBinRowMaxBlocks);
  const long long own = (long long)((rows + nbr - 1) / nbr) * g.nc[0];
  const long long nb = (n_atoms + msm::kBinChunk - 1) / msm::kBinChunk;
  P->bin2_blocks = (n_atoms > 0 && g.n_cells <= msm::kBinMaxCells && nb * g.n_cells <= msm::kBinMaxHist)
                       ? (int)nb : 0;
  // (every block of the one kernel walks all atoms of its system: right for a
  // single system's latency; in a batch the others are, 64 systems 1312 us
  // against 1357 with the one kernel for those of up to 32,768 atoms)
  const bool others = P->bin2_blocks > 0 || rows <= msm::kBinRowsMax;
  const bool one = n_atoms > 0 && n_atoms <= msm::kBinRowAtoms && own <= msm::kBinRowCells;
  g.bin_row_blocks = (one && !(P->in_batch && others)) ? nbr : 0;
  g.bin_blocks = g.bin_row_blocks == 0 ? P->bin2_blocks : 0;
  // otherwise by cell row first, then within each row, when the rows fit the
  // row binning's LDS histograms (else four kernels over the cells)
  const bool by_rows = n_atoms > 0 && g.bin_row_blocks == 0 && g.bin_blocks == 0 && rows <= msm::kBinRowsMax;
  g.binr_chunk = msm::kBinRChunk;
  if (!P->in_batch)
    for (g.binr_chunk = msm::kBinRMinChunk; g.binr_chunk < msm::kBinRChunk && n_atoms > msm::kBinRBlocks * g.binr_chunk;)
      g.binr_chunk *= 2;
  g.binr_blocks = by_rows ? (n_atoms + g.binr_chunk - 1) / g.binr_chunk : 0;
  set_row_items(g, g.item_chunks, P->in_batch);
  set_short_blocks(g, P->short_cap);
}

// Cell reach of a new plan: finer rows (higher reach) cut the short-range
// candidates that fail the cutoff test, but a 64-atom chunk of a thin row
// spans a long stretch of x, so every work item stages more atoms (on the
// 1M-atom water box reach 4 doubled the short-range time); the autotuner
// tries the finer cells.
int default_reach(int) { return 2; }

// Anterpolation tiles: start from 16 x 16 x 8 level-0 nodes and halve the
// largest side until there are at least `target` tiles (a launch then covers
// the 256 compute units twice).  Sides below 4 only while a tile has 128 atoms
// or more (a coarse grid, e.g. h = 10 A, has few nodes but as many atoms): the
// regions of smaller tiles are mostly overlap, which the gather adds up again
// (1,000 atoms on 12 nodes a side, tiles of 1 and of 4: anterpolation 6.6 and
// 6.8 us, gather 13.4 and 4.6; 9,000 atoms, order 6, tiles of 2 and 4: 17.0 and
// 10.5, 11.5 and 9.2).
void set_anterp_tiles(Geom& g, int target) {
  int t[3] = {16, 16, 8};
  auto tiles = [&]() {
    long long n = 1;
    for (int d = 0; d < 3; ++d) n *= (g.fmax[d] + t[d]) / t[d];
    return n;
  };
  while (tiles() < target) {
    int d = 0;
    for (int e = 1; e < 3; ++e)
      if (t[e] > t[d]) d = e;
    if (t[d] <= 1 || (t[d] <= 4 && g.n_atoms < 128 * tiles())) break;
    t[d] /= 2;
  }
  g.at_ext = 1;
  for (int d = 0; d < 3; ++d) {
    g.at[d] = t[d];
    g.atn[d] = (g.fmax[d] + t[d]) / t[d];              // tiles covering floor indices 0 .. fmax
    g.at_ext *= t[d] + g.order - 1;
  }
}

// A side stream's fork and join take the host 20 to 35 us (each wait of a
// stream for another's event 10 to 19, a launch 2.6), which is free only while
// the device is busy with earlier work, or in a graph.
//  - Systems whose rows are split finish the short range in 10 to 20 us: all on
//    one stream (1,000 atoms: 62 us; 70 with one side stream, 87 with two; 4,096
//    ions 72 us per step, 71, 91).  As a graph one side stream is right for them
//    too (48 us against 63 and 75), and periodic ones take it always: their grid
//    stages have twice the launches for the short range to hide behind (9,000
//    atoms: 123 us, 138 in order; as a graph 117, 135).
//  - The level-0 lattice cutoff beside the coarse levels costs nothing from
//    about 500 tiles and pays in batches (64 systems as a graph 1368 us, 1383
//    without; 16 systems 424 and 426; 1,000,000 atoms, 576 tiles: 1127 and 1126;
//    50,000, 63 tiles: 597 and 590; 24,000, 54 tiles: 140 and 104 as a graph).
void default_streams(msm::LaunchGeom& L, bool periodic) {
  L.streams = L.lattice0_tiles >= msm::kLattice0SideTiles && !periodic ? 3 : 2;
  L.capture_streams = L.streams;
  if (L.short_parts > 1 && !periodic) L.streams = 1;
}

void retune(msm_plan* P, const msm_tuning& t) {
  if (t.cell_reach != 0 && t.cell_reach != P->g.reach) set_cell_geometry(P, t.cell_reach);
  if (t.lattice_b && P->lat.b && t.lattice_b != P->lat.b)
    choose_lattice_tiles(P->g, P->lat.H, P->lat, t.lattice_b);
  Geom& g = P->g;
  if (t.item_chunks > 0) set_row_items(g, t.item_chunks, P->in_batch);
  if (t.short_blocks != 0) P->short_cap = t.short_blocks < 0 ? 0 : t.short_blocks;
  if (t.streams != 0) {
    P->streams = t.streams;
    P->streams_set = true;
  }
  if (t.short_after != 0) P->short_after = t.short_after;
  if (t.short_split != 0) P->short_split = t.short_split;
  set_short_blocks(g, P->short_cap);
  refresh_launch(P);
}

msm_status check_tuning(const msm_tuning* t) {
  if (!t) return fail(MSM_ERR_INVALID_ARG, "null tuning");
  if (t->lattice_b != 0 && t->lattice_b != 4 && t->lattice_b != 6 && t->lattice_b != 8)
    return fail(MSM_ERR_INVALID_ARG, "lattice_b must be 0, 4, 6 or 8");
  if (t->item_chunks < 0) return fail(MSM_ERR_INVALID_ARG, "item_chunks must be >= 0");
  if (t->short_blocks < -1) return fail(MSM_ERR_INVALID_ARG, "short_blocks must be >= -1");
  if (t->streams < 0 || t->streams > 3) return fail(MSM_ERR_INVALID_ARG, "streams must be 0 .. 3");
  if (t->short_after < 0 || t->short_after > 3) return fail(MSM_ERR_INVALID_ARG, "short_after must be 0 .. 3");
  if (t->short_split < 0 || t->short_split > 1000)
    return fail(MSM_ERR_INVALID_ARG, "short_split must be 0 .. 1000");
  if (t->cell_reach != 0 && (t->cell_reach < 2 || t->cell_reach > 4))
    return fail(MSM_ERR_INVALID_ARG, "cell_reach must be 0, 2, 3 or 4");
  if (t->reserved != 0) return fail(MSM_ERR_INVALID_ARG, "reserved tuning field must be zero");
  return MSM_OK;
}

hipError_t read_flags(const msm_plan* P, const char* ws, int32_t* flags) {
  int32_t w[msm::kStatusWords];
  const int nw = 64 + P->g.bin_row_blocks;
  hipError_t e = hipMemcpy(w, ws + P->lay.off[msm::kSecStatus], nw * sizeof(int32_t), hipMemcpyDeviceToHost);
  if (e != hipSuccess) return e;
  int32_t f = w[0];
  for (int b = 64; b < nw; ++b) f |= w[b];
  *flags = f;
  return hipSuccess;
}

msm::DevPtrs dev_ptrs(const msm_plan* P, void* ws) {
  char* b = static_cast<char*>(ws);
  const size_t* o = P->lay.off;
  msm::DevPtrs d;
  d.qgrid = (decltype(d.qgrid))(b + o[msm::kSecQGrid]);
  d.ucut = (decltype(d.ucut))(b + o[msm::kSecUCut]);
  d.u = (decltype(d.u))(b + o[msm::kSecU]);
  d.sorted = (decltype(d.sorted))(b + o[msm::kSecSorted]);
  d.perm = (decltype(d.perm))(b + o[msm::kSecPerm]);
  d.fshort = (decltype(d.fshort))(b + o[msm::kSecShort]);
  d.status = (decltype(d.status))(b + o[msm::kSecStatus]);
  d.counts = (decltype(d.counts))(b + o[msm::kSecCounts]);
  d.cell_start = (decltype(d.cell_start))(b + o[msm::kSecCellStart]);
  d.cursor = (decltype(d.cursor))(b + o[msm::kSecCursor]);
  d.cell_of = (decltype(d.cell_of))(b + o[msm::kSecCellOf]);
  d.tmp = (decltype(d.tmp))(b + o[msm::kSecTmp]);
  d.bin_hist = (decltype(d.bin_hist))(b + o[msm::kSecBinHist]);
  d.scan = (decltype(d.scan))(b + o[msm::kSecScan]);
  d.ant_part = (decltype(d.ant_part))(b + o[msm::kSecAntPart]);
  d.rows = (decltype(d.rows))(b + o[msm::kSecRows]);
  d.weights = (decltype(d.weights))(b + o[msm::kSecWeights]);
  d.lat_frags = (decltype(d.lat_frags))(b + o[msm::kSecLatFrags]);
  d.top = (decltype(d.top))(b + o[msm::kSecTop]);
  d.partials = (decltype(d.partials))(b + o[msm::kSecPartials]);
  d.lat_part = (decltype(d.lat_part))(b + o[msm::kSecAntPart]);
  d.excl_start = (decltype(d.excl_start))(P->excl_start);
  d.excl_idx = (decltype(d.excl_idx))(P->excl_idx);
  d.excl_nnz = P->excl_nnz;
  return d;
}

extern "C" {

const char* msm_status_string(msm_status s) {
  switch (s) {
    case MSM_OK: return "ok";
    case MSM_ERR_INVALID_ARG: return "invalid argument";
    case MSM_ERR_OUT_OF_BOX: return "atom outside the box";
    case MSM_ERR_NONFINITE: return "non-finite position or charge";
    case MSM_ERR_WORKSPACE: return "workspace missing or too small";
    case MSM_ERR_HIP: return "HIP runtime error";
    case MSM_ERR_UNSUPPORTED: return "unsupported configuration";
    case MSM_ERR_COINCIDENT: return "coincident atoms";
  }
  return "unknown status";
}

const char* msm_last_error(void) { return g_last_error.c_str(); }

msm_status msm_plan_create(const msm_params* prm, int32_t n_atoms, msm_plan** out) {
  if (!prm || !out) return fail(MSM_ERR_INVALID_ARG, "null params or output pointer");
  *out = nullptr;
  const msm_params& p = *prm;
  if (!finite_pos(p.cutoff)) return fail(MSM_ERR_INVALID_ARG, "cutoff must be finite and > 0");
  if (!finite_pos(p.spacing)) return fail(MSM_ERR_INVALID_ARG, "spacing must be finite and > 0");
  if (p.order != 4 && p.order != 6) return fail(MSM_ERR_INVALID_ARG, "order must be 4 or 6");
  if (p.split_m < 0 || p.split_m > 7) return fail(MSM_ERR_INVALID_ARG, "split_m must be in [0, 7]");
  if (p.levels < 0 || p.levels > msm::kMaxLevels)
    return fail(MSM_ERR_INVALID_ARG, "levels must be in [0, 12]");
  if (p.periodic != 0 && p.periodic != 1) return fail(MSM_ERR_INVALID_ARG, "periodic must be 0 or 1");
  if (n_atoms < 0) return fail(MSM_ERR_INVALID_ARG, "n_atoms must be >= 0");
  if (!std::isfinite(p.coulomb_k)) return fail(MSM_ERR_INVALID_ARG, "coulomb_k must be finite");
  for (int d = 0; d < 3; ++d) {
    if (!finite_pos(p.box_len[d])) return fail(MSM_ERR_INVALID_ARG, "box_len must be finite and > 0");
    if (!std::isfinite(p.box_lo[d])) return fail(MSM_ERR_INVALID_ARG, "box_lo must be finite");
  }
  // periodic grids: a whole number of nodes per period, halving at every level
  int per0[3] = {0, 0, 0};
  if (p.periodic) {
    for (int d = 0; d < 3; ++d) {
      const double t = p.box_len[d] / p.spacing;
      const double r = std::nearbyint(t);
      if (r < 1.0 || r > 1.0e6 || std::fabs(t - r) > 1e-9 * t)
        return fail(MSM_ERR_INVALID_ARG, "periodic: box_len / spacing must be an integer (at most 1e6)");
      if (2.0 * p.cutoff > p.box_len[d]) return fail(MSM_ERR_INVALID_ARG, "periodic: 2 cutoff must not exceed box_len");
      per0[d] = (int)r;
    }
  }

  msm_plan* P = new (std::nothrow) msm_plan();
  if (!P) return fail(MSM_ERR_INVALID_ARG, "out of host memory");
  static std::atomic<uint64_t> next_uid{1};
  P->uid = next_uid.fetch_add(1);
  P->p = p;
  Geom& g = P->g;
  std::memset(&g, 0, sizeof(g));
  const double a = p.cutoff, h = p.spacing;
  g.n_atoms = n_atoms;
  g.order = p.order;
  g.half = p.order / 2;
  g.h = (float)h;
  g.inv_h = (float)(1.0 / h);
  g.m = p.split_m ? p.split_m : p.order / 2;
  g.ke = p.coulomb_k != 0.0 ? p.coulomb_k : 1.0;
  double maxlen = 0.0;
  g.periodic = p.periodic;
  for (int d = 0; d < 3; ++d) {
    g.lo[d] = p.box_lo[d];
    g.hi[d] = p.box_lo[d] + p.box_len[d];
    g.lo_f[d] = (float)p.box_lo[d];
    g.len_f[d] = (float)p.box_len[d];
    g.len[d] = p.box_len[d];
    g.inv_len_f[d] = (float)(1.0 / p.box_len[d]);
    double fm = p.periodic ? (double)per0[d] : std::floor(p.box_len[d] / h);
    if (fm > 1.0e6) {
      delete P;
      return fail(MSM_ERR_UNSUPPORTED, "grid too fine for the box (more than 1e6 nodes per side)");
    }
    g.fmax[d] = (int)fm;
    maxlen = std::max(maxlen, p.box_len[d]);
  }

  // levels: given, or the fewest whose top interior spans <= 8 nodes per side
  // (periodic: whose top grid has <= 8 nodes per side, as far as the levels halve)
  int L = p.levels;
  if (L == 0 && p.periodic) {
    L = 1;
    for (;;) {
      bool big = false, even = true;
      for (int d = 0; d < 3; ++d) {
        big = big || (per0[d] >> (L - 1)) > 8;
        even = even && (per0[d] >> (L - 1)) % 2 == 0;
      }
      if (!big || !even || L == msm::kMaxLevels) break;
      ++L;
    }
  } else if (L == 0) {
    L = msm::kMaxLevels;
    for (int l = 1; l <= msm::kMaxLevels; ++l)
      if ((int)std::ceil(maxlen / std::ldexp(h, l - 1)) + 1 <= 8) {
        L = l;
        break;
      }
  }
  if (p.periodic)
    for (int d = 0; d < 3; ++d)
      if (per0[d] % (1 << (L - 1))) {
        delete P;
        return fail(MSM_ERR_INVALID_ARG, "periodic: box_len / spacing must be divisible by 2^(levels-1)");
      }
  g.levels = L;
  // periodic: level k holds its per0 / 2^k nodes of one period with ghost
  // copies on each side, as many as the widest stencil reaching past a period
  // needs (lattice half-width, restriction reach order - 1, basis support)
  if (p.periodic) {
    int H = 0;
    if (L > 1)
      while ((H + 1) * h < 2.0 * a) ++H;
    g.ghost = std::max({H, p.order - 1, g.half + 1});
  }
  // level 0 spans the nodes atoms in the box touch; level k+1 the nodes level k restricts to
  long long off = 0;
  for (int k = 0; k < L; ++k) {
    msm::Level& lv = g.lv[k];
    for (int d = 0; d < 3; ++d) {
      int lo, hi;
      if (p.periodic) {
        lv.per[d] = per0[d] >> k;
        lo = -g.ghost;
        hi = lv.per[d] - 1 + g.ghost;
      } else if (k == 0) {
        lo = -(g.half - 1);
        hi = g.fmax[d] + g.half;
      } else {
        const msm::Level& pv = g.lv[k - 1];
        lo = ceil_div2(pv.lo[d] - (p.order - 1));
        hi = floor_div2(pv.lo[d] + pv.n[d] - 1 + (p.order - 1));
      }
      lv.lo[d] = lo;
      lv.n[d] = hi - lo + 1;
    }
    long long cnt = (long long)lv.n[0] * lv.n[1] * lv.n[2];
    if (off + cnt > (1LL << 28)) {
      delete P;
      return fail(MSM_ERR_UNSUPPORTED, "grid hierarchy exceeds 2^28 nodes");
    }
    lv.off = (int)off;
    lv.count = (int)cnt;
    off += cnt;
  }
  g.total_nodes = (int)off;
  if (g.lv[L - 1].count > msm::kMaxTopNodes) {
    delete P;
    return fail(MSM_ERR_UNSUPPORTED, "top level too large for the all-pairs sum; use more levels");
  }

  set_anterp_tiles(g, msm::kAntTiles);
  // the lattice cutoff's partials live where the anterpolation's did, or in 8 MiB
  g.part_cap = std::max((long long)g.atn[0] * g.atn[1] * g.atn[2] * g.at_ext, 1048576LL);

  // smoothing constants
  double c[9];
  taylor_coeffs(g.m, c);
  for (int k = 0; k <= g.m; ++k) {
    g.dr[k] = (float)(2.0 * k * c[k] / std::pow(a, 2.0 * k + 1.0));
  }
  g.self = (float)(c[0] / a);
  g.inv_a = (float)(1.0 / a);
  g.inv_a2f = (float)(1.0 / (a * a));
  g.a2 = (float)(a * a);
  g.inv_a2 = (float)(1.0 / (a * a));

  // link cells: the finest reach any tuning may ask for sizes the cell
  // sections; the plan starts at the default reach
  g.a_win = (float)(a * (1.0 + 1e-4));
  g.item_chunks = 1;
  for (int r : {2, 3, 4}) {
    set_cell_geometry(P, r);
    P->max_cells = std::max(P->max_cells, g.n_cells);
    P->max_bin_hist = std::max(P->max_bin_hist, (long long)P->bin2_blocks * ((g.n_cells + 3) & ~3));
  }
  g.max_cells = P->max_cells;
  set_cell_geometry(P, default_reach(n_atoms));

  // lattice-cutoff stencil: W(n) = g^0(h |n|) for h |n| < 2a, rows along z
  if (L > 1) {
    const double rad = 2.0 * a / h;
    if (rad > 48.0) {
      delete P;
      return fail(MSM_ERR_UNSUPPORTED, "stencil radius 2a/h above 48 nodes");
    }
    int Rn = (int)std::ceil(rad);
    for (int nx = -Rn; nx <= Rn; ++nx)
      for (int ny = -Rn; ny <= Rn; ++ny) {
        int zr = -1;
        for (int nz = 0; nz <= Rn; ++nz) {
          double dist = h * std::sqrt((double)(nx * nx + ny * ny + nz * nz));
          if (dist < 2.0 * a) zr = nz;
        }
        if (zr < 0) continue;
        msm::StencilRow row{nx, ny, zr, (int)P->weights.size()};
        for (int nz = -zr; nz <= zr; ++nz) {
          double dist = h * std::sqrt((double)(nx * nx + ny * ny + nz * nz));
          double w0 = gamma_h(c, g.m, dist / a) / a - gamma_h(c, g.m, dist / (2.0 * a)) / (2.0 * a);
          P->weights.push_back((float)w0);
        }
        P->rows.push_back(row);
      }
  }
  // weight fragments of the tiled kernel
  if (L > 1) {
    int H = 0;
    for (const auto& r : P->rows) H = std::max(H, std::abs(r.nx));
    if (H <= msm::kLatMaxHalo) {
      auto weight = [&](int n2) {
        const double dist = h * std::sqrt((double)n2);
        return gamma_h(c, g.m, dist / a) / a - gamma_h(c, g.m, dist / (2.0 * a)) / (2.0 * a);
      };
      lattice_fragments(H, 2.0 * a / h, weight, P->lat, P->lat_frags);
      set_lattice_tiles(P, H);
    } else {
      P->lat.b = 0;
      P->lat.H = H;
    }
  }
  // top level (float64): T(d) = g^{l-1}(2^{l-1} h |d|) = gamma(r / A) / A, A = 2^{l-1} a
  // (periodic: the image sum K(d) over the node offsets of one period)
  if (p.periodic) {
    const msm::Level& T = g.lv[L - 1];
    periodic_top_table(c, g.m, std::ldexp(a, L - 1), std::ldexp(h, L - 1), T.per, p.box_len, P->top);
  } else {
    const msm::Level& T = g.lv[L - 1];
    const double A = std::ldexp(a, L - 1), hk = std::ldexp(h, L - 1);
    P->top.resize((size_t)T.count);
    for (int dz = 0; dz < T.n[2]; ++dz)
      for (int dy = 0; dy < T.n[1]; ++dy)
        for (int dx = 0; dx < T.n[0]; ++dx) {
          double r = hk * std::sqrt((double)(dx * dx + dy * dy + dz * dz));
          P->top[((size_t)dz * T.n[1] + dy) * T.n[0] + dx] = gamma_h(c, g.m, r / A) / A;
        }
  }
  P->n_partials = msm::interp_partials(g);

  // workspace layout
  Layout& lay = P->lay;
  size_t n = (size_t)std::max(n_atoms, 1);
  size_t nodes = (size_t)g.total_nodes;
  lay.bytes[msm::kSecQGrid] = nodes * sizeof(float);
  lay.bytes[msm::kSecUCut] = nodes * sizeof(float);
  lay.bytes[msm::kSecU] = nodes * sizeof(float);
  lay.bytes[msm::kSecSorted] = n * sizeof(float4);
  lay.bytes[msm::kSecPerm] = n * sizeof(int);
  lay.bytes[msm::kSecShort] = n * sizeof(float4);
  lay.bytes[msm::kSecStatus] = msm::kStatusWords * sizeof(int);
  lay.bytes[msm::kSecCounts] = ((size_t)P->max_cells + 1) * sizeof(int);
  lay.bytes[msm::kSecCellStart] = ((size_t)P->max_cells + 1) * sizeof(int);
  lay.bytes[msm::kSecCursor] = (size_t)P->max_cells * sizeof(int);
  lay.bytes[msm::kSecCellOf] = n * sizeof(int);
  lay.bytes[msm::kSecTmp] = n * sizeof(int);
  // sized for the two-kernel binning wherever it is possible (a batch may
  // switch a system to it)
  lay.bytes[msm::kSecBinHist] = std::max<size_t>((size_t)P->max_bin_hist, 1) * sizeof(int);
  // tile totals of the four-kernel binning's scan, or the row starts of the row binning
  lay.bytes[msm::kSecScan] = ((size_t)P->max_cells + 1) * sizeof(int);
  lay.bytes[msm::kSecRows] = std::max<size_t>(P->rows.size(), 1) * sizeof(msm::StencilRow);
  lay.bytes[msm::kSecWeights] = std::max<size_t>(P->weights.size(), 1) * sizeof(float);
  lay.bytes[msm::kSecLatFrags] = std::max<size_t>(P->lat_frags.size(), 1) * sizeof(uint16_t);
  lay.bytes[msm::kSecTop] = P->top.size() * sizeof(double);
  lay.bytes[msm::kSecPartials] = 10 * (size_t)P->n_partials * sizeof(double);
  lay.bytes[msm::kSecDesc] = sizeof(msm::SysDesc);
  // the anterpolation's partials and, once q^0 is gathered from them, the
  // lattice cutoff's share one section
  const size_t ant_bytes = (size_t)g.atn[0] * g.atn[1] * g.atn[2] * g.at_ext * sizeof(long long);
  auto place = [&]() {
    lay.bytes[msm::kSecAntPart] = std::max(ant_bytes, P->lat_part_max * sizeof(double));
    size_t o = 0;
    for (int s = 0; s < msm::kSecCount; ++s) {
      lay.off[s] = o;
      o += align256(lay.bytes[s]);
    }
    lay.total = o;
  };
  place();
  // a plan that the lattice's partials alone keep out of msm_compute_static
  // (many atoms on a small grid) splits its tiles less
  if (lay.total > msm::kStaticBytes && P->lat.b > 0 &&
      lay.total - align256(lay.bytes[msm::kSecAntPart]) + align256(ant_bytes) <= msm::kStaticBytes) {
    g.part_cap = (long long)(ant_bytes / sizeof(double));
    set_lattice_tiles(P, P->lat.H);
    place();
  }

  refresh_launch(P);
  *out = P;
  return MSM_OK;
}

msm_status msm_pair_plan_create(const msm_pair_params* pp, int32_t n_atoms, msm_plan** out) {
  if (!pp || !out) return fail(MSM_ERR_INVALID_ARG, "null params or output pointer");
  *out = nullptr;
  if (pp->kind < MSM_PAIR_CUTOFF || pp->kind > MSM_PAIR_WOLF)
    return fail(MSM_ERR_INVALID_ARG, "kind must be MSM_PAIR_CUTOFF, MSM_PAIR_SHIFTED_FORCE or MSM_PAIR_WOLF");
  if (pp->periodic != 0 && pp->periodic != 1) return fail(MSM_ERR_INVALID_ARG, "periodic must be 0 or 1");
  if (!finite_pos(pp->cutoff)) return fail(MSM_ERR_INVALID_ARG, "cutoff must be finite and > 0");
  for (int d = 0; d < 3; ++d)
    if (pp->periodic && finite_pos(pp->box_len[d]) && 2.0 * pp->cutoff > pp->box_len[d])
      return fail(MSM_ERR_INVALID_ARG, "periodic: 2 cutoff must not exceed box_len");
  if (!std::isfinite(pp->alpha) || pp->alpha < 0.0) return fail(MSM_ERR_INVALID_ARG, "alpha must be finite and >= 0");
  // the cells, binning and short-range pass of an MSM plan with cutoff rc; its
  // (unused) grid is one coarse level
  msm_params p{};
  p.cutoff = pp->cutoff;
  double maxlen = 0.0;
  for (int d = 0; d < 3; ++d) {
    p.box_lo[d] = pp->box_lo[d];
    p.box_len[d] = pp->box_len[d];
    if (std::isfinite(pp->box_len[d])) maxlen = std::max(maxlen, pp->box_len[d]);
  }
  p.spacing = std::max(pp->cutoff, maxlen / 8.0);
  p.order = 4;
  p.levels = 1;
  p.coulomb_k = pp->coulomb_k;
  msm_plan* P = nullptr;
  msm_status st = msm_plan_create(&p, n_atoms, &P);
  if (st != MSM_OK) return st;
  Geom& g = P->g;
  const double rc = pp->cutoff, al = pp->alpha;
  g.pair = pp->kind;
  g.periodic = pp->periodic;                     // pairs at their nearest image (the grid is unused)
  assign_short_rows(g);                          // periodic plans walk rows one at a time
  g.pk[0] = g.pk[1] = g.pk[2] = g.pk[3] = 0.f;
  g.self = 0.f;
  if (pp->kind == MSM_PAIR_SHIFTED_FORCE) {
    g.pk[0] = (float)(1.0 / rc);
    g.pk[1] = (float)(1.0 / (rc * rc));
  } else if (pp->kind == MSM_PAIR_WOLF) {
    const double two_over_sqrt_pi = 1.1283791670955126;
    g.pk[0] = (float)al;
    g.pk[1] = (float)(std::erfc(al * rc) / rc);
    g.pk[2] = (float)(al * two_over_sqrt_pi);
    g.pk[3] = (float)(-al * al * 1.4426950408889634);   // -alpha^2 log2(e)
    // every pair the device evaluates has alpha r <= alpha rc (the r < rc test,
    // with float rounding to spare); below x = 1 the fit is as good and beyond
    // x = 10 erfc(x) exp(-x^2) underflows float
    const double x_hi = std::min(std::max(al * rc * (1.0 + 1e-3), 1.0), 10.0);
    if (fit_wolf_erfc(x_hi, g.ec) > 1e-7) {
      msm_plan_destroy(P);
      return fail(MSM_ERR_UNSUPPORTED, "Wolf erfc fit failed");
    }
    // phi_i gains 2 s q_i with s = -(erfc(alpha rc)/(2 rc) + alpha/sqrt(pi)); the
    // assembly subtracts q_i self
    g.self = (float)(std::erfc(al * rc) / rc + al * two_over_sqrt_pi);
  }
  P->pp = *pp;
  refresh_launch(P);
  *out = P;
  return MSM_OK;
}

msm_status msm_plan_destroy(msm_plan* plan) {
  if (plan) {
    for (auto& e : plan->ev)
      if (e) (void)hipEventDestroy(e);
    destroy_aux(plan->aux);
  }
  delete plan;
  return MSM_OK;
}

msm_status msm_profile_enable(msm_plan* P, int32_t enable) {
  if (!P) return fail(MSM_ERR_INVALID_ARG, "null plan");
  if (enable < 0 || enable > 2) return fail(MSM_ERR_INVALID_ARG, "profile mode must be 0, 1 or 2");
  if (enable && !P->ev[0])
    for (auto& e : P->ev) {
      hipError_t r = hipEventCreate(&e);
      if (r != hipSuccess) return hip_fail(r, "create timing events");
    }
  P->profile = enable;
  P->profiled = false;
  return MSM_OK;
}

msm_status msm_profile_read(const msm_plan* P, float* ms, int32_t* n_stages) {
  if (!P || !ms || !n_stages) return fail(MSM_ERR_INVALID_ARG, "null argument");
  if (!P->profile) return fail(MSM_ERR_INVALID_ARG, "profiling is not enabled on this plan");
  if (!P->profiled) return fail(MSM_ERR_INVALID_ARG, "no evaluation was timed since profiling was enabled");
  hipError_t r;
  if (P->profile == 1) {
    r = hipEventSynchronize(P->ev[msm::kStageCount]);
    if (r != hipSuccess) return hip_fail(r, "wait for timing events");
    for (int i = 0; i < msm::kStageCount; ++i) {
      r = hipEventElapsedTime(&ms[i], P->ev[i], P->ev[i + 1]);
      if (r != hipSuccess) return hip_fail(r, "read timing events");
    }
  } else {
    float slot[msm::kLiveSlots];
    for (int i = 0; i < msm::kLiveSlots; ++i) {
      r = hipEventSynchronize(P->ev[msm::kLiveSlots + i]);
      if (r == hipSuccess) r = hipEventElapsedTime(&slot[i], P->ev[i], P->ev[msm::kLiveSlots + i]);
      if (r != hipSuccess) return hip_fail(r, "read timing events");
    }
    for (int i = 0; i < msm::kStageCount; ++i) ms[i] = slot[i];
    ms[msm::kStageShort] += slot[msm::kSlotShort2];
    ms[msm::kStageLattice] += slot[msm::kSlotLattice0];
  }
  *n_stages = msm::kStageCount;
  return MSM_OK;
}

msm_status msm_plan_info(const msm_plan* P, int32_t* levels, int32_t* grid_lo, int32_t* grid_n) {
  if (!P || !levels) return fail(MSM_ERR_INVALID_ARG, "null plan or levels pointer");
  *levels = P->g.levels;
  for (int k = 0; k < P->g.levels; ++k)
    for (int d = 0; d < 3; ++d) {
      if (grid_lo) grid_lo[3 * k + d] = P->g.lv[k].lo[d];
      if (grid_n) grid_n[3 * k + d] = P->g.lv[k].n[d];
    }
  return MSM_OK;
}

msm_status msm_plan_describe(const msm_plan* P, char* buf, size_t buf_bytes) {
  if (!P || !buf || buf_bytes == 0) return fail(MSM_ERR_INVALID_ARG, "null plan or buffer");
  const Geom& g = P->g;
  std::string o = "{";
  o += "\"pair\": " + std::to_string(g.pair) + ", \"levels\": " + std::to_string(g.levels);
  o += ", \"cells\": [" + std::to_string(g.nc[0]) + ", " + std::to_string(g.nc[1]) + ", " +
       std::to_string(g.nc[2]) + "], \"reach\": " + std::to_string(g.reach) +
       ", \"bin_blocks\": " + std::to_string(g.bin_blocks) +
       ", \"bin_row_blocks\": " + std::to_string(g.bin_row_blocks) + ", \"binr_blocks\": " +
       std::to_string(g.binr_blocks) +
       ", \"item_chunks\": " + std::to_string(g.item_chunks) + ", \"short_blocks\": " + std::to_string(g.short_blocks) +
       ", \"short_parts\": " + std::to_string(g.short_parts) +
       ", \"streams\": " + std::to_string(P->streams) + ", \"layout\": " + std::to_string(P->lg.streams) +
       ", \"graph_layout\": " + std::to_string(P->lg.capture_streams) + ", \"short_after\": " + std::to_string(P->short_after) +
       ", \"short_split\": " + std::to_string(P->short_split);
  o += ", \"taps\": " + std::to_string(P->weights.size()) + ", \"halo\": " + std::to_string(P->lat.H);
  o += ", \"lattice_b\": " + std::to_string(P->lat.b) + ", \"lattice_waves\": " + std::to_string(P->lat.b > 0 ? msm::lat_waves(P->lat.b) : 0) +
       ", \"lattice_lds\": " +
       std::to_string(P->lat.lds_bytes) + ", \"lattice_tiles\": [";
  for (int k = 0; k < P->lat.n; ++k) {
    const msm::LatTile& t = P->lat.t[k];
    if (k) o += ", ";
    o += "[16, 16, " + std::to_string(P->lat.b) + ", " + std::to_string(t.ntx * t.nty * t.ntz) + ", " +
         std::to_string(t.groups) + "]";
  }
  o += "], \"prolong_per_level\": " + std::to_string(P->lg.prolong_split ? 1 : 0);
  o += ", \"periodic\": " + std::to_string(g.periodic) + ", \"ghost\": " + std::to_string(g.ghost);
  o += ", \"workspace_bytes\": " + std::to_string(P->lay.total) + "}";
  std::strncpy(buf, o.c_str(), buf_bytes - 1);
  buf[buf_bytes - 1] = 0;
  return o.size() < buf_bytes ? MSM_OK : fail(MSM_ERR_INVALID_ARG, "buffer too small");
}

msm_status msm_workspace_bytes(const msm_plan* P, size_t* bytes) {
  if (!P || !bytes) return fail(MSM_ERR_INVALID_ARG, "null plan or bytes pointer");
  *bytes = P->lay.total;
  return MSM_OK;
}

msm_status msm_workspace_section(const msm_plan* P, int32_t section, size_t* offset, size_t* bytes) {
  if (!P || section < 0 || section > msm::kSecShort)
    return fail(MSM_ERR_INVALID_ARG, "null plan or unknown section");
  if (offset) *offset = P->lay.off[section];
  if (bytes) *bytes = P->lay.bytes[section];
  return MSM_OK;
}


}  // extern "C"

// Upload the plan's tables and descriptor into the workspace at ws (device)
// and clear its cell counters, on stream s; waits for the copies (they read
// pageable host memory of the plan).
msm_status init_workspace(const msm_plan* P, void* ws, hipStream_t s) {
  char* base = static_cast<char*>(ws);
  hipError_t e;
  if (!P->rows.empty()) {
    e = hipMemcpyAsync(base + P->lay.off[msm::kSecRows], P->rows.data(),
                       P->rows.size() * sizeof(msm::StencilRow), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "upload stencil rows");
    e = hipMemcpyAsync(base + P->lay.off[msm::kSecWeights], P->weights.data(),
                       P->weights.size() * sizeof(float), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return hip_fail(e, "upload stencil weights");
    if (!P->lat_frags.empty()) {
      e = hipMemcpyAsync(base + P->lay.off[msm::kSecLatFrags], P->lat_frags.data(),
                         P->lat_frags.size() * sizeof(uint16_t), hipMemcpyHostToDevice, s);
      if (e != hipSuccess) return hip_fail(e, "upload stencil fragments");
    }
  }
  e = hipMemcpyAsync(base + P->lay.off[msm::kSecTop], P->top.data(), P->top.size() * sizeof(double),
                     hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail(e, "upload top-level table");
  msm_plan* M = const_cast<msm_plan*>(P);
  M->desc.d = dev_ptrs(P, ws);
  e = hipMemcpyAsync(base + P->lay.off[msm::kSecDesc], &M->desc, sizeof(msm::SysDesc),
                     hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail(e, "upload descriptor");
  msm::LaunchGeom L = P->lg;
  L.sys = reinterpret_cast<const msm::SysDesc*>(base + P->lay.off[msm::kSecDesc]);
  e = msm::launch_init(L, s);
  if (e != hipSuccess) return hip_fail(e, "clear cell counters");
  // pageable-memory copies are staged before returning; the plan may be destroyed afterwards
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "workspace init");
  return MSM_OK;
}

extern "C" {

msm_status msm_workspace_init(const msm_plan* P, void* ws, size_t ws_bytes, msm_stream_t stream) {
  if (!P) return fail(MSM_ERR_INVALID_ARG, "null plan");
  if (!ws || ws_bytes < P->lay.total) return fail(MSM_ERR_WORKSPACE, "workspace missing or too small");
  const msm_status st = init_workspace(P, ws, reinterpret_cast<hipStream_t>(stream));
  if (st != MSM_OK) return st;
  const_cast<msm_plan*>(P)->ready.insert(ws);
  return MSM_OK;
}


static msm::LaunchGeom launch_geom(const msm_plan* P, void* ws) {
  msm::LaunchGeom L = P->lg;
  L.sys = reinterpret_cast<const msm::SysDesc*>(static_cast<char*>(ws) + P->lay.off[msm::kSecDesc]);
  return L;
}

static msm_status check_call(const msm_plan* P, const void* ws, size_t ws_bytes, const float* x,
                             const float* y, const float* z, const float* q, const float* fx,
                             const float* fy, const float* fz) {
  if (!P) return fail(MSM_ERR_INVALID_ARG, "null plan");
  if (!ws || ws_bytes < P->lay.total) return fail(MSM_ERR_WORKSPACE, "workspace missing or too small");
  if (!P->ready.count(ws)) return fail(MSM_ERR_WORKSPACE, "workspace not initialised for this plan");
  if (P->g.n_atoms > 0 && (!x || !y || !z || !q))
    return fail(MSM_ERR_INVALID_ARG, "null position or charge array");
  if (!((fx && fy && fz) || (!fx && !fy && !fz)))
    return fail(MSM_ERR_INVALID_ARG, "vector outputs must be all set or all null");
  return MSM_OK;
}

}  // extern "C"

msm_status plan_eval(const msm_plan* P, void* ws, size_t ws_bytes, msm_stream_t stream, const msm::Io& io,
                     bool potential) {
  msm_status st = check_call(P, ws, ws_bytes, io.x, io.y, io.z, io.q, io.fx, io.fy, io.fz);
  if (st != MSM_OK) return st;
  msm_plan* M = const_cast<msm_plan*>(P);
  std::lock_guard<std::mutex> lock(M->aux.mu);
  hipError_t e = ensure_aux(M->aux);
  if (e != hipSuccess) return hip_fail(e, "create auxiliary stream");
  msm::LaunchGeom L = launch_geom(P, ws);
  L.potential = potential;
  e = msm::launch_eval(msm::kModeForces, L, reinterpret_cast<hipStream_t>(stream), io,
                       P->profile ? M->ev : nullptr, &M->aux.cc, P->profile == 2);
  if (P->profile) M->profiled = true;
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  return MSM_OK;
}

extern "C" {

msm_status msm_compute(const msm_plan* P, void* ws, size_t ws_bytes, msm_stream_t stream,
                       const float* x, const float* y, const float* z, const float* q, float* fx,
                       float* fy, float* fz, float* phi, double* energy, double* virial) {
  return plan_eval(P, ws, ws_bytes, stream, msm::Io{x, y, z, q, fx, fy, fz, phi, energy, virial, nullptr}, false);
}

static msm_status eval_mode(int mode, const msm_plan* P, void* ws, size_t ws_bytes,
                            msm_stream_t stream, const float* x, const float* y, const float* z,
                            const float* q, float* fx, float* fy, float* fz, float* phi,
                            double* energy, const double* gscale) {
  msm_status st = check_call(P, ws, ws_bytes, x, y, z, q, fx, fy, fz);
  if (st != MSM_OK) return st;
  msm_plan* M = const_cast<msm_plan*>(P);
  std::lock_guard<std::mutex> lock(M->aux.mu);
  hipError_t e = ensure_aux(M->aux);
  if (e != hipSuccess) return hip_fail(e, "create auxiliary stream");
  const msm::Io io{x, y, z, q, fx, fy, fz, phi, energy, nullptr, gscale};
  e = msm::launch_eval(mode, launch_geom(P, ws), reinterpret_cast<hipStream_t>(stream), io, nullptr,
                       &M->aux.cc);
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  return MSM_OK;
}

msm_status msm_energy(const msm_plan* P, void* ws, size_t ws_bytes, msm_stream_t stream,
                      const float* x, const float* y, const float* z, const float* q,
                      double* energy) {
  if (!energy) return fail(MSM_ERR_INVALID_ARG, "null energy output");
  if (P && P->g.pair) return fail(MSM_ERR_UNSUPPORTED, "msm_energy is for multilevel-summation plans");
  return eval_mode(msm::kModeEnergy, P, ws, ws_bytes, stream, x, y, z, q, nullptr, nullptr, nullptr,
                   nullptr, energy, nullptr);
}

msm_status msm_backward(const msm_plan* P, void* ws, size_t ws_bytes, msm_stream_t stream,
                        const float* x, const float* y, const float* z, const float* q,
                        const double* grad_energy, float* dedx, float* dedy, float* dedz,
                        float* dedq) {
  if (!grad_energy) return fail(MSM_ERR_INVALID_ARG, "null grad_energy");
  if (P && P->g.pair) return fail(MSM_ERR_UNSUPPORTED, "msm_backward is for multilevel-summation plans");
  return eval_mode(msm::kModeGradient, P, ws, ws_bytes, stream, x, y, z, q, dedx, dedy, dedz, dedq,
                   nullptr, grad_energy);
}

msm_status msm_graph_destroy(msm_graph* G) {
  if (G) {
    if (G->exec) (void)hipGraphExecDestroy(G->exec);
    if (G->graph) (void)hipGraphDestroy(G->graph);
    delete G;
  }
  return MSM_OK;
}

msm_status msm_graph_capture(const msm_plan* P, void* ws, size_t ws_bytes, const float* x,
                             const float* y, const float* z, const float* q, float* fx, float* fy,
                             float* fz, float* phi, double* energy, double* virial, msm_graph** out) {
  if (!out) return fail(MSM_ERR_INVALID_ARG, "null output pointer");
  *out = nullptr;
  msm_status st = check_call(P, ws, ws_bytes, x, y, z, q, fx, fy, fz);
  if (st != MSM_OK) return st;
  msm_plan* M = const_cast<msm_plan*>(P);
  std::lock_guard<std::mutex> lock(M->aux.mu);
  hipError_t e = ensure_aux(M->aux);
  if (e != hipSuccess) return hip_fail(e, "create auxiliary stream");
  const msm::Io io{x, y, z, q, fx, fy, fz, phi, energy, virial, nullptr};
  msm::LaunchGeom L = launch_geom(P, ws);
  L.streams = L.capture_streams;
  return capture_graph(
      [&](hipStream_t cs) {
        return msm::launch_eval(msm::kModeForces, L, cs, io, nullptr, &M->aux.cc);
      },
      &M->tune_gen, out);
}

msm_status msm_graph_launch(const msm_graph* G, msm_stream_t stream) {
  if (!G || !G->exec) return fail(MSM_ERR_INVALID_ARG, "null graph");
  if (G->owner_gen && *G->owner_gen != G->gen)
    return fail(MSM_ERR_INVALID_ARG, "the plan or batch was re-tuned after this graph was captured");
  hipError_t e = hipGraphLaunch(G->exec, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "graph launch");
  return MSM_OK;
}

msm_status msm_status_query(const msm_plan* P, const void* ws, msm_stream_t stream,
                            int32_t* device_flags) {
  if (!P || !ws) return fail(MSM_ERR_INVALID_ARG, "null plan or workspace");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipError_t e = hipStreamSynchronize(s);
  if (e != hipSuccess) return hip_fail(e, "stream synchronize");
  int32_t flags = 0;
  e = read_flags(P, static_cast<const char*>(ws), &flags);
  if (e != hipSuccess) return hip_fail(e, "read status");
  if (device_flags) *device_flags = flags;
  if (flags & msm::kFlagNonFinite) return fail(MSM_ERR_NONFINITE, "non-finite position or charge");
  if (flags & msm::kFlagOutOfBox) return fail(MSM_ERR_OUT_OF_BOX, "atom outside the box");
  if (flags & msm::kFlagCoincident) return fail(MSM_ERR_COINCIDENT, "coincident atoms");
  if (flags & msm::kFlagBadExclusion) return fail(MSM_ERR_INVALID_ARG, "exclusion list entry out of range");
  return MSM_OK;
}

}  // extern "C"
