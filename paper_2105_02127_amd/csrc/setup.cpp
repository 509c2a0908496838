// Host set-up of libteno: geometry, faces, stencils, reference-space least
// squares and the device-ready packed layouts.  Runs once per mesh; the
// per-stage work happens in the HIP kernels.
//
//  * geometry and faces ............. Sec. 2.1 (semi-discrete form)
//  * stencils ........................ Sec. 3.1: central stencil of 2N_k cells
//    (the target and its 2N_k-1 nearest cells by periodic centroid distance)
//    and three third-order directional stencils (the target and the 11 nearest
//    cells whose centroid lies in the closed cone from the target centroid
//    through the two endpoints of one local edge); ties by lower user id.
//  * least squares ................... Sec. 2.2 eqs. 02-10: affine map of the
//    target onto the reference triangle, zero-mean monomial basis, rows
//    A_sl = int_{V'_s} psi_l, Householder QR, operator M = pinv(A) diag|V'_s|.
//    Monomial integrals use Radon's 7-point degree-5 rule (exact for every
//    basis function up to degree 5, i.e. order 6).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <thread>
#include <utility>

#include "internal.h"

namespace teno {

static thread_local std::string g_error;

void set_error(const std::string& msg) { g_error = msg; }
int fail(int code, const std::string& msg) {
  g_error = msg;
  return code;
}
const char* last_error() { return g_error.c_str(); }

Dims dims_for(int order, int nq_req) {
  Dims d;
  d.order = order;
  d.r = order - 1;
  int nk = (d.r + 1) * (d.r + 2) / 2;
  d.nu = nk - 1;
  d.nl = 2 * nk - 1;
  d.nq = nq_req > 0 ? nq_req : (order + 1) / 2;
  d.rows = 3 * kSmallRows + d.nl;
  d.rows4 = (d.rows + 3) / 4;
  d.J = 3 * kSmallCoef * kSmallRows + d.nu * d.nl;
  return d;
}

// ---------------------------------------------------------------------------
// simple parallel-for over [0, n) with std::thread
// ---------------------------------------------------------------------------
template <class F>
static void parallel_for(int n, int threads, F&& f, int chunk = 64) {
  if (threads <= 0) threads = (int)std::max(1u, std::thread::hardware_concurrency());
  threads = std::min(threads, std::max(1, n / chunk));
  if (threads <= 1) {
    for (int i = 0; i < n; ++i) f(i);
    return;
  }
  std::atomic<int> next{0};
  std::vector<std::thread> pool;
  for (int t = 0; t < threads; ++t)
    pool.emplace_back([&]() {
      for (;;) {
        int b = next.fetch_add(chunk);
        if (b >= n) break;
        int e = std::min(n, b + chunk);
        for (int i = b; i < e; ++i) f(i);
      }
    });
  for (auto& th : pool) th.join();
}

// ---------------------------------------------------------------------------
// geometry
// ---------------------------------------------------------------------------
// Minimum-image difference on the periodic axes (kx, ky: periods removed).
static inline void wrap_delta(const Mesh& m, double& dx, double& dy, double& kx, double& ky) {
  kx = ky = 0.0;
  if (m.P[0] > 0.0) {
    kx = std::nearbyint(dx / m.P[0]);
    dx -= m.P[0] * kx;
  }
  if (m.P[1] > 0.0) {
    ky = std::nearbyint(dy / m.P[1]);
    dy -= m.P[1] * ky;
  }
}

int mesh_create(int32_t n_vert, const double* xy, int32_t n_cell, const int32_t* tri,
                const double* period, Mesh& m) {
  if (n_vert <= 0 || n_cell <= 0 || !xy || !tri) return fail(TENO_EARG, "empty mesh");
  m.nv = n_vert;
  m.nc = n_cell;
  if (period) {
    m.P[0] = period[0];
    m.P[1] = period[1];
    if (!(m.P[0] >= 0.0 && m.P[1] >= 0.0))
      return fail(TENO_EARG, "period must be positive, or 0 for an open axis");
  }
  m.tri.assign(tri, tri + 3 * (size_t)n_cell);
  m.X.resize(6 * (size_t)n_cell);
  m.area.resize(n_cell);
  m.cen.resize(2 * (size_t)n_cell);
  for (int i = 0; i < n_cell; ++i) {
    int32_t* t = &m.tri[3 * (size_t)i];
    double px[3], py[3];
    for (int v = 0; v < 3; ++v) {
      if (t[v] < 0 || t[v] >= n_vert) return fail(TENO_EMESH, "vertex id out of range");
      px[v] = xy[2 * (size_t)t[v]];
      py[v] = xy[2 * (size_t)t[v] + 1];
    }
    for (int v = 1; v < 3; ++v) {
      double dx = px[v] - px[0], dy = py[v] - py[0], kx, ky;
      wrap_delta(m, dx, dy, kx, ky);
      px[v] = px[0] + dx;
      py[v] = py[0] + dy;
    }
    double twice = (px[1] - px[0]) * (py[2] - py[0]) - (px[2] - px[0]) * (py[1] - py[0]);
    if (twice < 0.0) {
      std::swap(t[1], t[2]);
      std::swap(px[1], px[2]);
      std::swap(py[1], py[2]);
      twice = -twice;
    }
    if (!(twice > 0.0)) return fail(TENO_EMESH, "degenerate triangle " + std::to_string(i));
    m.area[i] = 0.5 * twice;
    for (int v = 0; v < 3; ++v) {
      m.X[6 * (size_t)i + 2 * v] = px[v];
      m.X[6 * (size_t)i + 2 * v + 1] = py[v];
    }
    m.cen[2 * (size_t)i] = (px[0] + px[1] + px[2]) / 3.0;
    m.cen[2 * (size_t)i + 1] = (py[0] + py[1] + py[2]) / 3.0;
  }
  for (int a = 0; a < 2; ++a) {
    if (m.P[a] > 0.0) {
      m.lo[a] = 0.0;
      m.hi[a] = m.P[a];
      continue;
    }
    m.lo[a] = m.hi[a] = m.cen[a];
    for (int i = 0; i < n_cell; ++i) {
      m.lo[a] = std::min(m.lo[a], m.cen[2 * (size_t)i + a]);
      m.hi[a] = std::max(m.hi[a], m.cen[2 * (size_t)i + a]);
    }
    if (!(m.hi[a] > m.lo[a])) m.hi[a] = m.lo[a] + 1.0;
  }
  // Faces from directed edges: key (a, b) -> half-edge 3*cell+e.  An
  // undirected edge is one face; L is the cell with the lower user id.
  const size_t nh = 3 * (size_t)n_cell;
  std::vector<uint64_t> key(nh);
  std::vector<int32_t> order(nh);
  for (int i = 0; i < n_cell; ++i)
    for (int e = 0; e < 3; ++e) {
      uint64_t a = (uint32_t)m.tri[3 * (size_t)i + e], b = (uint32_t)m.tri[3 * (size_t)i + (e + 1) % 3];
      key[3 * (size_t)i + e] = (a << 32) | b;
    }
  for (size_t h = 0; h < nh; ++h) order[h] = (int32_t)h;
  std::sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return key[x] < key[y]; });
  for (size_t h = 1; h < nh; ++h)
    if (key[order[h]] == key[order[h - 1]]) return fail(TENO_EMESH, "non-manifold edge");
  m.cface.assign(nh, -1);
  for (size_t h = 0; h < nh; ++h) {
    int32_t he = order[h];
    uint64_t k = key[he];
    uint64_t twin = (k << 32) | (k >> 32);
    auto it = std::lower_bound(order.begin(), order.end(), twin,
                               [&](int32_t x, uint64_t v) { return key[x] < v; });
    const int ci = he / 3, ce = he % 3;
    if (it == order.end() || key[*it] != twin) {
      // an edge with one cell: a boundary face, allowed on meshes with an open axis
      if (!m.open()) return fail(TENO_EMESH, "open edge on a mesh periodic in both axes");
      int f = m.nf++;
      m.fL.push_back(ci);
      m.fLe.push_back(ce);
      m.fR.push_back(-1);
      m.fRe.push_back(-1);
      const double* X = &m.X[6 * (size_t)ci];
      double ex = X[2 * ((ce + 1) % 3)] - X[2 * ce];
      double ey = X[2 * ((ce + 1) % 3) + 1] - X[2 * ce + 1];
      double len = std::sqrt(ex * ex + ey * ey);
      m.flen.push_back(len);
      m.fnx.push_back(ey / len);
      m.fny.push_back(-ex / len);
      m.cface[3 * (size_t)ci + ce] = f;
      m.bface.push_back(f);
      continue;
    }
    int32_t ho = *it;
    int co = ho / 3, coe = ho % 3;
    if (co < ci || (co == ci && coe < ce)) continue;  // created from the other side
    int f = m.nf++;
    m.fL.push_back(ci);
    m.fLe.push_back(ce);
    m.fR.push_back(co);
    m.fRe.push_back(coe);
    const double* X = &m.X[6 * (size_t)ci];
    double ex = X[2 * ((ce + 1) % 3)] - X[2 * ce];
    double ey = X[2 * ((ce + 1) % 3) + 1] - X[2 * ce + 1];
    double len = std::sqrt(ex * ex + ey * ey);
    m.flen.push_back(len);
    m.fnx.push_back(ey / len);
    m.fny.push_back(-ex / len);
    m.cface[3 * (size_t)ci + ce] = f;
    m.cface[3 * (size_t)co + coe] = f;
  }
  m.bkind.assign(m.bface.size(), TENO_BC_TRANSMISSIVE);
  m.bstate.assign(4 * m.bface.size(), 0.0);
  return TENO_OK;
}

// ---------------------------------------------------------------------------
// neighbour search: uniform bins over the box (periodic axes wrap), search
// radius grown until the wanted count is found strictly inside the covered
// disc or every bin is covered
// ---------------------------------------------------------------------------
struct Bins {
  int n = 1;
  double wx = 1.0, wy = 1.0;
  std::vector<int32_t> start, cells;
};

// Bin coordinate of a centroid along axis a (periodic axes wrap).
static inline double bin_coord(const Mesh& m, int a, double x) {
  if (m.P[a] > 0.0) return x - m.P[a] * std::floor(x / m.P[a]);
  return x - m.lo[a];
}

static void bins_build(const Mesh& m, Bins& b) {
  double lx = m.hi[0] - m.lo[0], ly = m.hi[1] - m.lo[1];
  b.n = std::max(1, (int)std::floor(std::sqrt(m.nc * 0.5)));
  b.wx = lx / b.n;
  b.wy = ly / b.n;
  std::vector<int32_t> id(m.nc);
  b.start.assign((size_t)b.n * b.n + 1, 0);
  for (int i = 0; i < m.nc; ++i) {
    double x = bin_coord(m, 0, m.cen[2 * (size_t)i]), y = bin_coord(m, 1, m.cen[2 * (size_t)i + 1]);
    int bx = std::min(b.n - 1, std::max(0, (int)(x / b.wx)));
    int by = std::min(b.n - 1, std::max(0, (int)(y / b.wy)));
    id[i] = by * b.n + bx;
    b.start[id[i] + 1]++;
  }
  for (int k = 0; k < b.n * b.n; ++k) b.start[k + 1] += b.start[k];
  b.cells.resize(m.nc);
  std::vector<int32_t> pos(b.start.begin(), b.start.end() - 1);
  for (int i = 0; i < m.nc; ++i) b.cells[pos[id[i]]++] = i;
}

struct Hit {
  double d2;
  int32_t id;
};

static inline bool hit_less(const Hit& a, const Hit& b) {
  return a.d2 < b.d2 || (a.d2 == b.d2 && a.id < b.id);
}

// Closed cone test for directional stencil k of cell i (k = 3: everything).
static inline bool cone_ok(const Mesh& m, int i, int k, double dx, double dy) {
  if (k == 3) return true;
  const double* X = &m.X[6 * (size_t)i];
  double cx = m.cen[2 * (size_t)i], cy = m.cen[2 * (size_t)i + 1];
  int a = k, b = (k + 1) % 3;
  double ax = X[2 * a] - cx, ay = X[2 * a + 1] - cy;
  double bx = X[2 * b] - cx, by = X[2 * b + 1] - cy;
  return (dx * by - dy * bx) >= 0.0 && (ax * dy - ay * dx) >= 0.0;
}

// Cells j != i passing the cone test of stencil k, by distance.
static void search(const Mesh& m, const Bins& b, int i, int k, int want, std::vector<Hit>& scratch) {
  double cx = m.cen[2 * (size_t)i], cy = m.cen[2 * (size_t)i + 1];
  auto consider = [&](int j) {
    if (j == i) return;
    double dx = m.cen[2 * (size_t)j] - cx, dy = m.cen[2 * (size_t)j + 1] - cy, kx, ky;
    wrap_delta(m, dx, dy, kx, ky);
    if (!cone_ok(m, i, k, dx, dy)) return;
    scratch.push_back({dx * dx + dy * dy, j});
  };
  scratch.clear();
  bool full = b.n < 7;
  if (!full) {
    const int bx0 = std::min(b.n - 1, std::max(0, (int)(bin_coord(m, 0, cx) / b.wx)));
    const int by0 = std::min(b.n - 1, std::max(0, (int)(bin_coord(m, 1, cy) / b.wy)));
    const double w = std::min(b.wx, b.wy);
    int rad = 1;
    for (;;) {
      // bin range per axis: a periodic axis wraps (whole axis once the block
      // would overlap itself), an open axis is clipped
      int lo[2], hi[2];
      bool whole[2];
      const int c0[2] = {bx0, by0};
      for (int a = 0; a < 2; ++a) {
        if (m.P[a] > 0.0) {
          whole[a] = 2 * rad + 1 > b.n;
          lo[a] = whole[a] ? 0 : c0[a] - rad;
          hi[a] = whole[a] ? b.n - 1 : c0[a] + rad;
        } else {
          lo[a] = std::max(0, c0[a] - rad);
          hi[a] = std::min(b.n - 1, c0[a] + rad);
          whole[a] = lo[a] == 0 && hi[a] == b.n - 1;
        }
      }
      if (whole[0] && whole[1]) {
        full = true;
        break;
      }
      scratch.clear();
      for (int oy = lo[1]; oy <= hi[1]; ++oy)
        for (int ox = lo[0]; ox <= hi[0]; ++ox) {
          int bx = (ox + b.n) % b.n, by = (oy + b.n) % b.n;
          int bin = by * b.n + bx;
          for (int t = b.start[bin]; t < b.start[bin + 1]; ++t) consider(b.cells[t]);
        }
      // every cell outside the (2 rad + 1)^2 block is at least rad*w away
      double reach = (rad - 0.01) * w;
      if ((int)scratch.size() >= want) {
        std::nth_element(scratch.begin(), scratch.begin() + (want - 1), scratch.end(), hit_less);
        if (scratch[want - 1].d2 < reach * reach) break;
      }
      rad *= 2;
    }
  }
  if (full) {
    scratch.clear();
    for (int j = 0; j < m.nc; ++j) consider(j);
  }
}

// Stencil k of cell i: the `want` nearest cells in the closed cone (k < 3)
// or overall (k = 3).  Near a boundary a cone may hold fewer cells; the
// stencil is then completed with the nearest cells outside the cone.
static bool find_stencil(const Mesh& m, const Bins& b, int i, int k, int want,
                         std::vector<Hit>& scratch, int32_t* out) {
  search(m, b, i, k, want, scratch);
  int have = std::min<int>(want, (int)scratch.size());
  std::partial_sort(scratch.begin(), scratch.begin() + have, scratch.end(), hit_less);
  for (int s = 0; s < have; ++s) out[s] = scratch[s].id;
  if (have == want) return true;
  if (k == 3 || !m.open()) return false;
  search(m, b, i, 3, want + have, scratch);
  std::sort(scratch.begin(), scratch.end(), hit_less);
  for (const Hit& h : scratch) {
    if (have == want) break;
    if (std::find(out, out + have, h.id) == out + have) out[have++] = h.id;
  }
  return have == want;
}

// ---------------------------------------------------------------------------
// least squares (Sec. 2.2): basis, exact moments, Householder pseudo-inverse
// ---------------------------------------------------------------------------
static double fact(int n) {
  double f = 1.0;
  for (int k = 2; k <= n; ++k) f *= k;
  return f;
}

struct Basis {
  int n = 0;
  int ea[21], eb[21];
  double mean[21];  // average of xi^a eta^b over the reference triangle
};

static Basis basis_of(int r) {
  Basis B;
  for (int deg = 1; deg <= r; ++deg)
    for (int a = deg; a >= 0; --a) {
      B.ea[B.n] = a;
      B.eb[B.n] = deg - a;
      B.mean[B.n] = 2.0 * fact(a) * fact(deg - a) / fact(deg + 2);
      B.n++;
    }
  return B;
}

// Radon's seven-point rule (degree 5) on a triangle, barycentric form.
template <class T>
struct RadonRule {
  T l[7][3], w[7];
  RadonRule() {
    const T s15 = std::sqrt((T)15);
    const T a1 = (6 - s15) / 21, a2 = (6 + s15) / 21;
    const T w1 = (155 - s15) / 1200, w2 = (155 + s15) / 1200;
    T pts[7][3] = {{(T)1 / 3, (T)1 / 3, (T)1 / 3},
                   {a1, a1, 1 - 2 * a1}, {a1, 1 - 2 * a1, a1}, {1 - 2 * a1, a1, a1},
                   {a2, a2, 1 - 2 * a2}, {a2, 1 - 2 * a2, a2}, {1 - 2 * a2, a2, a2}};
    T ww[7] = {(T)9 / 40, w1, w1, w1, w2, w2, w2};
    std::memcpy(l, pts, sizeof(l));
    std::memcpy(w, ww, sizeof(w));
  }
};
typedef RadonRule<double> Radon;

// Householder QR of the m x n row-major matrix A in place: R on and above the
// diagonal, vectors (v_j = 1) below, factors in beta.  Returns min|R_jj|/max|R_jj|
// (0 on breakdown: not above `tiny`).
template <class T>
T householder(int m, int n, std::vector<T>& A, std::vector<T>& beta, T tiny) {
  beta.resize(n);
  std::vector<T> w(n);
  for (int j = 0; j < n; ++j) {
    T nrm2 = 0.0;
    for (int i = j; i < m; ++i) nrm2 += A[(size_t)i * n + j] * A[(size_t)i * n + j];
    T nrm = std::sqrt(nrm2);
    if (nrm == 0.0) return 0;
    T x0 = A[(size_t)j * n + j];
    T alpha = x0 > 0.0 ? -nrm : nrm;
    // v = x - alpha e_1, scaled to v_j = 1
    T v0 = x0 - alpha;
    for (int i = j + 1; i < m; ++i) A[(size_t)i * n + j] /= v0;
    T vv = 1.0;
    for (int i = j + 1; i < m; ++i) vv += A[(size_t)i * n + j] * A[(size_t)i * n + j];
    beta[j] = 2.0 / vv;
    // the columns to the right, row by row (each column's sum in row order)
    for (int c = j + 1; c < n; ++c) w[c] = A[(size_t)j * n + c];
    for (int i = j + 1; i < m; ++i) {
      const T v = A[(size_t)i * n + j];
      for (int c = j + 1; c < n; ++c) w[c] += v * A[(size_t)i * n + c];
    }
    for (int c = j + 1; c < n; ++c) {
      w[c] *= beta[j];
      A[(size_t)j * n + c] -= w[c];
    }
    for (int i = j + 1; i < m; ++i) {
      const T v = A[(size_t)i * n + j];
      for (int c = j + 1; c < n; ++c) A[(size_t)i * n + c] -= w[c] * v;
    }
    A[(size_t)j * n + j] = alpha;
  }
  T rmax = 0, rmin = INFINITY;
  for (int j = 0; j < n; ++j) {
    T d = std::fabs(A[(size_t)j * n + j]);
    rmax = std::max(rmax, d);
    rmin = std::min(rmin, d);
  }
  if (!(rmin > tiny * rmax)) return 0;
  return rmin / rmax;
}

// Op[l][s] = (R^{-1} Q_1^T)[l][s] * scale[s] of A = Q_1 R (m x n, row-major; A is
// overwritten).  Returns householder's ratio.
template <class T>
T pinv_scaled(int m, int n, std::vector<T>& A, const T* scale, T* Op, T tiny) {
  std::vector<T> beta;
  const T rc = householder(m, n, A, beta, tiny);
  if (rc == 0) return 0;
  // Q_1 (m x n): apply H_{n-1} ... H_0 to the first n columns of I
  std::vector<T> Q((size_t)m * n, 0.0);
  for (int j = 0; j < n; ++j) Q[(size_t)j * n + j] = 1.0;
  for (int j = n - 1; j >= 0; --j)
    for (int c = 0; c < n; ++c) {
      T s = Q[(size_t)j * n + c];
      for (int i = j + 1; i < m; ++i) s += A[(size_t)i * n + j] * Q[(size_t)i * n + c];
      s *= beta[j];
      Q[(size_t)j * n + c] -= s;
      for (int i = j + 1; i < m; ++i) Q[(size_t)i * n + c] -= s * A[(size_t)i * n + j];
    }
  // Op[:, s] = R^{-1} Q_1[s, :]^T * scale[s]
  std::vector<T> x(n);
  for (int s = 0; s < m; ++s) {
    for (int l = n - 1; l >= 0; --l) {
      T acc = Q[(size_t)s * n + l];
      for (int c = l + 1; c < n; ++c) acc -= A[(size_t)l * n + c] * x[c];
      x[l] = acc / A[(size_t)l * n + l];
    }
    for (int l = 0; l < n; ++l) Op[(size_t)l * m + s] = x[l] * scale[s];
  }
  return rc;
}

double pinv_scaled(int m, int n, std::vector<double>& A, const double* scale, double* Op) {
  return pinv_scaled<double>(m, n, A, scale, Op, 1e-13);
}

// Rows of the constrained system of one stencil of (user) cell i.
static void lsq_rows(const Mesh& m, const Basis& B, const Radon& rule, int i, const int32_t* mem,
                     int nrow, std::vector<double>& A, std::vector<double>& vol) {
  const double* X0 = &m.X[6 * (size_t)i];
  const double j00 = X0[2] - X0[0], j01 = X0[4] - X0[0];
  const double j10 = X0[3] - X0[1], j11 = X0[5] - X0[1];
  const double det = j00 * j11 - j01 * j10;
  const double i00 = j11 / det, i01 = -j01 / det, i10 = -j10 / det, i11 = j00 / det;
  A.assign((size_t)nrow * B.n, 0.0);
  vol.assign(nrow, 0.0);
  for (int s = 0; s < nrow; ++s) {
    int j = mem[s];
    double dx = m.cen[2 * (size_t)j] - m.cen[2 * (size_t)i];
    double dy = m.cen[2 * (size_t)j + 1] - m.cen[2 * (size_t)i + 1], kx, ky;
    wrap_delta(m, dx, dy, kx, ky);
    const double sx = -m.P[0] * kx, sy = -m.P[1] * ky;
    const double* Xj = &m.X[6 * (size_t)j];
    double q[3][2];
    for (int v = 0; v < 3; ++v) {
      double px = Xj[2 * v] + sx - X0[0], py = Xj[2 * v + 1] + sy - X0[1];
      q[v][0] = i00 * px + i01 * py;
      q[v][1] = i10 * px + i11 * py;
    }
    // reference-space volume: |V_s| / |det J|
    vol[s] = m.area[j] / det;
    // (xi^a eta^b as xi ... xi eta ... eta, each from the one before)
    double acc[21] = {};
    for (int g = 0; g < 7; ++g) {
      const double xi = rule.l[g][0] * q[0][0] + rule.l[g][1] * q[1][0] + rule.l[g][2] * q[2][0];
      const double eta = rule.l[g][0] * q[0][1] + rule.l[g][1] * q[1][1] + rule.l[g][2] * q[2][1];
      double p[21];
      for (int l = 0; l < B.n; ++l) {
        const int deg = B.ea[l] + B.eb[l], first = deg * (deg - 1) / 2 - 1;  // of degree deg - 1
        p[l] = B.eb[l] == 0 ? (deg == 1 ? xi : p[first] * xi)
                            : (deg == 1 ? eta : p[first + B.eb[l] - 1] * eta);
        acc[l] += rule.w[g] * p[l];
      }
    }
    for (int l = 0; l < B.n; ++l) A[(size_t)s * B.n + l] = vol[s] * (acc[l] - B.mean[l]);
  }
}

void stencil_operator(const Mesh& m, int cell, int k, double* M) {
  const bool big = k == 3;
  const int nrow = big ? m.d.nl : kSmallRows, t = m.inv[cell];
  int32_t mem[64];
  for (int s = 0; s < nrow; ++s)
    mem[s] = m.perm[m.idx[packed_idx_index(m, t, big ? large_row(s) : small_row(k, s))]];
  std::vector<double> A, vol;
  lsq_rows(m, basis_of(big ? m.d.r : 2), Radon(), cell, mem, nrow, A, vol);
  pinv_scaled(nrow, big ? m.d.nu : kSmallCoef, A, vol.data(), M);
}

double Operators::operator[](int64_t at) const {
  const Dims& d = mesh->d;
  const int cell = mesh->perm[at / d.J], small = kSmallRows * kSmallCoef;
  int e = (int)(at % d.J);
  const int k = e < 3 * small ? e / small : 3, n = k == 3 ? d.nu : kSmallCoef, nrow = k == 3 ? d.nl : kSmallRows;
  e -= k * small;
  std::vector<double> M((size_t)n * nrow);
  stencil_operator(*mesh, cell, k, M.data());
  return M[(size_t)(e % n) * nrow + e / n];
}

// Morton code of a point in [0,1)^2 on a 2^16 grid.
static uint32_t spread16(uint32_t x) {
  x &= 0xFFFF;
  x = (x | (x << 8)) & 0x00FF00FF;
  x = (x | (x << 4)) & 0x0F0F0F0F;
  x = (x | (x << 2)) & 0x33333333;
  x = (x | (x << 1)) & 0x55555555;
  return x;
}

// ---------------------------------------------------------------------------
// matrix-free least squares: block member lists, geometry records and the
// inverses of the normal matrices
// ---------------------------------------------------------------------------
// The operators a = M d of the least squares are not stored (but for the cells
// named below): with rows A_s (moments of the member about the target, in any
// basis) and weights |V_s|, a = (sum_s |V_s|^2 A_s A_s^T)^-1 sum_s |V_s|^2 A_s
// d_s.  The normal matrix squares the condition of the rows, so the basis is
// chosen to be almost orthogonal over the stencil: the frame of a block
// whitens the displacements of its stencils (also on stretched and sheared
// meshes), the polynomials are Hermite's, and each stencil's are centred on
// its members' mean (one-sided small stencils, stencils at a wall).  The
// matrices are formed and inverted in extended precision and stored in FP64.
// On jittered meshes the face values of random data come out closer to 128
// bits than with the stored operators of the reference triangle's monomials
// (rms, orders 3-6: x 0.3-0.02), and the rounding noise of their sums is x
// 0.7-1.9 of a plain product M d (orders 3-6, boxes included; monomials about
// the target would give x 2-55).  On graded meshes a few stencils, one-sided
// ones above all, would lose digits that their operators keep (to 2.6e-7
// against 1e-10 on a sector of 4 rad with radii 1 : e^6): normal_bound finds
// those, and their cells keep their operators.
typedef long double Ext;

// E[H_a(x + X) H_b(y + Y)] for 0 <= a + b <= r from the central moments
// mu[a][b] = E[H_a(X) H_b(Y)] (the binomial shift of an Appell sequence)
// (by degree, unrolled: a column's moments stay in registers)
template <int n>
static inline __attribute__((always_inline)) void shift_line(Ext x, Ext (&v)[6]) {
#pragma GCC unroll 6
  for (int i = 1; i <= n; ++i)
#pragma GCC unroll 6
    for (int a = n; a >= i; --a) v[a] += x * v[a - 1];
}
template <int r, int b = 0>
static inline __attribute__((always_inline)) void shift_lines(Ext x, const Ext (&in)[6][6], Ext (&out)[6][6]) {
  Ext v[6];
#pragma GCC unroll 6
  for (int a = 0; a <= r - b; ++a) v[a] = in[a][b];
  shift_line<r - b>(x, v);
#pragma GCC unroll 6
  for (int a = 0; a <= r - b; ++a) out[b][a] = v[a];
  if constexpr (b < r) shift_lines<r, b + 1>(x, in, out);
}
template <int r>
static void shift_moments(Ext x, Ext y, const Ext (&mu)[6][6], Ext (&out)[6][6]) {
  Ext t[6][6];  // [b][a]
  shift_lines<r>(x, mu, t);
  shift_lines<r>(y, t, out);
}
static void shift_moments(int r, Ext x, Ext y, const Ext (&mu)[6][6], Ext (&out)[6][6]) {
  if (r == 2) shift_moments<2>(x, y, mu, out);
  if (r == 3) shift_moments<3>(x, y, mu, out);
  if (r == 4) shift_moments<4>(x, y, mu, out);
  if (r == 5) shift_moments<5>(x, y, mu, out);
}

// X = (A^T A)^-1 of the m x n row-major A: Cholesky, or the triangular factor
// of a Householder QR where the normal matrix breaks down.
static void normal_inverse(int m, int n, std::vector<Ext>& A, std::vector<Ext>& X) {
  std::vector<Ext> L((size_t)n * n, 0);
  bool ok = true;
  std::vector<Ext> G((size_t)n * n);  // upper triangle of A^T A, four sums at a time
  for (int j = 0; j < n; ++j) {
    int i = j;
    for (; i + 3 < n; i += 4) {
      Ext s0 = 0, s1 = 0, s2 = 0, s3 = 0;
      for (int k = 0; k < m; ++k) {
        const Ext* a = &A[(size_t)k * n];
        const Ext x = a[j];
        s0 += a[i] * x;
        s1 += a[i + 1] * x;
        s2 += a[i + 2] * x;
        s3 += a[i + 3] * x;
      }
      Ext* g = &G[(size_t)j * n + i];
      g[0] = s0;
      g[1] = s1;
      g[2] = s2;
      g[3] = s3;
    }
    for (; i < n; ++i) {
      Ext s = 0;
      for (int k = 0; k < m; ++k) s += A[(size_t)k * n + i] * A[(size_t)k * n + j];
      G[(size_t)j * n + i] = s;
    }
  }
  // Cholesky, four rows of a column at a time
  for (int j = 0; j < n && ok; ++j) {
    const Ext* lj = &L[(size_t)j * n];
    Ext s = G[(size_t)j * n + j];
    for (int k = 0; k < j; ++k) s -= lj[k] * lj[k];
    if (!(s > G[(size_t)j * n + j] * 1e-16L)) {
      ok = false;
      break;
    }
    const Ext piv = std::sqrt(s);
    L[(size_t)j * n + j] = piv;
    int i = j + 1;
    for (; i + 3 < n; i += 4) {
      const Ext *g = &G[(size_t)j * n + i], *l0 = &L[(size_t)i * n], *l1 = l0 + n, *l2 = l1 + n, *l3 = l2 + n;
      Ext s0 = g[0], s1 = g[1], s2 = g[2], s3 = g[3];
      for (int k = 0; k < j; ++k) {
        const Ext x = lj[k];
        s0 -= l0[k] * x;
        s1 -= l1[k] * x;
        s2 -= l2[k] * x;
        s3 -= l3[k] * x;
      }
      L[(size_t)i * n + j] = s0 / piv;
      L[(size_t)(i + 1) * n + j] = s1 / piv;
      L[(size_t)(i + 2) * n + j] = s2 / piv;
      L[(size_t)(i + 3) * n + j] = s3 / piv;
    }
    for (; i < n; ++i) {
      Ext t = G[(size_t)j * n + i];
      for (int k = 0; k < j; ++k) t -= L[(size_t)i * n + k] * lj[k];
      L[(size_t)i * n + j] = t / piv;
    }
  }
  if (!ok) {
    for (int j = 0; j < n; ++j) {
      Ext nrm = 0;
      for (int i = j; i < m; ++i) nrm += A[(size_t)i * n + j] * A[(size_t)i * n + j];
      nrm = std::sqrt(nrm);
      const Ext alpha = A[(size_t)j * n + j] > 0 ? -nrm : nrm;
      A[(size_t)j * n + j] -= alpha;
      Ext vv = 0;
      for (int i = j; i < m; ++i) vv += A[(size_t)i * n + j] * A[(size_t)i * n + j];
      for (int c = j + 1; c < n && vv > 0; ++c) {
        Ext s = 0;
        for (int i = j; i < m; ++i) s += A[(size_t)i * n + j] * A[(size_t)i * n + c];
        s *= 2 / vv;
        for (int i = j; i < m; ++i) A[(size_t)i * n + c] -= s * A[(size_t)i * n + j];
      }
      L[(size_t)j * n + j] = alpha;
      for (int c = j + 1; c < n; ++c) L[(size_t)c * n + j] = A[(size_t)j * n + c];  // L = R^T
    }
  }
  // L^-1 (lower triangular; four columns at a time, zeros above the diagonal),
  // then X = L^-T L^-1
  std::vector<Ext> Li((size_t)n * (n + 4), 0);
  const int w = n + 4;
  for (int i = 0; i < n; ++i) {
    const Ext* l = &L[(size_t)i * n];
    for (int c = 0; c <= i; c += 4) {
      Ext s0 = i == c, s1 = i == c + 1, s2 = i == c + 2, s3 = i == c + 3;
      for (int k = c; k < i; ++k) {
        const Ext x = l[k], *q = &Li[(size_t)k * w + c];
        s0 -= x * q[0];
        s1 -= x * q[1];
        s2 -= x * q[2];
        s3 -= x * q[3];
      }
      Ext* q = &Li[(size_t)i * w + c];
      q[0] = s0 / l[i];
      q[1] = s1 / l[i];
      q[2] = s2 / l[i];
      q[3] = s3 / l[i];
    }
  }
  X.assign((size_t)n * n, 0);
  for (int i = 0; i < n; ++i)
    for (int j = i; j < n; j += 4) {
      Ext s0 = 0, s1 = 0, s2 = 0, s3 = 0;
      for (int k = j; k < n; ++k) {
        const Ext x = Li[(size_t)k * w + i], *q = &Li[(size_t)k * w + j];
        s0 += x * q[0];
        s1 += x * q[1];
        s2 += x * q[2];
        s3 += x * q[3];
      }
      const Ext s[4] = {s0, s1, s2, s3};
      for (int q = 0; q < 4 && j + q < n; ++q) X[(size_t)i * n + j + q] = X[(size_t)(j + q) * n + i] = s[q];
    }
}

// Functions of the least-squares bases at nine points of a cell's edges (Gauss,
// three per edge): in X = 3 xi - 1, Y = 3 eta - 1 (v), and in xi, eta (w), less
// their means.
struct FacePoints {
  double v[9][20], w[9][20];
  FacePoints(const Basis& B, const RadonRule<Ext>& rule) {
    for (int l = 0; l < B.n; ++l) {
      auto f = [&](Ext x, Ext y) {
        Ext p = 1;
        for (int i = 0; i < B.ea[l]; ++i) p *= x;
        for (int i = 0; i < B.eb[l]; ++i) p *= y;
        return p;
      };
      Ext mean = 0;
      for (int g = 0; g < 7; ++g) mean += rule.w[g] * f(3 * rule.l[g][1] - 1, 3 * rule.l[g][2] - 1);
      for (int q = 0; q < 9; ++q) {
        const double t = 0.5 + (q % 3 - 1) * 0.5 * std::sqrt(0.6);
        const double xi = q < 3 ? t : (q < 6 ? 1.0 - t : 0.0), eta = q < 3 ? 0.0 : (q < 6 ? t : 1.0 - t);
        v[q][l] = (double)(f(3 * (Ext)xi - 1, 3 * (Ext)eta - 1) - mean);
        w[q][l] = (double)f(xi, eta) - B.mean[l];
      }
    }
  }
};

// What a normal matrix may cost.  Where the weights |V|^2 of a stencil's members
// span orders of magnitude (a one-sided stencil of a graded mesh, completed with
// far larger cells), or its members lie near a curve of the basis' degree, N has
// lost the digits that its operator still has: the sums of the large members'
// rows round at a size that the weak directions of N multiply.  A first-order
// bound of that, for differences of size one: the rounded row sums (magnitudes of
// the rows in `rows`) through |N|, the shift and expansion of the Hermite
// functions and the map to the reference triangle, all with absolute values, at
// the points of the cell's edges.  Rounding is random where the bound adds
// magnitudes: errors against 128 bits reach it at most (jittered, stretched and
// graded meshes, orders 3-6).
static double normal_bound(int r, int n, const std::vector<Ext>& N, const double* rows, double cx,
                           double cy, const double* J, const FacePoints& at) {
  // magnitudes of the coefficients of x^(n-2k) in H_n, [n][k]
  constexpr double h = kHermite;
  static const double expand[6][3] = {{1}, {1}, {1, h}, {1, 3 * h}, {1, 6 * h, 3 * h * h}, {1, 10 * h, 15 * h * h}};
  auto mono = [](int d, int k) { return d * (d + 1) / 2 - 1 + k; };
  double c[20], t[20];
  for (int i = 0; i < n; ++i) {
    c[i] = 0.0;
    for (int j = 0; j < n; ++j) c[i] += std::fabs((double)N[(size_t)i * n + j]) * rows[j];
  }
  cx = std::fabs(cx);
  cy = std::fabs(cy);
  for (int b = 0; b < r; ++b)
    for (int i = 0; i < r - b; ++i)
      for (int a = r - b - 1; a >= i; --a)
        if (a + b >= 1) c[mono(a + b, b)] += cx * c[mono(a + b + 1, b)];
  for (int a = 0; a < r; ++a)
    for (int i = 0; i < r - a; ++i)
      for (int b = r - a - 1; b >= i; --b)
        if (a + b >= 1) c[mono(a + b, b)] += cy * c[mono(a + b + 1, b + 1)];
  for (int axis = 0; axis < 2; ++axis)
    for (int o = 0; o < r; ++o)
      for (int e = 0; e <= r - o; ++e)  // e: the exponent that H_e expands
        for (int k = 1; o + e >= 1 && o + e + 2 * k <= r; ++k) {
          const int d = o + e + 2 * k;
          c[mono(o + e, axis ? e : o)] += expand[e + 2 * k][k] * c[mono(d, axis ? e + 2 * k : o)];
        }
  double sum[20];
  const double j0 = std::fabs(J[0]), j1 = std::fabs(J[1]), j2 = std::fabs(J[2]), j3 = std::fabs(J[3]);
  for (int d = 1; d <= r; ++d) {  // sum of c_k (j0 X + j1 Y)^(d-k) (j2 X + j3 Y)^k
    for (int q = 0; q <= d; ++q) t[q] = 0.0;
    for (int k = 0; k <= d; ++k) {
      double p[7] = {c[mono(d, k)]};
      for (int i = 0; i < d; ++i) {
        const double u = i < d - k ? j0 : j2, v = i < d - k ? j1 : j3;
        for (int q = i + 1; q >= 0; --q) p[q] = (q <= i ? u * p[q] : 0.0) + (q > 0 ? v * p[q - 1] : 0.0);
      }
      for (int q = 0; q <= d; ++q) t[q] += p[q];
    }
    for (int q = 0; q <= d; ++q) sum[mono(d, q)] = t[q];
  }
  double worst = 0.0;
  for (int q = 0; q < 9; ++q) {
    double x = 0.0;
    for (int l = 0; l < n; ++l) x += sum[l] * std::fabs(at.v[q][l]);
    worst = std::max(worst, x);
  }
  return worst * 1.1e-16;
}

// M of one stencil (Op[l][s], l < B.n) of user cell i in extended precision, in
// the basis X = 3 xi - 1, Y = 3 eta - 1 less its means; false on breakdown.
// Solved in monomials of coordinates that give the members' centroids mean zero
// and unit variance, then expanded.
static bool extended_operator(const Mesh& m, const Basis& B, const RadonRule<Ext>& rule, int i,
                              const int32_t* mem, int nrow, std::vector<Ext>& Op) {
  const int n = B.n;
  const double* X0 = &m.X[6 * (size_t)i];
  const Ext j00 = (Ext)X0[2] - X0[0], j01 = (Ext)X0[4] - X0[0];
  const Ext j10 = (Ext)X0[3] - X0[1], j11 = (Ext)X0[5] - X0[1];
  const Ext det = j00 * j11 - j01 * j10;
  std::vector<Ext> q((size_t)nrow * 6), A((size_t)nrow * n), vol(nrow);  // q: vertices (X, Y)
  Ext mx = 0, my = 0, sxx = 0, sxy = 0, syy = 0;
  auto centroid = [&](int s, int a) { return (q[6 * s + a] + q[6 * s + 2 + a] + q[6 * s + 4 + a]) / 3; };
  for (int s = 0; s < nrow; ++s) {
    const int j = mem[s];
    double dx = m.cen[2 * (size_t)j] - m.cen[2 * (size_t)i];
    double dy = m.cen[2 * (size_t)j + 1] - m.cen[2 * (size_t)i + 1], kx, ky;
    wrap_delta(m, dx, dy, kx, ky);
    const double* Xj = &m.X[6 * (size_t)j];
    for (int v = 0; v < 3; ++v) {
      const Ext px = (Ext)Xj[2 * v] - (Ext)m.P[0] * kx - X0[0];
      const Ext py = (Ext)Xj[2 * v + 1] - (Ext)m.P[1] * ky - X0[1];
      q[6 * s + 2 * v] = 3 * (j11 * px - j01 * py) / det - 1;
      q[6 * s + 2 * v + 1] = 3 * (j00 * py - j10 * px) / det - 1;
    }
    const Ext* t = &q[6 * s];
    vol[s] = ((t[2] - t[0]) * (t[5] - t[1]) - (t[4] - t[0]) * (t[3] - t[1])) / 18;
    mx += centroid(s, 0) / nrow;
    my += centroid(s, 1) / nrow;
  }
  for (int s = 0; s < nrow; ++s) {
    const Ext x = centroid(s, 0) - mx, y = centroid(s, 1) - my;
    sxx += x * x / nrow;
    sxy += x * y / nrow;
    syy += y * y / nrow;
  }
  // x = ax (X - mx), y = bx (X - mx) + by (Y - my)
  const Ext l11 = std::sqrt(sxx), l21 = sxy / l11;
  Ext l22 = syy - l21 * l21;
  l22 = l22 > 1e-24L * syy ? std::sqrt(l22) : std::sqrt(syy);
  const Ext ax = 1 / l11, bx = -l21 / (l11 * l22), by = 1 / l22;
  auto averages = [&](const Ext* t, Ext* out) {
    for (int l = 0; l < n; ++l) out[l] = 0;
    for (int g = 0; g < 7; ++g) {
      Ext X = -mx, Y = -my, px[6], py[6];
      for (int v = 0; v < 3; ++v) {
        X += rule.l[g][v] * t[2 * v];
        Y += rule.l[g][v] * t[2 * v + 1];
      }
      px[0] = py[0] = 1;
      for (int e = 1; e < 6; ++e) {
        px[e] = px[e - 1] * (ax * X);
        py[e] = py[e - 1] * (bx * X + by * Y);
      }
      for (int l = 0; l < n; ++l) out[l] += rule.w[g] * px[B.ea[l]] * py[B.eb[l]];
    }
  };
  const Ext ref[6] = {-1, -1, 2, -1, -1, 2};
  Ext mean[20], av[20];
  averages(ref, mean);
  for (int s = 0; s < nrow; ++s) {
    averages(&q[6 * s], av);
    for (int l = 0; l < n; ++l) A[(size_t)s * n + l] = vol[s] * (av[l] - mean[l]);
  }
  std::vector<Ext> c((size_t)n * nrow, 0);
  if (!(pinv_scaled<Ext>(nrow, n, A, vol.data(), c.data(), 0.0L) > 0)) return false;
  // each function's polynomial in X, Y: p[a][b] of X^a Y^b
  Op.assign((size_t)n * nrow, 0);
  for (int l = 0; l < n; ++l) {
    Ext p[6][6] = {{1}};
    const int deg = B.ea[l] + B.eb[l];
    for (int e = 0; e < deg; ++e) {
      const Ext u = e < B.ea[l] ? ax : bx, v = e < B.ea[l] ? 0 : by, w = -u * mx - v * my;
      for (int a = e + 1; a >= 0; --a)
        for (int b = e + 1 - a; b >= 0; --b)
          p[a][b] = w * p[a][b] + (a > 0 ? u * p[a - 1][b] : 0) + (b > 0 ? v * p[a][b - 1] : 0);
    }
    for (int k = 0; k < n; ++k)
      if (B.ea[k] + B.eb[k] <= deg)
        for (int s = 0; s < nrow; ++s) Op[(size_t)k * nrow + s] += p[B.ea[k]][B.eb[k]] * c[(size_t)l * nrow + s];
  }
  return true;
}

// ... and what the stored operator costs that is formed in FP64 in the reference
// triangle's monomials (lsq_rows, pinv_scaled), for the same differences: its error
// against `op` and the rounding of its sums.
static double operator_error(const Mesh& m, const Basis& B, const Radon& rule, int i, const int32_t* mem,
                             int nrow, const std::vector<Ext>& op, const FacePoints& at) {
  const int n = B.n;
  std::vector<double> A, vol, dbl((size_t)n * nrow);
  lsq_rows(m, B, rule, i, mem, nrow, A, vol);
  if (pinv_scaled(nrow, n, A, vol.data(), dbl.data()) == 0.0) return 0.0;
  double worst = 0.0;
  for (int q = 0; q < 9; ++q) {
    double t = 0.0;
    for (int s = 0; s < nrow; ++s) {
      Ext x = 0, e = 0;
      for (int l = 0; l < n; ++l) {
        x += op[(size_t)l * nrow + s] * at.v[q][l];
        e += (Ext)dbl[(size_t)l * nrow + s] * at.w[q][l];
      }
      t += std::fabs((double)(e - x)) + 1.1e-16 * std::fabs((double)x);
    }
    worst = std::max(worst, t);
  }
  return worst;
}

// A cell is solved with operators where the bound of a stencil is above both a
// floor (values of size one) and a multiple of that.  Errors are 0.1-0.2 of the
// bound where it is large (small stencils; 0.05-0.1 the large one) and 0.2-0.7 of
// operator_error: these ratios are where the two meet.
constexpr double kBoundFloor = 2e-13;
constexpr double bound_ratio(bool big) { return big ? 30.0 : 10.0; }

// A stencil member as a block sees it: the cell and its periodic image.
struct Image {
  int32_t id;
  int kx, ky;
  bool operator<(const Image& o) const {
    return id != o.id ? id < o.id : (kx != o.kx ? kx < o.kx : ky < o.ky);
  }
  bool operator==(const Image& o) const { return id == o.id && kx == o.kx && ky == o.ky; }
};

// Images and the slots they were first given, open addressing.
struct ImageSlots {
  std::vector<std::pair<Image, int>> at;
  size_t used = 0;
  explicit ImageSlots(size_t n) : at(n, {Image{-1, 0, 0}, 0}) {}
  size_t place(const Image& im) const {
    uint64_t h = (uint64_t)(uint32_t)im.id << 16 ^ (uint64_t)(uint32_t)(im.kx * 256 + im.ky);
    size_t k = (h * 0x9E3779B97F4A7C15ull >> 20) & (at.size() - 1);
    while (at[k].first.id >= 0 && !(at[k].first == im)) k = (k + 1) & (at.size() - 1);
    return k;
  }
  bool add(const Image& im, int slot) {  // false: was there
    if (2 * used >= at.size()) {
      ImageSlots twice(2 * at.size());
      for (auto& e : at)
        if (e.first.id >= 0) twice.add(e.first, e.second);
      *this = std::move(twice);
    }
    auto& e = at[place(im)];
    if (e.first.id >= 0) return false;
    e = {im, slot};
    ++used;
    return true;
  }
  int slot(const Image& im) const { return at[place(im)].second; }
};

// Packed order of positions [lo, hi): bisection along the longer side of the
// box of the centroids (wrapped on periodic axes), at multiples of `unit` cells
// down to one block, then of a tile.
static void pack_bisect(Mesh& m, int lo, int hi, int unit, int threads) {
  if (hi - lo <= unit) {
    if (unit > kTile) pack_bisect(m, lo, hi, kTile, 1);
    return;
  }
  auto at = [&](int i, int a) { return bin_coord(m, a, m.cen[2 * (size_t)m.perm[i] + a]); };
  double mn[2] = {INFINITY, INFINITY}, mx[2] = {-INFINITY, -INFINITY};
  for (int k = lo; k < hi; ++k)
    for (int a = 0; a < 2; ++a) {
      const double x = at(m.pack[k], a);
      mn[a] = std::min(mn[a], x);
      mx[a] = std::max(mx[a], x);
    }
  const int a = mx[1] - mn[1] > mx[0] - mn[0] ? 1 : 0;
  const int nb = (hi - lo + unit - 1) / unit, mid = lo + (nb / 2) * unit;
  std::nth_element(m.pack.begin() + lo, m.pack.begin() + mid, m.pack.begin() + hi, [&](int x, int y) {
    const double dx = at(x, a), dy = at(y, a);
    return dx < dy || (dx == dy && x < y);
  });
  if (threads > 1 && hi - lo > 4096) {
    std::thread left([&]() { pack_bisect(m, lo, mid, unit, threads / 2); });
    pack_bisect(m, mid, hi, unit, threads - threads / 2);
    left.join();
  } else {
    pack_bisect(m, lo, mid, unit, 1);
    pack_bisect(m, mid, hi, unit, 1);
  }
}

// False: no layout fits.  (Cells that are compact in no sense, which the limit on
// 16 consecutive ones has let through, may scatter more when bisected: then tiles
// are the runs of the internal order that the limit speaks of.)
static bool pack_blocks(Mesh& m, int most_tiles, bool bisect) {
  const Dims& d = m.d;
  const int nc = m.nc, r = d.r, nu = d.nu, units = rec_units(nu);
  // images relative to the origin cell o (both internal): K of cell j
  auto image_of = [&](int j, int o, int& kx, int& ky) {
    const int uj = m.perm[j], uo = m.perm[o];
    double dx = m.cen[2 * (size_t)uj] - m.cen[2 * (size_t)uo];
    double dy = m.cen[2 * (size_t)uj + 1] - m.cen[2 * (size_t)uo + 1], fx, fy;
    wrap_delta(m, dx, dy, fx, fy);
    kx = (int)fx;
    ky = (int)fy;
  };
  m.pack.assign(m.n_pad, -1);
  std::vector<std::vector<Image>> lists;
  int n_blocks = 0;
  // as many tiles per block as the LDS allows
  for (m.bwaves = most_tiles, m.nbuf = 2;;) {
    const int W = m.bwaves, cells = W * kTile;
    n_blocks = (m.n_tiles + W - 1) / W;
    for (int t = 0; t < nc; ++t) m.pack[t] = t;
    if (bisect) pack_bisect(m, 0, nc, cells,
                m.prm.n_threads > 0 ? m.prm.n_threads : (int)std::max(1u, std::thread::hardware_concurrency()));
    for (int t = 0; t < nc; t += kTile)
      std::sort(m.pack.begin() + t, m.pack.begin() + std::min(nc, t + kTile));
    lists.assign(n_blocks, {});
    std::atomic<int> top{0}, top_tile{0};
    parallel_for(n_blocks, m.prm.n_threads, [&](int b) {
      std::vector<Image>& u = lists[b];
      const int t0 = b * cells, t1 = std::min(nc, t0 + cells), origin = m.pack[t0];
      std::vector<Image> own(cells);
      for (int c = 0; c < cells; ++c) {
        Image& im = own[c];
        im.id = m.pack[std::min(t0 + c, nc - 1)];
        image_of(im.id, origin, im.kx, im.ky);
      }
      // the block's own cells, then the other members by id
      ImageSlots seen(2048), tile(512);
      u = own;
      for (const Image& im : own) seen.add(im, 0);
      int most = 0;
      for (int t = t0; t < t1; ++t) {
        if (t % kTile == 0) tile = ImageSlots(512);
        for (int row = 0; row < d.rows; ++row) {
          Image im;
          im.id = m.idx[packed_idx_index(m, m.pack[t], row)];
          image_of(im.id, m.pack[t], im.kx, im.ky);
          im.kx += own[t - t0].kx;
          im.ky += own[t - t0].ky;
          if (seen.add(im, 0)) u.push_back(im);
          tile.add({im.id, 0, 0}, 0);
        }
        most = std::max(most, (int)tile.used);
      }
      for (int cur = top_tile.load(); most > cur && !top_tile.compare_exchange_weak(cur, most);) {
      }
      std::sort(u.begin() + cells, u.end());
      int cur = top.load();
      while ((int)u.size() > cur && !top.compare_exchange_weak(cur, (int)u.size())) {
      }
    }, 1);
    m.bmax = top.load();
    const bool ch = m.prm.characteristic != 0;
    const int lds = group_lds_bytes(buffer_stride(nu, m.bmax, W, ch), m.bmax, m.nbuf);
    if (layout_fits(nu, W, m.bmax, m.nbuf, (top_tile.load() + 15) / 16 * 16, ch) &&
        (lds <= (m.nbuf == 2 ? lds_budget(W) : kLdsPerCu / 2) || (W == 1 && m.nbuf == 1)))
      break;
    if (W == 1 && m.nbuf == 1) {
      if (!bisect) return false;
      bisect = false;
      continue;
    }
    // two buffers do not fit: one, in workgroups of four or fewer
    if (m.nbuf == 2 && W == 4) {
      m.nbuf = 1;
    } else {
      m.nbuf = 1;
      m.bwaves = std::max(1, W / 2);
    }
  }
  m.boff.assign(n_blocks + 1, 0);
  for (int b = 0; b < n_blocks; ++b) m.boff[b + 1] = m.boff[b] + (int32_t)lists[b].size();
  m.bmem.assign((size_t)n_blocks * m.bmax, 0);
  m.brec.resize((size_t)m.boff[n_blocks] * units * 2);
  const int nw = slot_words(d.nl), nq4 = normal_quads(nu);
  m.bslot.assign((size_t)m.n_tiles * nw * 64, 0);
  m.N.resize((size_t)m.n_tiles * nq4 * 128);
  m.jac.resize((size_t)m.n_pad * 4);
  m.centre.assign((size_t)m.n_pad * 8, 0.0f);
  // exact for every moment needed (degree 5)
  const RadonRule<Ext> rule;
  const Radon rule64;
  const Basis Bs = basis_of(2), Bl = basis_of(r);
  const FacePoints at_small(Bs, rule), at_large(Bl, rule);
  std::vector<uint8_t> keep(m.n_pad, 0);  // solved with operators, by packed position
  auto users = [&](int cell, int k, int32_t* mem) {  // members of stencil k, user ids
    const int nrow = k == 3 ? d.nl : kSmallRows;
    for (int s = 0; s < nrow; ++s)
      mem[s] = m.perm[m.idx[packed_idx_index(m, cell, k == 3 ? large_row(s) : small_row(k, s))]];
  };
  parallel_for(n_blocks, m.prm.n_threads, [&](int b) {
    const std::vector<Image>& u = lists[b];
    const int cells = m.bwaves * kTile;
    const int t0 = b * cells, t1 = std::min(nc, t0 + cells);
    // ---- frame: whitens the displacements of the large stencils ----
    double cxx = 0, cxy = 0, cyy = 0;
    for (int t = t0; t < t1; ++t)
      for (int s = 0; s < d.nl; ++s) {
        const int ui = m.perm[m.pack[t]];
        const int uj = m.perm[m.idx[packed_idx_index(m, m.pack[t], large_row(s))]];
        double dx = m.cen[2 * (size_t)uj] - m.cen[2 * (size_t)ui];
        double dy = m.cen[2 * (size_t)uj + 1] - m.cen[2 * (size_t)ui + 1], kx, ky;
        wrap_delta(m, dx, dy, kx, ky);
        cxx += dx * dx;
        cxy += dx * dy;
        cyy += dy * dy;
      }
    const double n0 = (double)(t1 - t0) * d.nl;
    const double l11 = std::sqrt(cxx / n0), l21 = cxy / n0 / l11;
    double l22 = std::sqrt(std::max(0.0, cyy / n0 - l21 * l21));
    if (!(l22 > 1e-12 * l11)) l22 = l11;
    const Ext f00 = 1 / (Ext)l11, f10 = -(Ext)l21 / ((Ext)l11 * l22), f11 = 1 / (Ext)l22;
    // ---- records ----
    const double* Xo = &m.X[6 * (size_t)m.perm[m.pack[t0]]];
    const Ext o[2] = {((Ext)Xo[0] + Xo[2] + Xo[4]) / 3, ((Ext)Xo[1] + Xo[3] + Xo[5]) / 3};
    std::vector<double> rec(u.size() * (nu + 1));
    for (size_t k = 0; k < u.size(); ++k) {
      const double* Xj = &m.X[6 * (size_t)m.perm[u[k].id]];
      Ext q[3][2], c[2] = {0, 0};
      for (int v = 0; v < 3; ++v) {
        const Ext px = (Ext)Xj[2 * v] - (Ext)m.P[0] * u[k].kx - o[0];
        const Ext py = (Ext)Xj[2 * v + 1] - (Ext)m.P[1] * u[k].ky - o[1];
        q[v][0] = f00 * px;
        q[v][1] = f10 * px + f11 * py;
        c[0] += q[v][0] / 3;
        c[1] += q[v][1] / 3;
      }
      for (int v = 0; v < 3; ++v)
        for (int a = 0; a < 2; ++a) q[v][a] -= c[a];
      const Ext vol = ((q[1][0] - q[0][0]) * (q[2][1] - q[0][1]) -
                       (q[2][0] - q[0][0]) * (q[1][1] - q[0][1])) / 2;
      double* R = &rec[k * (nu + 1)];
      R[0] = (double)c[0];
      R[1] = (double)c[1];
      R[2] = (double)(vol * vol);
      Ext hx[7][6], hy[7][6];
      for (int g = 0; g < 7; ++g) {
        Ext x = 0, y = 0;
        for (int v = 0; v < 3; ++v) {
          x += rule.l[g][v] * q[v][0];
          y += rule.l[g][v] * q[v][1];
        }
        hx[g][0] = hy[g][0] = 1;
        hx[g][1] = x;
        hy[g][1] = y;
        for (int n = 2; n <= r; ++n) {
          hx[g][n] = x * hx[g][n - 1] - (Ext)kHermite * (n - 1) * hx[g][n - 2];
          hy[g][n] = y * hy[g][n - 1] - (Ext)kHermite * (n - 1) * hy[g][n - 2];
        }
      }
      int l = 3;
      for (int deg = 2; deg <= r; ++deg)
        for (int e = deg; e >= 0; --e, ++l) {
          Ext s = 0;
          for (int g = 0; g < 7; ++g) s += rule.w[g] * hx[g][e] * hy[g][deg - e];
          R[l] = (double)s;
        }
      m.bmem[(size_t)b * m.bmax + k] = u[k].id;
      double* out = &m.brec[((size_t)m.boff[b] + k) * units * 2];
      for (int x = 0; x < units * 2; ++x) out[x] = x < nu + 1 ? R[x] : 0.0;
    }
    // ---- slots and normal inverses ----
    auto moments = [&](int k, Ext (&mu)[6][6]) {
      const double* R = &rec[(size_t)k * (nu + 1)];
      mu[0][0] = 1;
      mu[1][0] = mu[0][1] = 0;
      int l = 3;
      for (int deg = 2; deg <= r; ++deg)
        for (int e = deg; e >= 0; --e, ++l) mu[e][deg - e] = R[l];
    };
    std::vector<Ext> A, X, op;
    int32_t mem[64];
    ImageSlots at_slot(2048);
    for (size_t k = 0; k < u.size(); ++k) at_slot.add(u[k], (int)k);
    for (int c = 0; c < cells; ++c) {
      const int t = t0 + c, tile = t / kTile, tc = t % kTile;
      if (tile >= m.n_tiles) break;
      const bool live = t < nc;
      uint32_t* sl = &m.bslot[(size_t)tile * nw * 64];
      auto put = [&](int lane, int grp, int slot) {
        uint32_t& w = sl[(size_t)(grp / 3) * 64 + lane];
        const int sh = kSlotBits * (grp % 3);
        w = (w & ~(((1u << kSlotBits) - 1) << sh)) | (uint32_t)slot << sh;
      };
      for (int g = 0; g < 4; ++g)
        for (int grp = 0; grp < nw * 3; ++grp) put(tc * 4 + g, grp, c);
      double* Nt = &m.N[(size_t)tile * nq4 * 128];
      for (int q = 0; q < nq4; ++q)
        for (int x = 0; x < 8; ++x) Nt[(size_t)q * 128 + tc * 8 + x] = 0.0;
      double* J = &m.jac[(size_t)t * 4];
      J[0] = J[3] = 1.0;
      J[1] = J[2] = 0.0;
      if (!live) continue;
      {
        const double* Xi = &m.X[6 * (size_t)m.perm[m.pack[t]]];
        for (int v = 0; v < 2; ++v) {
          const Ext ex = ((Ext)Xi[2 * v + 2] - Xi[0]) / 3, ey = ((Ext)Xi[2 * v + 3] - Xi[1]) / 3;
          J[v] = (double)(f00 * ex);
          J[2 + v] = (double)(f10 * ex + f11 * ey);
        }
      }
      Ext mu0[6][6], own[6][6];
      moments(c, mu0);
      const double* R0 = &rec[(size_t)c * (nu + 1)];
      int grp0 = 0, quad0 = 0;
      std::vector<int> slots(d.nl);
      for (int k = 0; k < 4; ++k) {
        const bool big = k == 3;
        const int nrow = big ? d.nl : kSmallRows, n = big ? nu : kSmallCoef, rk = big ? r : 2;
        A.assign((size_t)nrow * n, 0);
        Ext cx = 0, cy = 0;
        slots.resize(std::max(nrow, d.nl));
        for (int s = 0; s < nrow; ++s) {
          Image im;
          im.id = m.idx[packed_idx_index(m, m.pack[t], big ? large_row(s) : small_row(k, s))];
          image_of(im.id, m.pack[t], im.kx, im.ky);
          im.kx += u[c].kx;
          im.ky += u[c].ky;
          const int slot = at_slot.slot(im);
          put(tc * 4 + s % 4, grp0 + s / 4, slot);
          slots[s] = slot;
          const double* R = &rec[(size_t)slot * (nu + 1)];
          cx += ((Ext)R[0] - R0[0]) / nrow;
          cy += ((Ext)R[1] - R0[1]) / nrow;
        }
        // the centre; a large stencil's that is nearly the target's centroid
        // is taken there (the kernel then skips the shift back)
        if (big && cx * cx + cy * cy < 0.04L) cx = cy = 0;
        const float fx = (float)cx, fy = (float)cy;
        m.centre[((size_t)t * 4 + k) * 2] = fx;
        m.centre[((size_t)t * 4 + k) * 2 + 1] = fy;
        shift_moments(rk, -(Ext)fx, -(Ext)fy, mu0, own);
        double size[20] = {};
        for (int s = 0; s < nrow; ++s) {
          Ext mu[6][6], sh[6][6];
          moments(slots[s], mu);
          const double* R = &rec[(size_t)slots[s] * (nu + 1)];
          shift_moments(rk, (Ext)R[0] - R0[0] - fx, (Ext)R[1] - R0[1] - fy, mu, sh);
          const Ext w = std::sqrt((Ext)R[2]);
          int l = 0;
          for (int deg = 1; deg <= rk; ++deg)
            for (int e = deg; e >= 0; --e, ++l) {
              A[(size_t)s * n + l] = w * (sh[e][deg - e] - own[e][deg - e]);
              size[l] += R[2] * (std::fabs((double)sh[e][deg - e]) + std::fabs((double)own[e][deg - e]));
            }
        }
        normal_inverse(nrow, n, A, X);
        const Basis& B = big ? Bl : Bs;
        const double bound = normal_bound(rk, n, X, size, fx, fy, J, big ? at_large : at_small);
        if (!(bound <= kBoundFloor) && !keep[t]) {
          const int user = m.perm[m.pack[t]];
          users(m.pack[t], k, mem);
          if (extended_operator(m, B, rule, user, mem, nrow, op) &&
              !(bound <= bound_ratio(big) * operator_error(m, B, rule64, user, mem, nrow, op,
                                                      big ? at_large : at_small)))
            keep[t] = 1;
        }
        int j = 0;
        for (int i = 0; i < n; ++i)
          for (int q = i; q < n; ++q, ++j)
            Nt[(size_t)(quad0 + j / 8) * 128 + tc * 8 + j % 8] = (double)X[(size_t)i * n + q];
        grp0 += row_groups(nrow);
        quad0 += sym_quads(n);
      }
    }
  }, 1);
  // ---- cells solved with operators ----
  std::vector<int32_t> at;  // packed position of each
  for (int t = 0; t < nc; ++t)
    if (keep[t]) at.push_back(t);
  const int n_kept = (int)(at.size() + kKeptCells - 1) / kKeptCells;
  const int groups = kept_groups(d.nl), chunks = kept_chunks(d.nl, nu);
  m.kept.assign((size_t)n_kept * kKeptCells, -1);
  m.kept_rows.assign((size_t)n_kept * groups * 64, 0);
  m.kept_ops.assign((size_t)n_kept * chunks * 64, 0.0);
  parallel_for((int)at.size(), m.prm.n_threads, [&](int i) {
    const int cell = m.pack[at[i]], set = i / kKeptCells, lane = i % kKeptCells * 16;
    int32_t* rows = &m.kept_rows[(size_t)set * groups * 64 + lane];
    double* out = &m.kept_ops[(size_t)set * chunks * 64 + lane];
    std::vector<Ext> op[4];
    int32_t mem[64];
    for (int k = 0; k < 4; ++k) {
      users(cell, k, mem);
      if (!extended_operator(m, k == 3 ? Bl : Bs, rule, m.perm[cell], mem, k == 3 ? d.nl : kSmallRows, op[k])) {
        keep[at[i]] = 0;  // (set-up has refused meshes where this could be)
        return;
      }
    }
    m.kept[i] = cell;
    int grp = 0, chunk = 0;
    for (int k = 0; k < 4; ++k) {
      const int nrow = k == 3 ? d.nl : kSmallRows, n = k == 3 ? nu : kSmallCoef;
      for (int s = 0; s < kept_row_groups(nrow) * 16; ++s) {
        rows[(size_t)(grp + s / 16) * 64 + s % 16] =
            s < nrow ? m.idx[packed_idx_index(m, cell, k == 3 ? large_row(s) : small_row(k, s))] : cell;
        for (int l = 0; l < n && s < nrow; ++l)
          out[((size_t)chunk + (s / 16) * n + l) * 64 + s % 16] = (double)op[k][(size_t)l * nrow + s];
      }
      grp += kept_row_groups(nrow);
      chunk += kept_row_groups(nrow) * n;
    }
  }, 1);
  for (int t : at)
    if (keep[t]) m.pack[t] = -1;
  return true;
}

int mesh_setup(Mesh& m, const teno_params& p) {
  if (p.order < 3 || p.order > 6) return fail(TENO_EARG, "order must be 3..6");
  if (p.variant < 0 || p.variant > 2) return fail(TENO_EARG, "variant must be 0, 1 or 2");
  if (p.variant == 2 && !(p.dk_prime > 1.0)) return fail(TENO_EARG, "CWENO needs dk_prime > 1");
  if (p.characteristic != 0 && p.characteristic != 1)
    return fail(TENO_EARG, "characteristic must be 0 or 1");
  if (!(p.ct >= 0.0 && p.ct <= 1.0 / 3.0)) return fail(TENO_EARG, "C_T must lie in [0, 1/3]");
  if (p.power < 1 || p.power > 16) return fail(TENO_EARG, "power must be 1..16");
  if (p.n_quad != 0 && (p.n_quad < 2 || p.n_quad > 3)) return fail(TENO_EARG, "n_quad must be 0, 2 or 3");
  m.prm = p;
  m.d = dims_for(p.order, p.n_quad);
  const Dims& d = m.d;
  const int nc = m.nc;
  // stencil rows are addressed as cell * 4 ceil(rows / 4) + row in 32 bits
  if ((int64_t)(nc + kTile) * d.rows4 * 4 >= (int64_t)INT32_MAX)
    return fail(TENO_EARG, "mesh too large: " + std::to_string(nc) + " cells at order " +
                               std::to_string(p.order) + " exceed 32-bit stencil-row indices");

  // ---- cell order ----
  m.perm.resize(nc);
  for (int i = 0; i < nc; ++i) m.perm[i] = i;
  if (p.reorder) {
    std::vector<uint32_t> code(nc);
    for (int i = 0; i < nc; ++i) {
      double x = bin_coord(m, 0, m.cen[2 * (size_t)i]) / (m.hi[0] - m.lo[0]);
      double y = bin_coord(m, 1, m.cen[2 * (size_t)i + 1]) / (m.hi[1] - m.lo[1]);
      x = std::min(std::max(x, 0.0), 1.0);
      y = std::min(std::max(y, 0.0), 1.0);
      uint32_t qx = std::min<uint32_t>(65535u, (uint32_t)(x * 65536.0));
      uint32_t qy = std::min<uint32_t>(65535u, (uint32_t)(y * 65536.0));
      code[i] = spread16(qx) | (spread16(qy) << 1);
    }
    std::sort(m.perm.begin(), m.perm.end(), [&](int a, int b) {
      return code[a] < code[b] || (code[a] == code[b] && a < b);
    });
  }
  m.inv.assign(nc, 0);
  for (int t = 0; t < nc; ++t) m.inv[m.perm[t]] = t;

  m.n_tiles = (nc + kTile - 1) / kTile;
  m.n_pad = m.n_tiles * kTile;
  try {
    m.idx.assign((size_t)m.n_tiles * d.rows4 * kTile * 4, 0);
  } catch (...) {
    return fail(TENO_ENOMEM, "host allocation of the stencils failed");
  }

  Bins bins;
  bins_build(m, bins);
  const Basis Bs = basis_of(2), Bl = basis_of(d.r);
  const Radon rule;
  std::mutex mu;
  int err_code = TENO_OK, err_cell = nc;
  std::string err_msg;
  double rc_min = 1.0;
  parallel_for(nc, p.n_threads, [&](int i) {
    std::vector<Hit> scratch;
    std::vector<double> A, vol, beta;
    int32_t mem[64];
    const int t = m.inv[i];
    double rc_local = 1.0;
    for (int k = 0; k < 4; ++k) {
      const bool big = (k == 3);
      const Basis& B = big ? Bl : Bs;
      const int nrow = big ? d.nl : kSmallRows;
      auto report = [&](int code, const std::string& msg) {
        std::lock_guard<std::mutex> g(mu);
        if (i < err_cell) {
          err_cell = i;
          err_code = code;
          err_msg = msg;
        }
      };
      if (!find_stencil(m, bins, i, k, nrow, scratch, mem)) {
        report(TENO_ESTENCIL, "too few stencil candidates at cell " + std::to_string(i));
        return;
      }
      for (int s = 0; s < nrow; ++s) {
        double dx = m.cen[2 * (size_t)mem[s]] - m.cen[2 * (size_t)i];
        double dy = m.cen[2 * (size_t)mem[s] + 1] - m.cen[2 * (size_t)i + 1], kx, ky;
        wrap_delta(m, dx, dy, kx, ky);
        if ((m.P[0] > 0.0 && std::fabs(dx) > 0.4 * m.P[0]) ||
            (m.P[1] > 0.0 && std::fabs(dy) > 0.4 * m.P[1])) {
          report(TENO_ESTENCIL, "mesh too small for the stencil at cell " + std::to_string(i));
          return;
        }
      }
      lsq_rows(m, B, rule, i, mem, nrow, A, vol);
      const double rc = householder(nrow, B.n, A, beta, 1e-13);
      if (rc == 0.0) {
        report(TENO_ERANK, "rank-deficient least-squares matrix at cell " + std::to_string(i));
        return;
      }
      rc_local = std::min(rc_local, rc);
      for (int s = 0; s < nrow; ++s)
        m.idx[packed_idx_index(m, t, big ? large_row(s) : small_row(k, s))] = m.inv[mem[s]];
    }
    std::lock_guard<std::mutex> g(mu);
    rc_min = std::min(rc_min, rc_local);
  });
  if (err_code != TENO_OK) return fail(err_code, err_msg);
  m.min_rcond = rc_min;

  // ---- per-cell face data (internal order) ----
  m.nbinfo.assign((size_t)m.n_pad * 4, 0);
  m.geo.assign((size_t)m.n_pad * 10, 0.0);
  m.user_of.assign(m.n_pad, 0);
  for (int t = 0; t < m.n_pad; ++t) {
    if (t >= nc) {
      m.geo[(size_t)t * 10 + 9] = 1.0;  // padding cells: unit area, no neighbours
      continue;
    }
    int i = m.perm[t];
    m.user_of[t] = i;
    int32_t bits = 0;
    for (int e = 0; e < 3; ++e) {
      int f = m.cface[3 * (size_t)i + e];
      bool isL = (m.fL[f] == i && m.fLe[f] == e);
      int other = isL ? m.fR[f] : m.fL[f];
      int oe = isL ? m.fRe[f] : m.fLe[f];
      if (other < 0) {  // boundary face: the cell itself, as its L side
        other = i;
        oe = 0;
      }
      m.nbinfo[(size_t)t * 4 + e] = m.inv[other];
      bits |= (oe & 3) << (2 * e);
      if (isL) bits |= 1 << (6 + e);
      m.geo[(size_t)t * 10 + 3 * e + 0] = m.fnx[f];
      m.geo[(size_t)t * 10 + 3 * e + 1] = m.fny[f];
      m.geo[(size_t)t * 10 + 3 * e + 2] = m.flen[f];
    }
    m.nbinfo[(size_t)t * 4 + 3] = bits;
    m.geo[(size_t)t * 10 + 9] = m.area[i];
  }

  // ---- face-ordered data for the flux kernels ----
  {
    std::vector<int32_t> order(m.nf), rank(m.nf);
    for (int f = 0; f < m.nf; ++f) order[f] = f;
    std::sort(order.begin(), order.end(), [&](int a, int b) {
      const int la = m.inv[m.fL[a]], lb = m.inv[m.fL[b]];
      return la < lb || (la == lb && m.fLe[a] < m.fLe[b]);
    });
    m.face_cells.assign((size_t)m.nf * 4, 0);
    m.face_geo.assign((size_t)m.nf * 4, 0.0);
    std::vector<int32_t> bidx(m.nf, -1);
    for (size_t b = 0; b < m.bface.size(); ++b) bidx[m.bface[b]] = (int32_t)b;
    for (int k = 0; k < m.nf; ++k) {
      const int f = order[k];
      rank[f] = k;
      // a boundary face names its own cell on both sides (the kernel loads
      // unconditionally and replaces the outer state) and its index in .w
      const bool bnd = m.fR[f] < 0;
      m.face_cells[(size_t)k * 4 + 0] = m.inv[m.fL[f]];
      m.face_cells[(size_t)k * 4 + 1] = m.inv[bnd ? m.fL[f] : m.fR[f]];
      m.face_cells[(size_t)k * 4 + 2] = (m.fLe[f] & 3) | (((bnd ? m.fLe[f] : m.fRe[f]) & 3) << 2);
      m.face_cells[(size_t)k * 4 + 3] = bnd ? bidx[f] : -1;
      m.face_geo[(size_t)k * 4 + 0] = m.fnx[f];
      m.face_geo[(size_t)k * 4 + 1] = m.fny[f];
      m.face_geo[(size_t)k * 4 + 2] = m.flen[f];
    }
    m.bface_sorted.resize(m.bface.size());
    for (size_t b = 0; b < m.bface.size(); ++b) m.bface_sorted[b] = rank[m.bface[b]];
    m.cell_faces.assign((size_t)m.n_pad * 4, 0);
    m.vol.assign(m.n_pad, 1.0);
    for (int t = 0; t < nc; ++t) {
      const int i = m.perm[t];
      int32_t bits = 0;
      for (int e = 0; e < 3; ++e) {
        const int f = m.cface[3 * (size_t)i + e];
        m.cell_faces[(size_t)t * 4 + e] = rank[f];
        if (m.fL[f] == i && m.fLe[f] == e) bits |= 1 << e;
      }
      m.cell_faces[(size_t)t * 4 + 3] = bits;
      m.vol[t] = m.area[i];
    }
  }

  // ---- distinct stencil members of 16 consecutive cells: a shuffled order is
  //      refused ----
  {
    std::atomic<int> top{1};
    parallel_for(m.n_tiles, p.n_threads, [&](int tile) {
      ImageSlots u(1024);
      for (int t = tile * kTile; t < std::min(nc, (tile + 1) * kTile); ++t)
        for (int r = 0; r < d.rows; ++r) u.add({m.idx[packed_idx_index(m, t, r)], 0, 0}, 0);
      const int n = (int)u.used;
      int cur = top.load();
      while (n > cur && !top.compare_exchange_weak(cur, n)) {
      }
    });
    if (top.load() > kMaxTileMembers)
      return fail(TENO_ESTENCIL, "a 16-cell tile has " + std::to_string(top.load()) +
                                     " distinct stencil members (limit " +
                                     std::to_string(kMaxTileMembers) +
                                     "); keep the default cell reordering");
  }
  if (!pack_blocks(m, block_tiles(d.order), true))
    return fail(TENO_ESTENCIL, "a tile's distinct stencil members do not fit the device's local memory");

  // ---- distinct members of each (packed) tile, the adjoint's accumulators ----
  {
    std::vector<std::vector<int32_t>> lists(m.n_tiles);
    std::atomic<int> umax{1};
    const int nw = adj_words(d.nl);
    m.aslot.assign((size_t)m.n_tiles * nw * 64, 0);
    parallel_for(m.n_tiles, p.n_threads, [&](int tile) {
      std::vector<int32_t>& u = lists[tile];
      for (int t = tile * kTile; t < (tile + 1) * kTile; ++t)
        for (int r = 0; r < d.rows && m.pack[t] >= 0; ++r)
          u.push_back(m.idx[packed_idx_index(m, m.pack[t], r)]);
      std::sort(u.begin(), u.end());
      u.erase(std::unique(u.begin(), u.end()), u.end());
      int cur = umax.load();
      while ((int)u.size() > cur && !umax.compare_exchange_weak(cur, (int)u.size())) {
      }
      // each row's slot in the tile's list and the round of the adjoint's
      // addition: the rows 4j..4j+3 of a stencil are added by all cells at
      // once (lane order c * 4 + g), and the lanes of such a group that name
      // the same member add in lane order, one round each, so that no two
      // lanes of one LDS instruction hit the same address
      uint32_t* as = &m.aslot[(size_t)tile * nw * 64];
      std::vector<uint16_t> seen(u.size());
      int grp = 0;
      for (int k = 0; k < 4; ++k) {
        const int r0 = k == 3 ? large_row(0) : small_row(k, 0), nrow = k == 3 ? d.nl : kSmallRows;
        for (int j = 0; j < row_groups(nrow); ++j, ++grp) {
          std::fill(seen.begin(), seen.end(), 0);
          for (int lane = 0; lane < 64; ++lane) {
            const int t = tile * kTile + lane / 4, row = 4 * j + lane % 4;
            if (m.pack[t] < 0 || row >= nrow) continue;
            const int id = m.idx[packed_idx_index(m, m.pack[t], r0 + row)];
            const int s = (int)(std::lower_bound(u.begin(), u.end(), id) - u.begin());
            as[(size_t)(grp / 2) * 64 + lane] |= (uint32_t)((s & 511) | seen[s]++ << 9) << (16 * (grp % 2));
          }
        }
      }
    });
    m.ustride = (umax.load() + 15) / 16 * 16;
    m.tmem.assign((size_t)m.n_tiles * m.ustride, 0);
    m.tcount.assign(m.n_tiles, 0);
    for (int tile = 0; tile < m.n_tiles; ++tile) {
      const auto& u = lists[tile];
      m.tcount[tile] = (int32_t)u.size();
      for (int k = 0; k < m.ustride; ++k)
        m.tmem[(size_t)tile * m.ustride + k] = u.empty() ? 0 : u[std::min<size_t>(k, u.size() - 1)];
    }
  }

  // ---- reverse member lists for the adjoint gather: the (tile, slot)
  //      entries naming each cell, by tile ----
  m.rev_ptr.assign(nc + 1, 0);
  for (int tile = 0; tile < m.n_tiles; ++tile)
    for (int k = 0; k < m.tcount[tile]; ++k) m.rev_ptr[m.tmem[(size_t)tile * m.ustride + k] + 1]++;
  // a kept cell's rows, one entry each
  auto kept_row = [&](size_t e) {  // whether entry e of kept_rows is a row
    const int lane = e % 64, grp = (int)(e / 64 % kept_groups(d.nl));
    const int gs = kept_row_groups(kSmallRows), j = grp < 3 * gs ? grp % gs : grp - 3 * gs;
    return m.kept[e / 64 / kept_groups(d.nl) * kKeptCells + lane / 16] >= 0 &&
           16 * j + lane % 16 < (grp < 3 * gs ? kSmallRows : d.nl);
  };
  for (size_t e = 0; e < m.kept_rows.size(); ++e)
    if (kept_row(e)) m.rev_ptr[m.kept_rows[e] + 1]++;
  if ((int64_t)m.n_tiles * m.ustride + (int64_t)m.kept_rows.size() > INT32_MAX)
    return fail(TENO_EARG, "mesh too large: adjoint entries exceed 32-bit indices");
  for (int t = 0; t < nc; ++t) m.rev_ptr[t + 1] += m.rev_ptr[t];
  m.rev_ent.assign(std::max<int32_t>(1, m.rev_ptr[nc]), 0);
  {
    std::vector<int32_t> fill(m.rev_ptr.begin(), m.rev_ptr.end() - 1);
    for (int tile = 0; tile < m.n_tiles; ++tile)
      for (int k = 0; k < m.tcount[tile]; ++k) {
        const int j = m.tmem[(size_t)tile * m.ustride + k];
        m.rev_ent[fill[j]++] = tile * m.ustride + k;
      }
    for (size_t e = 0; e < m.kept_rows.size(); ++e)
      if (kept_row(e)) m.rev_ent[fill[m.kept_rows[e]]++] = m.n_tiles * m.ustride + (int32_t)e;
  }
  m.M.mesh = &m;
  m.ready = true;
  return TENO_OK;
}

}  // namespace teno
