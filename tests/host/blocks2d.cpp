// Test driver (CPU only) of the triangle kernels' block data: the LDS layout of
// the staged blocks and what set-up packs for them.  Includes csrc/setup.cpp, whose
// internals it calls; run by tests/test_blocks_host.py:
//   blocks2d layout                                every layout, ranges disjoint
//   blocks2d mesh <dir> <tag> order variant char   one mesh's blocks
//   blocks2d solve <dir> <tag> order every [runs]  the least squares of the block
//       data in the kernels' arithmetic, against a 128-bit solution (runs: packed
//       again in tiles that are runs of the internal order)
//   blocks2d faces <dir> <tag> order every         face states of the linear scheme
//       in 128 bits at every so-manieth cell: <tag>.u holds the states, user order;
//       writes <tag>.cells and <tag>.faces [cell][point][4]
// where <dir>/<tag>.txt holds "n_vert n_cell px py" and <tag>.xy, <tag>.tri the
// arrays.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <random>
#include <string>
#include <vector>

#include "../../paper_2105_02127_amd/csrc/setup.cpp"
#include "../../paper_2105_02127_amd/csrc/tables.h"

using namespace teno;

static void die(const std::string& what) {
  std::fprintf(stderr, "FAILED: %s\n", what.c_str());
  std::exit(3);
}

// ---- LDS layout -------------------------------------------------------------
// What a workgroup writes while it computes block k of a mesh: the staged block
// k + 1 and its ids, the Gram matrices of block k over its members, the ids of
// block k + 2 (over those of block k, which are read).  No range may meet
// another that is live, and all lie inside the allocation.
struct Range {
  int lo, hi;
  const char* what;
};

static void check_layout(int order, int waves, int members, int buffers, bool characteristic) {
  const Dims d = dims_for(order, 0);
  const int stride = buffer_stride(d.nu, members, waves, characteristic);
  const int total = group_lds_bytes(stride, members, buffers);
  char at[160];
  std::snprintf(at, sizeof(at), "order %d, %d waves, %d members, %d buffers, characteristic %d", order,
                waves, members, buffers, (int)characteristic);
  for (int k = 0; k < 2; ++k) {
    const int cur = buffer_offset(stride, buffers, k), next = buffer_offset(stride, buffers, k + 1);
    const int staged = block_lds_bytes(d.nu, members);
    std::vector<Range> live;
    live.push_back({cur, cur + (characteristic ? gram_bytes(waves) : staged), "the current block"});
    if (buffers == 2) live.push_back({next, next + staged, "the next block"});
    for (int b = 0; b < buffers; ++b) {
      const int o = ids_offset(stride, members, buffers, b);
      live.push_back({o, o + 4 * members, "a list of ids"});
    }
    live.push_back({cur, cur + 0, ""});
    for (size_t i = 0; i < live.size(); ++i) {
      if (live[i].lo < 0 || live[i].hi > total || live[i].lo % 16)
        die(std::string(live[i].what) + " leaves the allocation at " + at);
      for (size_t j = 0; j < i; ++j)
        if (live[i].lo < live[j].hi && live[j].lo < live[i].hi && live[i].hi > live[i].lo)
          die(std::string(live[i].what) + " overlaps " + live[j].what + " at " + at);
    }
    if (cur + staged > total || staged > stride) die(std::string("a staged block at ") + at);
  }
}

static int all_layouts() {
  int n = 0;
  // what does not fit is told apart: slots past their ten bits, the adjoint's
  // accumulators, two buffers, a single one
  for (int order = 3; order <= 6; ++order) {
    const int nu = dims_for(order, 0).nu;
    const int one = kLdsPerCu / (block_lds_bytes(nu, 1) + 4) - 64;  // members that surely fit
    if (!layout_fits(nu, 1, one < 1024 ? one : 1024, 1, 384, true)) die("a layout that fits was refused");
    if (layout_fits(nu, 1, 1025, 1, 16, false) || layout_fits(nu, 1, 16, 1, 528, false) ||
        layout_fits(nu, 1, kLdsPerCu / block_lds_bytes(nu, 1) + 1, 1, 16, false) ||
        layout_fits(nu, 8, one / 2 + 128, 2, 16, false) || layout_fits(nu, 8, one / 2, 1, 512, false))
      die("a layout that does not fit was accepted");
  }
  // a batch charges a mesh for the tiles it has
  for (int order = 3; order <= 6; ++order)
    for (int tiles = 1; tiles <= 20; ++tiles) {
      double sum = 0.0;
      for (int b = 0; b * block_tiles(order) < tiles; ++b) sum += block_cost(order, block_tiles(order), tiles, b);
      if (sum != tiles * block_cost(order, 1, 1, 0)) die("the cost of a part of a block");
    }
  for (int order = 3; order <= 6; ++order)
    for (int waves = 1; waves <= block_tiles(order); waves *= 2)
      for (int members = waves * kTile; members <= 1 << kSlotBits; ++members)
        for (int buffers = 1; buffers <= 2; ++buffers)
          for (int ch = 0; ch < 2; ++ch, ++n) check_layout(order, waves, members, buffers, ch != 0);
  return n;
}

// ---- meshes -----------------------------------------------------------------
template <class T>
static std::vector<T> slurp(const std::string& path, size_t n) {
  std::vector<T> v(n);
  std::ifstream f(path, std::ios::binary);
  f.read(reinterpret_cast<char*>(v.data()), (std::streamsize)(n * sizeof(T)));
  if (!f) die("cannot read " + path);
  return v;
}

static void load_mesh(const std::string& base, Mesh& m) {
  int nv = 0, nc = 0;
  double per[2] = {0, 0};
  std::ifstream(base + ".txt") >> nv >> nc >> per[0] >> per[1];
  const auto xy = slurp<double>(base + ".xy", 2 * (size_t)nv);
  const auto tri = slurp<int32_t>(base + ".tri", 3 * (size_t)nc);
  if (mesh_create(nv, xy.data(), nc, tri.data(), per, m)) die(last_error());
}

static void set_up(Mesh& m, int order, int variant, int characteristic) {
  teno_params p{};
  p.order = order;
  p.variant = variant;
  p.characteristic = characteristic;
  p.power = 6;
  p.ct = 1e-6;
  p.eps = 1e-12;
  p.gamma = 1.4;
  p.reorder = 1;
  p.dk_prime = 1e4;
  if (mesh_setup(m, p)) die(last_error());
}

// ---- least squares ------------------------------------------------------------
// The kernels' arithmetic on the host, stencil by stencil (kernels.hpp:
// stencil_sums, NormalMatrix::apply, hermite_to_monomials, Frame::to_basis,
// operator_sums), for differences drawn from [-1, 1], against Householder QR in
// 128 bits on the reference triangle in the basis X = 3 xi - 1, Y = 3 eta - 1.
typedef __float128 Quad;

static int mono(int d, int k) { return d * (d + 1) / 2 - 1 + k; }

static void shift(int r, double x, double y, const double* mu, double* out) {
  double t[6][6];
  for (int b = 0; b <= r; ++b) {
    double v[6];
    for (int a = 0; a <= r - b; ++a) v[a] = a + b >= 2 ? mu[mono(a + b, b) - 2] : (a + b == 0 ? 1 : 0);
    for (int i = 1; i <= r - b; ++i)
      for (int a = r - b; a >= i; --a) v[a] = std::fma(x, v[a - 1], v[a]);
    for (int a = 0; a <= r - b; ++a) t[a][b] = v[a];
  }
  for (int a = 0; a <= r; ++a) {
    double v[6];
    for (int b = 0; b <= r - a; ++b) v[b] = t[a][b];
    for (int i = 1; i <= r - a; ++i)
      for (int b = r - a; b >= i; --b) v[b] = std::fma(y, v[b - 1], v[b]);
    for (int b = 0; b <= r - a; ++b)
      if (a + b >= 1) out[mono(a + b, b)] = v[b];
  }
}

static void to_reference(int r, double* c, double cx, double cy, const double* J) {
  const double h = kHermite;
  const double expand[6][3] = {{1}, {1}, {1, -h}, {1, -3 * h}, {1, -6 * h, 3 * h * h}, {1, -10 * h, 15 * h * h}};
  for (int b = 0; b < r; ++b)
    for (int i = 0; i < r - b; ++i)
      for (int a = r - b - 1; a >= i; --a)
        if (a + b >= 1) c[mono(a + b, b)] = std::fma(-cx, c[mono(a + b + 1, b)], c[mono(a + b, b)]);
  for (int a = 0; a < r; ++a)
    for (int i = 0; i < r - a; ++i)
      for (int b = r - a - 1; b >= i; --b)
        if (a + b >= 1) c[mono(a + b, b)] = std::fma(-cy, c[mono(a + b + 1, b + 1)], c[mono(a + b, b)]);
  for (int axis = 0; axis < 2; ++axis)
    for (int o = 0; o < r; ++o)
      for (int e = 0; e <= r - o; ++e)
        for (int k = 1; o + e >= 1 && o + e + 2 * k <= r; ++k)
          c[mono(o + e, axis ? e : o)] = std::fma(expand[e + 2 * k][k], c[mono(o + e + 2 * k, axis ? e + 2 * k : o)],
                                                  c[mono(o + e, axis ? e : o)]);
  for (int d = 1; d <= r; ++d) {
    double t[7] = {};
    for (int k = 0; k <= d; ++k) {
      double p[7] = {c[mono(d, k)]};
      for (int i = 0; i < d; ++i)
        for (int q = i + 1; q >= 0; --q) {
          const double u = J[i < d - k ? 0 : 2], v = J[i < d - k ? 1 : 3];
          p[q] = std::fma(u, q <= i ? p[q] : 0.0, q > 0 ? v * p[q - 1] : 0.0);
        }
      for (int q = 0; q <= d; ++q) t[q] += p[q];
    }
    for (int q = 0; q <= d; ++q) c[mono(d, q)] = t[q];
  }
}

static Quad quad_sqrt(Quad x) {
  Quad y = std::sqrt((long double)x);
  for (int i = 0; i < 2 && y > 0; ++i) y = (y + x / y) / 2;
  return y;
}

struct Exact {
  Quad l[7][3], w[7];
  Exact() {  // Radon's rule of degree 5
    const Quad s = quad_sqrt(15), a[2] = {(6 - s) / 21, (6 + s) / 21};
    w[0] = (Quad)9 / 40;
    for (int v = 0; v < 3; ++v) l[0][v] = (Quad)1 / 3;
    for (int h = 0; h < 2; ++h)
      for (int k = 0; k < 3; ++k) {
        for (int v = 0; v < 3; ++v) l[1 + 3 * h + k][v] = v == k ? 1 - 2 * a[h] : a[h];
        w[1 + 3 * h + k] = (h ? 155 + s : 155 - s) / 1200;
      }
  }
  static void powers(int r, Quad x, Quad y, Quad* out) {
    for (int d = 1; d <= r; ++d)
      for (int k = 0; k <= d; ++k) {
        Quad p = 1;
        for (int i = 0; i < d - k; ++i) p *= x;
        for (int i = 0; i < k; ++i) p *= y;
        out[mono(d, k)] = p;
      }
  }
  void averages(int r, int n, const Quad (&q)[3][2], Quad* out) const {
    for (int i = 0; i < n; ++i) out[i] = 0;
    for (int g = 0; g < 7; ++g) {
      Quad x = -1, y = -1, p[20];
      for (int v = 0; v < 3; ++v) {
        x += 3 * l[g][v] * q[v][0];
        y += 3 * l[g][v] * q[v][1];
      }
      powers(r, x, y, p);
      for (int i = 0; i < n; ++i) out[i] += w[g] * p[i];
    }
  }
  // coefficients for the differences d, and the operator op[s][n]
  void solve(const Mesh& m, int cell, int r, int n, int nrow, const int* members, const double* d,
             Quad* c, Quad* mean, std::vector<Quad>& op) const {
    const double* X0 = &m.X[6 * (size_t)cell];
    const Quad j00 = (Quad)X0[2] - X0[0], j01 = (Quad)X0[4] - X0[0];
    const Quad j10 = (Quad)X0[3] - X0[1], j11 = (Quad)X0[5] - X0[1], det = j00 * j11 - j01 * j10;
    const Quad ref[3][2] = {{0, 0}, {1, 0}, {0, 1}};
    averages(r, n, ref, mean);
    const int w = n + nrow + 1;  // A, identity (scaled), right-hand side
    std::vector<Quad> A((size_t)nrow * w, 0);
    for (int s = 0; s < nrow; ++s) {
      const int j = members[s];
      Quad q[3][2], av[20];
      double k[2];
      for (int a = 0; a < 2; ++a)
        k[a] = m.P[a] > 0 ? std::nearbyint((m.cen[2 * (size_t)j + a] - m.cen[2 * (size_t)cell + a]) / m.P[a]) : 0;
      for (int v = 0; v < 3; ++v) {
        const Quad px = (Quad)m.X[6 * (size_t)j + 2 * v] - (Quad)m.P[0] * k[0] - X0[0];
        const Quad py = (Quad)m.X[6 * (size_t)j + 2 * v + 1] - (Quad)m.P[1] * k[1] - X0[1];
        q[v][0] = (j11 * px - j01 * py) / det;
        q[v][1] = (j00 * py - j10 * px) / det;
      }
      const Quad vol = ((q[1][0] - q[0][0]) * (q[2][1] - q[0][1]) - (q[2][0] - q[0][0]) * (q[1][1] - q[0][1])) / 2;
      averages(r, n, q, av);
      for (int i = 0; i < n; ++i) A[(size_t)s * w + i] = vol * (av[i] - mean[i]);
      A[(size_t)s * w + n + s] = vol;
      A[(size_t)s * w + n + nrow] = vol * (Quad)d[s];
    }
    for (int j = 0; j < n; ++j) {
      Quad s = 0, vv = 0;
      for (int i = j; i < nrow; ++i) s += A[(size_t)i * w + j] * A[(size_t)i * w + j];
      s = quad_sqrt(s);
      const Quad alpha = A[(size_t)j * w + j] > 0 ? -s : s;
      A[(size_t)j * w + j] -= alpha;
      for (int i = j; i < nrow; ++i) vv += A[(size_t)i * w + j] * A[(size_t)i * w + j];
      for (int k = j + 1; k < w; ++k) {
        Quad t = 0;
        for (int i = j; i < nrow; ++i) t += A[(size_t)i * w + j] * A[(size_t)i * w + k];
        t *= 2 / vv;
        for (int i = j; i < nrow; ++i) A[(size_t)i * w + k] -= t * A[(size_t)i * w + j];
      }
      A[(size_t)j * w + j] = alpha;
    }
    op.resize((size_t)nrow * n);
    for (int k = 0; k <= nrow; ++k)
      for (int i = n - 1; i >= 0; --i) {
        Quad t = A[(size_t)i * w + n + k];
        for (int j = i + 1; j < n; ++j) t -= A[(size_t)i * w + j] * c[j];
        c[i] = t / A[(size_t)i * w + i];
        if (k < nrow) op[(size_t)k * n + i] = c[i];
      }
  }
};

// Face-value error that the mesh's FP64 operator (in the monomials of xi, eta) may
// make for differences of up to one: its own error and the rounding of its sums.
static double operator_worst(const Mesh& m, int cell, int k, int r, int n, int nrow,
                             const std::vector<Quad>& op, const Quad* mean) {
  double worst = 0.0;
  std::vector<double> M((size_t)n * nrow);
  stencil_operator(m, m.perm[cell], k, M.data());
  for (int e = 0; e < 3; ++e)
    for (int q = 0; q < 3; ++q) {
      const Quad p = (Quad)0.5 + (q - 1) * (Quad)0.3872983346207417;
      const Quad xi = e == 0 ? p : (e == 1 ? 1 - p : 0), eta = e == 0 ? 0 : (e == 1 ? p : 1 - p);
      Quad x[20], y[20];
      Exact::powers(r, 3 * xi - 1, 3 * eta - 1, x);
      Exact::powers(r, xi, eta, y);
      double t = 0.0;
      for (int s = 0; s < nrow; ++s) {
        Quad a = 0, b = 0;
        for (int d = 1, l = 0; d <= r; ++d)
          for (int j = 0; j <= d; ++j, ++l) {
            double f = 2.0;  // mean of xi^(d-j) eta^j
            for (int i = 1; i <= j; ++i) f *= i;
            for (int i = d - j + 1; i <= d + 2; ++i) f /= i;
            a += op[(size_t)s * n + l] * (x[l] - mean[l]);
            b += (Quad)M[(size_t)l * nrow + s] * (y[l] - (Quad)f);
          }
        t += std::fabs((double)(b - a)) + 1.1e-16 * std::fabs((double)a);
      }
      worst = std::max(worst, t);
    }
  return worst;
}

// prints, for the small and the large stencils, their number, how many are of cells
// solved with operators, the worst face value, the worst that the FP64 operators may
// make, and the largest ratio of a stencil's error to 2e-13 + 2 times that
static void solve_all(const Mesh& m, int every) {
  const Exact ex;
  const Dims& d = m.d;
  const int units2 = 2 * rec_units(d.nu), cells = m.bwaves * kTile, nw = slot_words(d.nl);
  std::mt19937 gen(1);
  std::uniform_real_distribution<double> uni(-1, 1);
  int n_all[2] = {0, 0}, n_kept[2] = {0, 0};
  double worst[2] = {0, 0}, stored[2] = {0, 0}, ratio[2] = {0, 0};
  // every packed position, then the cells solved with operators (pack -1)
  const int n_pos = m.n_pad + (int)m.kept.size();
  for (int t = 0; t < n_pos; t += every) {
    const bool kept = t >= m.n_pad;
    const int cell = kept ? m.kept[t - m.n_pad] : m.pack[t];
    if (cell < 0) continue;
    const int tile = t / kTile, tc = t % kTile, blk = kept ? 0 : t / cells;
    const int set = (t - m.n_pad) / kKeptCells, lane0 = (t - m.n_pad) % kKeptCells * 16;
    const double* rec = &m.brec[(size_t)m.boff[blk] * units2];
    const double* R0 = kept ? rec : rec + (size_t)(t - blk * cells) * units2;
    const double* ops = kept ? &m.kept_ops[(size_t)set * kept_chunks(d.nl, d.nu) * 64 + lane0] : nullptr;
    int grp0 = 0, quad0 = 0, kgrp = 0;
    for (int k = 0; k < 4; ++k) {
      const bool big = k == 3;
      const int nrow = big ? d.nl : kSmallRows, n = big ? d.nu : kSmallCoef, r = big ? d.r : 2;
      double diff[64], c[20] = {}, h[20], mo[20], r0 = 0.0;
      int members[64];
      const double cx = kept ? 0 : m.centre[((size_t)t * 4 + k) * 2], cy = kept ? 0 : m.centre[((size_t)t * 4 + k) * 2 + 1];
      std::vector<double> rhs(n, 0.0);
      for (int s = 0; s < nrow; ++s) {
        diff[s] = uni(gen);
        const int idx = m.idx[packed_idx_index(m, cell, big ? large_row(s) : small_row(k, s))];
        members[s] = m.perm[idx];
        const int grp = grp0 + s / 4, lane = tc * 4 + s % 4;
        if (kept) {
          if (m.kept_rows[((size_t)set * kept_groups(d.nl) + kgrp + s / 16) * 64 + lane0 + s % 16] != idx)
            die("a kept row names another cell");
          for (int i = 0; i < n; ++i) c[i] = std::fma(ops[((s / 16) * n + i) * 64 + s % 16], diff[s], c[i]);
          continue;
        }
        const int slot = m.bslot[((size_t)tile * nw + grp / 3) * 64 + lane] >> (kSlotBits * (grp % 3)) &
                         ((1 << kSlotBits) - 1);
        if (m.bmem[(size_t)blk * m.bmax + slot] != idx) die("a row slot names another cell");
        const double* R = rec + (size_t)slot * units2;
        shift(r, R[0] - (R0[0] + cx), R[1] - (R0[1] + cy), R + 3, mo);
        const double x = diff[s] * R[2];
        r0 += x;
        for (int i = 0; i < n; ++i) rhs[i] = std::fma(mo[i], x, rhs[i]);
      }
      if (!kept) {
        shift(r, -cx, -cy, R0 + 3, h);
        for (int i = 0; i < n; ++i) rhs[i] = std::fma(-h[i], r0, rhs[i]);
        for (int i = 0, e = 0; i < n; ++i)
          for (int j = i; j < n; ++j, ++e) {
            const double x = m.N[((size_t)tile * normal_quads(d.nu) + quad0 + e / 8) * 128 + tc * 8 + e % 8];
            c[i] = std::fma(x, rhs[j], c[i]);
            if (i != j) c[j] = std::fma(x, rhs[i], c[j]);
          }
        to_reference(r, c, cx, cy, &m.jac[(size_t)t * 4]);
      }
      Quad want[20], mean[20];
      double err = 0.0;
      std::vector<Quad> op;
      ex.solve(m, m.perm[cell], r, n, nrow, members, diff, want, mean, op);
      for (int e = 0; e < 3; ++e)
        for (int q = 0; q < 3; ++q) {
          const Quad p = (Quad)0.5 + (q - 1) * (Quad)0.3872983346207417;
          Quad x[20], s = 0;
          Exact::powers(r, 3 * (e == 0 ? p : (e == 1 ? 1 - p : 0)) - 1, 3 * (e == 0 ? 0 : (e == 1 ? p : 1 - p)) - 1, x);
          for (int i = 0; i < n; ++i) s += (c[i] - want[i]) * (x[i] - mean[i]);
          err = std::max(err, std::fabs((double)s));
        }
      ++n_all[big];
      n_kept[big] += kept;
      if (kept) ops += (size_t)kept_row_groups(nrow) * n * 64;
      kgrp += kept_row_groups(nrow);
      worst[big] = std::max(worst[big], err);
      const double es = operator_worst(m, cell, k, r, n, nrow, op, mean);
      stored[big] = std::max(stored[big], es);
      ratio[big] = std::max(ratio[big], err / (2e-13 + 2 * es));
      grp0 += row_groups(nrow);
      quad0 += sym_quads(n);
    }
  }
  for (int b = 0; b < 2; ++b)
    std::printf("%s stencils %d kept %d worst %.2e operators %.2e ratio %.2e\n", b ? "large" : "small", n_all[b],
                n_kept[b], worst[b], stored[b], ratio[b]);
}

template <int P>
static void linear_faces(const Mesh& m, const std::string& base, int every) {
  using O = OrderT<P>;
  const Exact ex;
  const auto U = slurp<double>(base + ".u", 4 * (size_t)m.nc);
  std::vector<int32_t> cells;
  std::vector<double> out;
  for (int i = 0; i < m.nc; i += every) {
    int members[64];
    double diff[64];
    Quad c[4][20], mean[20];
    std::vector<Quad> op;
    for (int s = 0; s < O::NL; ++s) members[s] = m.perm[m.idx[packed_idx_index(m, m.inv[i], large_row(s))]];
    for (int v = 0; v < 4; ++v) {
      for (int s = 0; s < O::NL; ++s) diff[s] = U[4 * (size_t)members[s] + v] - U[4 * (size_t)i + v];
      ex.solve(m, i, O::R, O::NU, O::NL, members, diff, c[v], mean, op);
    }
    cells.push_back(i);
    for (int q = 0; q < 3 * O::NQ; ++q)
      for (int v = 0; v < 4; ++v) {
        Quad x = U[4 * (size_t)i + v];
        for (int l = 0; l < O::NU; ++l) x += c[v][l] * (Quad)FaceBasis<O::R, O::NQ>::P.v[q][l];
        out.push_back((double)x);
      }
  }
  std::ofstream(base + ".cells", std::ios::binary)
      .write(reinterpret_cast<const char*>(cells.data()), (std::streamsize)(cells.size() * 4));
  std::ofstream(base + ".faces", std::ios::binary)
      .write(reinterpret_cast<const char*>(out.data()), (std::streamsize)(out.size() * 8));
}

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "layout")) {
    std::printf("%d layouts ok\n", all_layouts());
    return 0;
  }
  Mesh m;
  if (argc < 5) return 2;
  load_mesh(std::string(argv[2]) + "/" + argv[3], m);
  const int order = std::atoi(argv[4]);
  if ((argc == 6 || argc == 7) && !std::strcmp(argv[1], "solve")) {
    set_up(m, order, 0, 0);
    if (argc == 7 && (!pack_blocks(m, 1, false) || m.bwaves != 1)) die("no layout in runs");
    solve_all(m, std::atoi(argv[5]));
    return 0;
  }
  if (argc == 6 && !std::strcmp(argv[1], "faces")) {
    const std::string base = std::string(argv[2]) + "/" + argv[3];
    set_up(m, order, 1, 0);
    const int every = std::atoi(argv[5]);
    if (order == 3) linear_faces<3>(m, base, every);
    if (order == 4) linear_faces<4>(m, base, every);
    if (order == 5) linear_faces<5>(m, base, every);
    if (order == 6) linear_faces<6>(m, base, every);
    return 0;
  }
  if (argc != 7 || std::strcmp(argv[1], "mesh")) return 2;
  const int variant = std::atoi(argv[5]), ch = std::atoi(argv[6]);
  set_up(m, order, variant, ch);
  check_layout(order, m.bwaves, m.bmax, m.nbuf, ch != 0);
  if (!layout_fits(m.d.nu, m.bwaves, m.bmax, m.nbuf, m.ustride, ch != 0)) die("a layout that does not fit");
  const int stride = buffer_stride(m.d.nu, m.bmax, m.bwaves, ch != 0);
  long peak = 0;  // kB (ru_maxrss would count the parent's)
  std::ifstream status("/proc/self/status");
  for (std::string line; std::getline(status, line);)
    if (std::sscanf(line.c_str(), "VmHWM: %ld", &peak) == 1) break;
  std::printf("bwaves %d nbuf %d bmax %d blocks %d lds %d peak_kb %ld\n", m.bwaves, m.nbuf, m.bmax,
              (int)m.boff.size() - 1, group_lds_bytes(stride, m.bmax, m.nbuf), peak);
  return 0;
}
