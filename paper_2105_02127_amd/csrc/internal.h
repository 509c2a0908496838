// Library-internal data shared by the host set-up and the device launches.
#pragma once

#include <cstdint>
#include <memory>
#include <string>
#include <utility>
#include <vector>

#include "../../include/teno.h"

namespace teno {

// Cells per wavefront tile of the reconstruction kernels: four of the 64 lanes
// per cell.
constexpr int kTile = 16;

// Sizes of one order (Sec. 2.2 eq. 03 with N_k counting the constant term;
// N_s = 2 N_k cells including the target, so 2 N_k - 1 least-squares rows).
struct Dims {
  int order = 0, r = 0;
  int nu = 0;      // unknowns of the large stencil, N_k - 1
  int nl = 0;      // rows of the large stencil
  int nq = 0;      // Gauss points per face
  int rows = 0;    // all stencil rows: 3 * 11 small + nl
  int rows4 = 0;   // rows rounded up to a multiple of 4 (int4 loads)
  int J = 0;       // operator entries per cell: 3 * 5 * 11 + nu * nl
};

Dims dims_for(int order, int nq_req);

// Largest number of distinct stencil members that 16 consecutive cells of the
// internal order may have.
constexpr int kMaxTileMembers = 384;
static_assert(kMaxTileMembers <= 512, "member slots take 9 bits of the adjoint's slot word");

constexpr int kSmallRows = 11;
constexpr int kSmallCoef = 5;

// ---- matrix-free least squares (device layouts) ---------------------------
// Cells are packed in an order of their own, recursive bisection of the
// centroids into blocks of several tiles and into tiles of 16 (the Morton
// order's runs are compact only where they fall on its quadrants); this
// section's arrays and the adjoint's lists are in packed order.  A block stages
// the distinct members of all its cells' stencils in LDS: per member a geometry
// record and its state.  A record holds, in the block's frame: the centroid (x, y), the weight |V|^2 of the
// member's row, and the central moments E[H_a(X) H_b(Y)], 2 <= a + b <= r, in
// the basis order (xx, xy, yy, xxx, ...).  H_n is the monic Hermite polynomial
// of variance kHermite; being an Appell sequence it shifts by the binomial
// rule that monomials obey, so the rows of an almost orthogonal basis cost
// what monomial rows cost.  A stencil's basis is centred on the mean of its
// members (its centre, exact in FP32).  Records are stored with the stride they
// have in LDS, an odd number of 16-byte units, so that they start on different
// banks and the copy to LDS is a plain one.
constexpr double kHermite = 0.4;  // the frame has unit variance over a stencil
constexpr int rec_units(int nu) { return ((nu + 2) / 2) | 1; }  // nu + 1 doubles
// LDS of one staged block: states (32 B each), records.
constexpr int block_lds_bytes(int nu, int members) { return members * (16 * rec_units(nu) + 32); }
// A workgroup holds two of them (one when they do not fit), and as many lists of
// member ids (padded to whole wavefront loads).  In characteristic variables a
// wavefront's Gram matrices (4 stencils x 10 entries per cell) take the place of
// its block's members once these are read, and at order 3 they are the longer of
// the two: the buffers lie buffer_stride apart, and the lists behind them.  Host
// and kernels form every offset from these functions.
constexpr int kCharGramDoubles = kTile * 4 * 10;
constexpr int gram_bytes(int waves) { return waves * kCharGramDoubles * (int)sizeof(double); }
constexpr int ids_bytes(int members) { return (members + 63) / 64 * 256; }
constexpr int buffer_stride(int nu, int members, int waves, bool characteristic) {
  const int staged = block_lds_bytes(nu, members), gram = characteristic ? gram_bytes(waves) : 0;
  return staged > gram ? staged : gram;
}
constexpr int buffer_offset(int stride, int buffers, int k) { return (buffers == 2 ? k & 1 : 0) * stride; }
constexpr int ids_offset(int stride, int members, int buffers, int k) {
  return buffers * stride + (buffers == 2 ? k & 1 : 0) * ids_bytes(members);
}
constexpr int group_lds_bytes(int stride, int members, int buffers) {
  return buffers * (stride + ids_bytes(members));
}
constexpr int kLdsPerCu = 160 * 1024;
// A tile by itself (small meshes): its staged block; over it, once read, the
// coefficients [15 + nu][64] and in characteristic variables the Gram matrices.
constexpr int small_lds_bytes(int nu, int members, bool characteristic) {
  const int staged = block_lds_bytes(nu, members);
  const int coef = (3 * 5 + nu) * 512 + (characteristic ? gram_bytes(1) : 0);
  return staged > coef ? staged : coef;
}
// The adjoint: the block's records, and an accumulator per member of each tile.
constexpr int adjoint_lds_bytes(int nu, int members, int waves, int ustride) {
  return 16 * rec_units(nu) * members + waves * ustride * 4 * (int)sizeof(double);
}
constexpr int kSlotBits = 10;       // of a member's slot in its block
constexpr int kMaxAdjMembers = 512; // of a tile: nine bits of the adjoint's slots
constexpr bool layout_fits(int nu, int waves, int members, int buffers, int ustride, bool characteristic) {
  return members <= 1 << kSlotBits && ustride <= kMaxAdjMembers &&
         group_lds_bytes(buffer_stride(nu, members, waves, characteristic), members, buffers) <= kLdsPerCu &&
         small_lds_bytes(nu, members, characteristic) <= kLdsPerCu &&
         adjoint_lds_bytes(nu, members, waves, ustride) <= kLdsPerCu;
}
// Tiles (wavefronts) per block: workgroups of four, two or more to a CU, at
// orders 3 and 4; at orders 5 and 6, whose records are longer and whose
// registers allow two wavefronts per SIMD, one of eight, whose cells share more
// members.
constexpr int block_tiles(int order) { return order >= 5 ? 8 : 4; }
constexpr int kMaxBlockTiles = 8;
// Time of a block's reconstruction relative to others', by which a batch's ranges
// are balanced: us of 180,000 cells by order, for the tiles that the block has.
constexpr double block_cost(int order, int tiles_per_block, int n_tiles, int block) {
  const int left = n_tiles - block * tiles_per_block;
  const double us = order == 3 ? 49.0 : (order == 4 ? 69.0 : (order == 5 ? 109.0 : 178.0));
  return us * (left < tiles_per_block ? left : tiles_per_block);
}
// LDS a workgroup of w tiles may take to keep eight wavefronts on a CU
constexpr int lds_budget(int w) { return w >= 8 ? kLdsPerCu : kLdsPerCu / 8 * w; }
// Packed symmetric inverses of the normal matrices of a cell's stencils: three
// small ones (degree 2), then the large one, each its upper triangle row by
// row in 16-byte pairs.  Lane g of a cell loads pairs 4q + g, so a tile holds
// [q][64 lanes][2]; a stencil is padded to whole groups of four pairs.
constexpr int sym_quads(int n) { return ((n * (n + 1) / 2 + 1) / 2 + 3) / 4; }
constexpr int normal_quads(int nu) { return 3 * sym_quads(kSmallCoef) + sym_quads(nu); }
// Row slots of a tile: lane g of a cell owns rows 4j + g of each stencil; its
// member slots, ten bits each, three to a word, stencil by stencil and j by j,
// in words [word][64 lanes].  Lanes without a row name their own cell
// (difference 0).
constexpr int row_groups(int nrow) { return (nrow + 3) / 4; }
constexpr int lane_groups(int nl) { return 3 * row_groups(kSmallRows) + row_groups(nl); }
constexpr int slot_words(int nl) { return (lane_groups(nl) + 2) / 3; }
// Cells of which a stencil's normal matrix would cost digits (setup.cpp,
// normal_bound) are solved with the operators of all four stencils instead, four
// to a wavefront: lane h of a cell's sixteen owns rows 16j + h of each stencil.
// M^T in the basis of the reference triangle, per four cells [chunk][64 lanes], a
// chunk per group of rows and coefficient, stencil by stencil.  Rare: none on a
// jittered periodic mesh.
constexpr int kKeptCells = 4;
constexpr int kept_row_groups(int nrow) { return (nrow + 15) / 16; }
constexpr int kept_groups(int nl) { return 3 * kept_row_groups(kSmallRows) + kept_row_groups(nl); }
constexpr int kept_chunks(int nl, int nu) {
  return 3 * kept_row_groups(kSmallRows) * kSmallCoef + kept_row_groups(nl) * nu;
}
constexpr int adj_words(int nl) { return (lane_groups(nl) + 1) / 2; }  // 16 bits each

void set_error(const std::string& msg);
int fail(int code, const std::string& msg);

// Vectors whose elements resize leaves unset: their pages are first touched by the
// threads that fill them.
template <class T>
struct Unset : std::allocator<T> {
  template <class U>
  struct rebind {
    typedef Unset<U> other;
  };
  template <class U>
  void construct(U* p) {
    ::new ((void*)p) U;
  }
  template <class U, class... A>
  void construct(U* p, A&&... a) {
    ::new ((void*)p) U(std::forward<A>(a)...);
  }
};

// Operator entries by position (packed_M_offset), formed on request: nothing is
// stored, so a whole stencil is better read through stencil_operator.
struct Mesh;
struct Operators {
  const Mesh* mesh = nullptr;
  double operator[](int64_t at) const;
};

struct Mesh {
  // ---- geometry, user order ----
  int nv = 0, nc = 0, nf = 0;
  double P[2] = {0.0, 0.0};           // period per axis, 0 = open axis
  double lo[2] = {0.0, 0.0}, hi[2] = {1.0, 1.0};  // box of the centroids (open axes)
  std::vector<int32_t> tri;           // [nc][3] counter-clockwise
  std::vector<double> X;              // [nc][3][2] vertices unwrapped about v0
  std::vector<double> area, cen;      // [nc], [nc][2]
  std::vector<int32_t> fL, fR, fLe, fRe;  // face -> L/R cell (user id), local edges
  std::vector<double> fnx, fny, flen;     // unit normal out of L, edge length
  std::vector<int32_t> cface;         // [nc][3] face of each local edge
  // boundary faces (an edge with one cell, on an open axis): fR = fRe = -1
  std::vector<int32_t> bface;         // [n_bface] face id, in creation order
  std::vector<int32_t> bkind;         // [n_bface] TENO_BC_* (default transmissive)
  std::vector<double> bstate;         // [n_bface][4] prescribed states
  bool open() const { return !(P[0] > 0.0 && P[1] > 0.0); }

  // ---- set-up ----
  bool ready = false;
  teno_params prm{};
  Dims d;
  std::vector<int32_t> perm, inv;     // perm[internal] = user, inv[user] = internal
  double min_rcond = 1.0;

  // ---- packed device images, internal order, tile-major ----
  int n_pad = 0, n_tiles = 0;
  Operators M;                  // after set-up
  std::vector<int32_t> idx;     // [n_tiles][rows4][16][4] stencil members (internal; host)
  // distinct stencil members of each tile (the adjoint's accumulators)
  int ustride = 0;              // list length per tile (largest count, rounded up)
  std::vector<int32_t> tmem;    // [n_tiles][ustride] sorted, padded with the last
  std::vector<int32_t> tcount;  // [n_tiles] distinct members of each tile (unpadded)
  std::vector<int32_t> nbinfo;  // [n_pad][4]: 3 neighbours + packed edge/side bits
  std::vector<double> geo;      // [n_pad][10]: (nx, ny, len) x 3 edges, area
  std::vector<int32_t> user_of; // [n_pad] user id (diagnostics)
  // face-ordered flux data: faces sorted by their L cell's internal index
  std::vector<int32_t> face_cells;  // [nf][4]: L, R (internal; L again on a boundary
                                    //   face), eL | eR << 2, boundary index or -1
  std::vector<double> face_geo;     // [nf][4]: nx, ny (out of L), |A|, 0
  std::vector<int32_t> bface_sorted; // [n_bface]: face-ordered index of boundary face b
  std::vector<int32_t> cell_faces;  // [n_pad][4]: sorted face of local edges 0..2;
                                    //   bit e of [3] set when the cell is that face's L
  std::vector<double> vol;          // [n_pad] |V| (1 for padding cells)
  // matrix-free least squares: blocks of bwaves tiles, nbuf of them in LDS
  int bwaves = 0, nbuf = 2;
  int bmax = 0;                    // largest member count of a block
  std::vector<int32_t> pack;       // [n_pad] internal cell of each packed position, -1: none
  std::vector<int32_t> boff;       // [n_blocks + 1] first member of a block
  std::vector<int32_t> bmem;       // [n_blocks][bmax] member cells (internal), the block's own
                                   // first; rest 0: read at once, without boff
  std::vector<double, Unset<double>> brec;  // geometry records, rec_units units each
  std::vector<uint32_t> bslot;     // [n_tiles][slot_words][64]
  std::vector<double, Unset<double>> N;     // [n_tiles][normal_quads][64][2]
  std::vector<double, Unset<double>> jac;   // [n_pad][4]: a third of the map's columns, block frame
  std::vector<float> centre;       // [n_pad][4][2]: centre of each stencil's basis, block
                                   // frame, relative to the cell
  // cells solved with operators (-1 in pack)
  std::vector<int32_t> kept;       // [kKeptCells n] internal cell, -1: none
  std::vector<int32_t> kept_rows;  // [n][kept_groups][64] member of each row (no row: the cell)
  std::vector<double> kept_ops;    // [n][kept_chunks][64]
  // adjoint accumulation order, by lane and row group as bslot, 16 bits each,
  // [n_tiles][adj_words][64]: slot in the tile's list | round << 9, where
  // round = how many earlier lanes of the row group name the same member
  std::vector<uint32_t> aslot;
  // reverse member lists (adjoint gather): the tile member slots naming cell j
  std::vector<int32_t> rev_ptr; // [n_cell + 1]
  std::vector<int32_t> rev_ent; // tile * ustride + slot, by tile; then the rows of kept
                                // cells, n_tiles * ustride + position in kept_rows
};

// Stencil row order of a cell: rows 0..32 hold the three small stencils
// (row s of small stencil k is row 11k + s), then the nl large-stencil rows.
constexpr int small_row(int k, int s) { return kSmallRows * k + s; }
constexpr int large_row(int s) { return 3 * kSmallRows + s; }

// Entry l of row s of stencil k (3 = large) of an internal cell.
inline int64_t packed_M_offset(const Dims& d, int internal, int k, int s, int l) {
  return (int64_t)internal * d.J + (k < 3 ? (k * kSmallRows + s) * kSmallCoef
                                          : 3 * kSmallRows * kSmallCoef + s * d.nu) + l;
}

inline int64_t packed_idx_index(const Mesh& m, int internal, int row) {
  int t = internal / kTile, c = internal % kTile;
  return (((int64_t)t * m.d.rows4 + (row >> 2)) * kTile + c) * 4 + (row & 3);
}

int mesh_create(int32_t n_vert, const double* xy, int32_t n_cell, const int32_t* tri,
                const double* period, Mesh& m);
int mesh_setup(Mesh& m, const teno_params& p);
// M[l][s] of stencil k of (user) cell, in the monomials xi^a eta^b of the reference
// triangle less their means, formed on request.
void stencil_operator(const Mesh& m, int cell, int k, double* M);

}  // namespace teno

struct teno_mesh {
  teno::Mesh m;
};
