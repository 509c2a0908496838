// Test driver (CPU only) of the triangle kernels' block data: the LDS layout of
// the staged blocks and what set-up packs for them.  Built with csrc/setup.cpp
// and run by tests/test_blocks_host.py:
//   blocks2d layout                                every layout, ranges disjoint
//   blocks2d mesh <dir> <tag> order variant char   one mesh's blocks
// where <dir>/<tag>.txt holds "n_vert n_cell px py" and <tag>.xy, <tag>.tri the
// arrays.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <string>
#include <vector>

#include "../../paper_2105_02127_amd/csrc/internal.h"

using namespace teno;

namespace teno {
const char* last_error();
}

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
  const Dims d = dims_for(order, 0, !characteristic);
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

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "layout")) {
    std::printf("%d layouts ok\n", all_layouts());
    return 0;
  }
  if (argc != 7 || std::strcmp(argv[1], "mesh")) return 2;
  const int order = std::atoi(argv[4]), variant = std::atoi(argv[5]), ch = std::atoi(argv[6]);
  Mesh m;
  load_mesh(std::string(argv[2]) + "/" + argv[3], m);
  set_up(m, order, variant, ch);
  check_layout(order, m.bwaves, m.bmax, m.nbuf, ch != 0);
  const int stride = buffer_stride(m.d.nu, m.bmax, m.bwaves, ch != 0);
  std::printf("bwaves %d nbuf %d bmax %d blocks %d lds %d\n", m.bwaves, m.nbuf, m.bmax,
              (int)m.boff.size() - 1, group_lds_bytes(stride, m.bmax, m.nbuf));
  return 0;
}
