"""Prolonged ghost regions of a mesh (the list that the ghost fill, the stage
kernel's flux registers and the tagger work from) against the definition: the
region's offset, with components that leave the domain through a wall set to
zero, points at a position without a same-level patch.  Walls and periodic
sides, child ratios 1 to 8, random refinement; the list is compared exactly.
Also the rows reported as changed: after applying them a copy of the tables
equals the tables."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include "forest.hpp"
using namespace amr;
#define REQUIRE(c) do { if (!(c)) { printf("line %d\n", __LINE__); return 1; } } while (0)
int main(int argc, char** argv) {
  amr_config cfg;
  std::memset(&cfg, 0, sizeof cfg);
  cfg.dim = atoi(argv[1]);
  cfg.base_cells = atoi(argv[2]);
  cfg.max_levels = argc - 4;
  for (int l = 0; l < cfg.max_levels; ++l) cfg.patch_cells[l] = atoi(argv[4 + l]);
  for (int j = 0; j < 3; ++j) cfg.periodic[j] = atoi(argv[3]) >> j & 1;
  long long total = 0;
  for (int l = 0; l < cfg.max_levels; ++l) {
    long long m = 1;
    for (int j = 0; j < cfg.dim; ++j) m *= (cfg.base_cells << l) / cfg.patch_cells[l];
    total += m;
  }
  cfg.max_patches = (int)total;
  Forest f;
  f.init(cfg);
  f.map_dirty.clear();
  f.touched.clear();
  f.touched_kids.clear();
  auto level = f.level, parent = f.parent, nchild = f.nchild, coord = f.coord, child = f.child,
       map = f.map;
  std::mt19937 rng(3);
  auto uniform = [&] { return std::uniform_real_distribution<>(0, 1)(rng); };
  long long entries = 0;
  for (int it = 0; it < 12; ++it) {
    std::vector<uint8_t> rq(f.max_patches), cq(f.max_patches);
    const double x0[3] = {uniform(), uniform(), uniform()}, rad = 0.1 + 0.3 * uniform();
    for (int p = 0; p < f.max_patches; ++p) {
      if (!f.active[p]) continue;
      double d = 0;
      for (int j = 0; j < f.dim; ++j) {
        const double x = (f.coord[3 * p + j] + 0.5) / f.np[f.level[p]] - x0[j];
        d += x * x;
      }
      rq[p] = d < rad * rad && uniform() < 0.7;
      cq[p] = d >= rad * rad && uniform() < 0.5;
    }
    std::vector<int> created, deleted;
    f.regrid(rq.data(), cq.data(), created, deleted);
    REQUIRE(f.validate().empty() && f.validate_change(created).empty());
    for (int m : f.map_dirty) map[m] = f.map[m];
    for (int q : f.touched) {
      level[q] = f.level[q];
      parent[q] = f.parent[q];
      nchild[q] = f.nchild[q];
      for (int j = 0; j < 3; ++j) coord[3 * q + j] = f.coord[3 * q + j];
    }
    for (int q : f.touched_kids) {
      nchild[q] = f.nchild[q];
      for (int k = 0; k < f.maxc; ++k) child[q * f.maxc + k] = f.child[q * f.maxc + k];
    }
    f.map_dirty.clear();
    f.touched.clear();
    f.touched_kids.clear();
    REQUIRE(level == f.level && parent == f.parent && nchild == f.nchild && coord == f.coord &&
            child == f.child && map == f.map);

    const std::vector<int> order = f.sorted_active();
    std::vector<int> want, faces, got{-5};
    for (int pid : order) {
      if (!f.is_leaf(pid) || f.level[pid] == 0) continue;
      const int l = f.level[pid], *c = &f.coord[3 * pid];
      for (const auto& off : f.moore()) {
        int o[3], code = 0, mul = 1, zero = 0;
        for (int j = 0; j < 3; ++j) {
          const int v = c[j] + off[j];
          o[j] = j < f.dim && !f.periodic[j] && (v < 0 || v >= f.np[l]) ? 0 : off[j];
          code += (off[j] + 1) * mul;
          mul *= 3;
          zero += off[j] == 0;
        }
        if (f.neighbour(l, c, o[0], o[1], o[2]) >= 0) continue;
        want.insert(want.end(), {pid, code});
        if (zero == 2) faces.insert(faces.end(), {pid, code});
      }
    }
    const size_t second = f.prolonged_regions(order, got);
    REQUIRE(got.front() == -5 && second == 1 + want.size());
    want.insert(want.end(), faces.begin(), faces.end());
    REQUIRE(std::vector<int>(got.begin() + 1, got.end()) == want);
    entries += (long long)want.size();
    const std::vector<int> bricks = f.leaves_brick_order();
    REQUIRE((int)bricks.size() == f.count_leaves());
    for (size_t i = 1; i < bricks.size(); ++i) REQUIRE(f.level[bricks[i - 1]] <= f.level[bricks[i]]);
  }
  REQUIRE(entries > 0 || f.np[0] == 1);  // one level-0 patch: level 1 is complete
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("forest")
    (d / "main.cpp").write_text(DRIVER)
    csrc = os.path.join(ROOT, "paper_2508_05020_amd", "csrc")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run([shutil.which("g++"), "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{csrc}",
                    f"-I{ROOT}/include", f"-I{rocm}/include", str(d / "main.cpp"),
                    os.path.join(csrc, "forest.cpp"), "-lpthread", "-o", str(d / "main")], check=True)
    return str(d / "main")


@pytest.mark.parametrize("dim,base,patches", [
    (1, 64, "16,16"), (1, 64, "8,8,8"), (1, 32, "8,16"), (2, 64, "32,16,16"), (2, 96, "24,24,24"), (2, 32, "8,16"),
    (2, 64, "32,8"), (3, 64, "16,16,8"), (3, 32, "8,8,8"), (3, 16, "8,16"), (3, 8, "8,8")])
@pytest.mark.parametrize("periodic", [0, 1, 2, 7])
def test_prolonged_regions(driver, dim, base, patches, periodic):
    r = subprocess.run([driver, str(dim), str(base), str(periodic), *patches.split(",")],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
