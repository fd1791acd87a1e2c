#include <algorithm>
#include <array>
#include <sstream>
#include <thread>

#include "forest.hpp"

namespace amr {

void Forest::init(const amr_config& cfg) {
  dim = cfg.dim;
  nlev = cfg.max_levels;
  max_patches = cfg.max_patches;
  coarsen_rule = cfg.coarsen_rule;
  for (int j = 0; j < 3; ++j) periodic[j] = j < dim ? cfg.periodic[j] : 1;
  maxc = 1;
  long long mapsize = 0;
  for (int l = 0; l < nlev; ++l) {
    n[l] = cfg.patch_cells[l];
    np[l] = (cfg.base_cells << l) / n[l];
    ratio[l] = (l + 1 < nlev) ? 2 * n[l] / cfg.patch_cells[l + 1] : 0;
    int c = 1;
    for (int j = 0; j < dim; ++j) c *= ratio[l];
    if (l + 1 < nlev) maxc = std::max(maxc, c);
    map_off[l] = (int)mapsize;
    long long m = 1;
    for (int j = 0; j < dim; ++j) m *= np[l];
    mapsize += m;
  }
  // slot ranges: explicit capacities where given, level 0 exact otherwise;
  // the remaining slots are shared equally by the other finer levels, a
  // level never getting more than its patch count, with what a capped level
  // leaves over shared again among the rest
  long long l0 = 1;
  for (int j = 0; j < dim; ++j) l0 *= np[0];
  long long full[kMaxLev] = {}, c[kMaxLev] = {};
  long long left = max_patches;
  std::vector<int> open;
  for (int l = 0; l < nlev; ++l) {
    full[l] = 1;
    for (int j = 0; j < dim; ++j) full[l] *= np[l];
    if (cfg.level_capacity[l] > 0) c[l] = std::min<long long>(cfg.level_capacity[l], full[l]);
    else if (l == 0) c[l] = l0;
    else {
      open.push_back(l);
      continue;
    }
    left -= c[l];
  }
  while (!open.empty()) {
    const long long share = std::max<long long>(1, left / (long long)open.size());
    std::vector<int> still;
    for (int l : open) {
      if (full[l] <= share) {
        c[l] = full[l];
        left -= c[l];
      } else {
        still.push_back(l);
      }
    }
    if (still.size() == open.size()) {
      for (int l : still) c[l] = share;
      left -= share * (long long)still.size();
      break;
    }
    open.swap(still);
  }
  long long used = 0;
  for (int l = 0; l < nlev; ++l) {
    pid_base[l] = (int)used;
    cap[l] = (int)c[l];
    used += c[l];
  }
  if (used > max_patches) throw std::invalid_argument("level capacities exceed max_patches");
  if (cap[0] < l0) throw std::invalid_argument("max_patches below the level-0 patch count");

  level.assign(max_patches, -1);
  parent.assign(max_patches, -1);
  nchild.assign(max_patches, 0);
  child.assign((size_t)max_patches * maxc, -1);
  coord.assign((size_t)max_patches * 3, 0);
  active.assign(max_patches, 0);
  map.assign(mapsize, -1);
  map_dirty.clear();
  touched.clear();
  touched_kids.clear();
  for (int l = 0; l < nlev; ++l) {
    free_[l].words.assign((cap[l] + 63) / 64, ~0ull);
    if (cap[l] % 64) free_[l].words.back() = (1ull << (cap[l] % 64)) - 1;
    free_[l].low = 0;
  }

  moore_.clear();
  const int rz = dim >= 3 ? 1 : 0, ry = dim >= 2 ? 1 : 0;
  for (int dz = -rz; dz <= rz; ++dz)
    for (int dy = -ry; dy <= ry; ++dy)
      for (int dx = -1; dx <= 1; ++dx)
        if (dx || dy || dz) moore_.push_back({dx, dy, dz});

  for (int l = 1; l < nlev; ++l) {
    const int r = ratio[l - 1];
    const int rr[3] = {r, dim >= 2 ? r : 1, dim >= 3 ? r : 1};
    child_regions_[l].assign((size_t)rr[0] * rr[1] * rr[2], {});
    for (size_t k = 0; k < child_regions_[l].size(); ++k) {
      const int pos[3] = {(int)k % r, (int)k / r % rr[1], (int)k / (r * rr[1])};
      for (const auto& off : moore_) {
        int d = 0, code = 0, mul = 1;
        for (int j = 0; j < 3; ++j) {
          const int w = pos[j] + off[j];
          d += (w < 0 ? 0 : (w >= rr[j] ? 2 : 1)) * mul;
          code += (off[j] + 1) * mul;
          mul *= 3;
        }
        child_regions_[l][k][d] |= 1u << code;
      }
    }
  }

  const int m0 = np[0];
  for (int z = 0; z < (dim >= 3 ? m0 : 1); ++z)
    for (int y = 0; y < (dim >= 2 ? m0 : 1); ++y)
      for (int x = 0; x < m0; ++x) {
        const int c[3] = {x, y, z};
        alloc(0, c, -1);
      }
}


bool Forest::shifted(int l, const int c[3], const int off[3], int out[3]) const {
  out[0] = out[1] = out[2] = 0;
  for (int j = 0; j < dim; ++j) {
    int v = c[j] + off[j];
    if (v < 0 || v >= np[l]) {
      if (!periodic[j]) return false;
      v = ((v % np[l]) + np[l]) % np[l];
    }
    out[j] = v;
  }
  return true;
}

void Forest::covering(int l, const int c[3], int out[3]) const {
  out[0] = out[1] = out[2] = 0;
  for (int j = 0; j < dim; ++j) out[j] = (c[j] * n[l] / 2) / n[l - 1];
}

int Forest::alloc(int l, const int c[3], int par) {
  FreeSlots& fs = free_[l];
  while (fs.low < fs.words.size() && !fs.words[fs.low]) ++fs.low;
  if (fs.low == fs.words.size()) return -1;
  const int pid = pid_base[l] + (int)(64 * fs.low) + __builtin_ctzll(fs.words[fs.low]);
  fs.words[fs.low] &= fs.words[fs.low] - 1;
  level[pid] = l;
  parent[pid] = par;
  nchild[pid] = 0;
  active[pid] = 1;
  for (int j = 0; j < 3; ++j) coord[3 * pid + j] = c[j];
  const int mi = map_index(l, c);
  map[mi] = pid;
  map_dirty.push_back(mi);
  touched.push_back(pid);
  return pid;
}

void Forest::release(int pid) {
  const int l = level[pid];
  const int c[3] = {coord[3 * pid], coord[3 * pid + 1], coord[3 * pid + 2]};
  const int mi = map_index(l, c);
  map[mi] = -1;
  map_dirty.push_back(mi);
  touched.push_back(pid);
  active[pid] = 0;
  level[pid] = -1;
  parent[pid] = -1;
  nchild[pid] = 0;
  const size_t slot = pid - pid_base[l];
  free_[l].words[slot / 64] |= 1ull << (slot % 64);
  free_[l].low = std::min(free_[l].low, slot / 64);
}

// Algorithm 1: a leaf p first makes each absent Moore neighbour q exist by
// refining the level l-1 patch that covers q (recursively), then receives its
// children.  Positions outside a non-periodic domain count as present.
void Forest::refine(int pid, std::vector<int>& created) {
  if (!active[pid]) throw MeshError("refinement of an inactive patch");
  if (!is_leaf(pid)) return;
  const int l = level[pid];
  if (l + 1 >= nlev) throw MeshError("refinement beyond the finest level");
  const int c[3] = {coord[3 * pid], coord[3 * pid + 1], coord[3 * pid + 2]};
  for (const auto& off : moore_) {
    int q[3];
    if (!shifted(l, c, off.data(), q)) continue;
    if (lookup(l, q) >= 0) continue;
    if (l == 0) throw MeshError("missing level-0 patch");
    int r[3];
    covering(l, q, r);
    const int rp = lookup(l - 1, r);
    if (rp < 0) throw MeshError("covering patch of a missing neighbour is absent");
    refine(rp, created);
  }
  const int rr = ratio[l];
  const int rz = dim >= 3 ? rr : 1, ry = dim >= 2 ? rr : 1;
  touched_kids.push_back(pid);
  int k = 0;
  for (int oz = 0; oz < rz; ++oz)
    for (int oy = 0; oy < ry; ++oy)
      for (int ox = 0; ox < rr; ++ox) {
        int cc[3] = {c[0] * rr + ox, dim >= 2 ? c[1] * rr + oy : 0, dim >= 3 ? c[2] * rr + oz : 0};
        const int q = alloc(l + 1, cc, pid);
        if (q < 0) throw CapacityError("patch pool of a level exhausted");
        child[(size_t)pid * maxc + k] = q;
        nchild[pid] = ++k;
        created.push_back(q);
      }
}

// Algorithm 2, text reading: P needs children, all of them leaves, and none
// of them may be a Moore neighbour of a same-level patch that has children.
// The literal rule instead refuses level 0 and any P with a Moore neighbour
// that has children.
bool Forest::coarsening_allowed(int pid) const {
  if (!active[pid] || is_leaf(pid)) return false;
  const int l = level[pid];
  for (int k = 0; k < nchild[pid]; ++k)
    if (!is_leaf(child[(size_t)pid * maxc + k])) return false;
  if (coarsen_rule == AMR_COARSEN_LITERAL) {
    if (l == 0) return false;
    const int c[3] = {coord[3 * pid], coord[3 * pid + 1], coord[3 * pid + 2]};
    for (const auto& off : moore_) {
      int q[3];
      if (!shifted(l, c, off.data(), q)) continue;
      const int qp = lookup(l, q);
      if (qp >= 0 && !is_leaf(qp)) return false;
    }
    return true;
  }
  // the layer of patches around the children, which fill their parent
  int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};  // the children, then with the layer
  for (int j = 0; j < dim; ++j) {
    lo[j] = coord[3 * pid + j] * ratio[l];
    hi[j] = lo[j] + ratio[l] - 1;
  }
  for (int z = lo[2] - (dim >= 3); z <= hi[2] + (dim >= 3); ++z)
    for (int y = lo[1] - (dim >= 2); y <= hi[1] + (dim >= 2); ++y) {
      const bool across = z >= lo[2] && z <= hi[2] && y >= lo[1] && y <= hi[1];
      const int step = across ? hi[0] - lo[0] + 2 : 1;  // inside, only the two ends in x
      for (int x = lo[0] - 1; x <= hi[0] + 1; x += step) {
        int q[3] = {x, y, z};
        bool in = true;
        for (int j = 0; j < dim; ++j)
          if (q[j] < 0 || q[j] >= np[l + 1]) {
            in &= periodic[j] != 0;
            q[j] += q[j] < 0 ? np[l + 1] : -np[l + 1];
          }
        if (!in) continue;
        const int qp = lookup(l + 1, q);
        if (qp >= 0 && parent[qp] != pid && !is_leaf(qp)) return false;
      }
    }
  return true;
}

void Forest::delete_children(int pid, std::vector<int>& deleted) {
  touched_kids.push_back(pid);
  for (int k = 0; k < nchild[pid]; ++k) {
    const int ch = child[(size_t)pid * maxc + k];
    deleted.push_back(ch);
    release(ch);
    child[(size_t)pid * maxc + k] = -1;
  }
  nchild[pid] = 0;
}

static bool order_less(const Forest& f, int a, int b) {
  if (f.level[a] != f.level[b]) return f.level[a] < f.level[b];
  for (int j = 2; j >= 0; --j)
    if (f.coord[3 * a + j] != f.coord[3 * b + j]) return f.coord[3 * a + j] < f.coord[3 * b + j];
  return a < b;
}

void Forest::regrid(const uint8_t* refine_req, const uint8_t* coarsen_req,
                    std::vector<int>& created, std::vector<int>& deleted) {
  std::vector<int> rq, cq;
  for (int pid = 0; pid < max_patches; ++pid) {
    if (!active[pid]) continue;
    if (refine_req && refine_req[pid] && is_leaf(pid) && level[pid] + 1 < nlev) rq.push_back(pid);
    if (coarsen_req && coarsen_req[pid] && !is_leaf(pid)) cq.push_back(pid);
  }
  std::sort(rq.begin(), rq.end(), [&](int a, int b) { return order_less(*this, a, b); });
  try {
    for (int pid : rq)
      if (active[pid] && is_leaf(pid)) refine(pid, created);
  } catch (const CapacityError&) {
    // undo: remove every patch created in this pass, newest first
    for (auto it = created.rbegin(); it != created.rend(); ++it) {
      const int q = *it;
      const int par = parent[q];
      release(q);
      if (par >= 0) {
        touched_kids.push_back(par);
        nchild[par] = 0;
        for (int k = 0; k < maxc; ++k) child[(size_t)par * maxc + k] = -1;
      }
    }
    created.clear();
    throw;
  }
  std::vector<uint8_t> fresh_parent(max_patches, 0);
  for (int q : created) fresh_parent[parent[q]] = 1;
  std::sort(cq.begin(), cq.end(), [&](int a, int b) {
    if (level[a] != level[b]) return level[a] > level[b];
    return order_less(*this, a, b);
  });
  coarsened_.clear();
  for (int pid : cq) {
    if (!active[pid] || fresh_parent[pid]) continue;
    if (coarsening_allowed(pid)) {
      delete_children(pid, deleted);
      coarsened_.push_back(pid);
    }
  }
}

std::string Forest::validate_change(const std::vector<int>& created) const {
  // R2 can only fail at patches with children near the change: the parents
  // of created patches (and the patches Algorithm 1 refined around them,
  // which are parents of created patches too), and patches one level below a
  // coarsened patch that border its former children.
  auto r2 = [&](int q) -> bool {
    const int l = level[q];
    const int c[3] = {coord[3 * q], coord[3 * q + 1], coord[3 * q + 2]};
    for (const auto& off : moore_)
      if (neighbour(l, c, off[0], off[1], off[2]) == -1) return false;
    return true;
  };
  int checked = -1;  // siblings are created together: their parent is checked once
  for (int q : created) {
    const int l = level[q];
    const int c[3] = {coord[3 * q], coord[3 * q + 1], coord[3 * q + 2]};
    if (!active[q] || lookup(l, c) != q) return "patch map disagrees with the patch table";
    int r[3];
    covering(l, c, r);
    if (lookup(l - 1, r) != parent[q]) return "parent link broken";
    if (parent[q] != checked && !r2(parent[q]))
      return "R2: a refined patch has an absent Moore neighbour";
    checked = parent[q];
  }
  for (int p : coarsened_) {
    const int l = level[p] + 1;
    if (l >= nlev) continue;
    // former children's region on level l, grown by one patch
    const int r = ratio[level[p]];
    int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    for (int j = 0; j < dim; ++j) {
      lo[j] = coord[3 * p + j] * r - 1;
      hi[j] = coord[3 * p + j] * r + r;
    }
    for (int z = lo[2]; z <= (dim >= 3 ? hi[2] : lo[2]); ++z)
      for (int y = lo[1]; y <= (dim >= 2 ? hi[1] : lo[1]); ++y)
        for (int x = lo[0]; x <= hi[0]; ++x) {
          int q3[3] = {x, y, z};
          bool in = true;
          for (int j = 0; j < dim; ++j) {
            int& v = q3[j];
            if (v < 0 || v >= np[l]) {
              if (!periodic[j]) in = false;
              else v = (v % np[l] + np[l]) % np[l];
            }
          }
          if (!in) continue;
          const int q = lookup(l, q3);
          if (q >= 0 && !is_leaf(q) && !r2(q))
            return "R2: a patch with children borders a coarsened region";
        }
  }
  return "";
}

std::string Forest::validate() const {
  std::ostringstream why;
  const int m0 = np[0];
  for (int z = 0; z < (dim >= 3 ? m0 : 1); ++z)
    for (int y = 0; y < (dim >= 2 ? m0 : 1); ++y)
      for (int x = 0; x < m0; ++x) {
        const int c[3] = {x, y, z};
        if (lookup(0, c) < 0) return "R1: a level-0 patch is missing";
      }
  for (int pid = 0; pid < max_patches; ++pid) {
    if (!active[pid]) continue;
    const int l = level[pid];
    const int c[3] = {coord[3 * pid], coord[3 * pid + 1], coord[3 * pid + 2]};
    if (lookup(l, c) != pid) return "patch map disagrees with the patch table";
    if (l > 0) {
      int r[3];
      covering(l, c, r);
      if (lookup(l - 1, r) != parent[pid]) return "parent link broken";
    }
    if (nchild[pid]) {
      for (const auto& off : moore_) {
        int q[3];
        if (!shifted(l, c, off.data(), q)) continue;
        if (lookup(l, q) < 0) {
          why << "R2: patch " << pid << " has children but a Moore neighbour is absent";
          return why.str();
        }
      }
    }
  }
  return "";
}

int Forest::levels_in_use() const {
  int m = 0;
  for (int pid = 0; pid < max_patches; ++pid)
    if (active[pid]) m = std::max(m, level[pid] + 1);
  return m;
}

int Forest::count_active() const {
  int c = 0;
  for (int pid = 0; pid < max_patches; ++pid) c += active[pid] ? 1 : 0;
  return c;
}

int Forest::count_leaves() const {
  int c = 0;
  for (int pid = 0; pid < max_patches; ++pid) c += (active[pid] && nchild[pid] == 0) ? 1 : 0;
  return c;
}

namespace {
// bits for the values 0 .. v - 1
int key_width(long long v) {
  int b = 0;
  while (b < 62 && (1LL << b) < v) ++b;
  return b;
}

// Ascending order of distinct keys whose bits [lo, hi) alone decide it: LSD
// radix sort in equal digits of at most 11 bits (a count table that stays in
// L1 and is cheap to clear), a comparison sort for few keys.  The brick order of
// 1 to 10 k leaves took 193 us on average with a comparison sort below 4096 keys
// and 16-bit digits of the whole key above, 119 us so.
void sort_keys(std::vector<uint64_t>& keys, int lo, int hi) {
  if (keys.size() < 256) {
    std::sort(keys.begin(), keys.end());
    return;
  }
  const int passes = (hi - lo + 10) / 11;
  std::vector<uint64_t> tmp(keys.size());
  std::vector<uint32_t> cnt;
  for (int p = 0; p < passes; ++p) {
    const int sh = lo + (hi - lo) * p / passes;
    const int w = lo + (hi - lo) * (p + 1) / passes - sh;
    const uint64_t mask = (1ull << w) - 1;
    cnt.assign((1u << w) + 1, 0u);
    for (const uint64_t k : keys) ++cnt[((k >> sh) & mask) + 1];
    for (size_t i = 1; i < cnt.size(); ++i) cnt[i] += cnt[i - 1];
    for (const uint64_t k : keys) tmp[cnt[(k >> sh) & mask]++] = k;
    keys.swap(tmp);
  }
}
}  // namespace

std::vector<int> Forest::sorted_active() const {
  std::vector<int> out;
  // small level maps: their index order is (z, y, x) within a level, so a
  // scan of the maps level by level yields the order without sorting
  if (map.size() <= 4 * (size_t)max_patches) {
    for (int l = 0; l < nlev; ++l) {
      size_t cells = 1;
      for (int j = 0; j < dim; ++j) cells *= (size_t)np[l];
      const int* m = map.data() + map_off[l];
      for (size_t i = 0; i < cells; ++i)
        if (m[i] >= 0) out.push_back(m[i]);
    }
    return out;
  }
  // (level, z, y, x, pid) packed into one 64-bit key when the fields fit,
  // each field as wide as this forest needs, else the comparator
  int npmax = 1;
  for (int l = 0; l < nlev; ++l) npmax = std::max(npmax, np[l]);
  const int bp = key_width(max_patches), bc = key_width(npmax), bl = key_width(nlev);
  const int ob = bl + dim * bc;  // ordering bits above the pid field
  if (bp + ob <= 64) {
    std::vector<uint64_t> keys;
    for (int pid = 0; pid < max_patches; ++pid) {
      if (!active[pid]) continue;
      uint64_t k = (uint64_t)level[pid];
      for (int j = dim - 1; j >= 0; --j) k = (k << bc) | (uint64_t)coord[3 * pid + j];
      keys.push_back((k << bp) | (uint64_t)pid);
    }
    sort_keys(keys, bp, bp + ob);
    out.reserve(keys.size());
    const uint64_t pm = (bp >= 64) ? ~0ull : ((1ull << bp) - 1);
    for (uint64_t k : keys) out.push_back((int)(k & pm));
    return out;
  }
  for (int pid = 0; pid < max_patches; ++pid)
    if (active[pid]) out.push_back(pid);
  std::sort(out.begin(), out.end(), [&](int a, int b) { return order_less(*this, a, b); });
  return out;
}


namespace {
// The low bits of v spread to every second (third) bit position.
uint64_t spread2(uint64_t v) {
  v &= 0xffffffffull;
  v = (v | (v << 16)) & 0x0000ffff0000ffffull;
  v = (v | (v << 8)) & 0x00ff00ff00ff00ffull;
  v = (v | (v << 4)) & 0x0f0f0f0f0f0f0f0full;
  v = (v | (v << 2)) & 0x3333333333333333ull;
  return (v | (v << 1)) & 0x5555555555555555ull;
}
uint64_t spread3(uint64_t v) {
  v &= 0x1fffffull;
  v = (v | (v << 32)) & 0x001f00000000ffffull;
  v = (v | (v << 16)) & 0x001f0000ff0000ffull;
  v = (v | (v << 8)) & 0x100f00f00f00f00full;
  v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
  return (v | (v << 2)) & 0x1249249249249249ull;
}
// Morton code of a patch position: bit b of coordinate j at bit b dim + j
// (x lowest; 13 bits per coordinate).
uint64_t morton(const int* c, int dim) {
  const uint64_t m13 = (1u << 13) - 1;
  if (dim == 1) return (uint64_t)c[0] & m13;
  if (dim == 2) return spread2(c[0] & m13) | (spread2(c[1] & m13) << 1);
  return spread3(c[0] & m13) | (spread3(c[1] & m13) << 1) | (spread3(c[2] & m13) << 2);
}
}  // namespace

std::vector<int> Forest::leaves_brick_order() const {
  // (level, Morton code, pid) packed into one key, each field as wide as this
  // forest needs; else the comparator on (level, code, pid)
  std::vector<int> out;
  bool packed = max_patches <= (1 << 21) && nlev <= 16;
  int npmax = 1;
  for (int l = 0; l < nlev; ++l) npmax = std::max(npmax, np[l]);
  packed &= npmax <= (1 << 13);
  if (packed) {
    const int bp = key_width(max_patches), bm = dim * key_width(npmax);
    std::vector<uint64_t> keys;
    for (int pid = 0; pid < max_patches; ++pid) {
      if (!active[pid] || nchild[pid]) continue;
      keys.push_back(((((uint64_t)level[pid] << bm) | morton(&coord[3 * pid], dim)) << bp) |
                     (uint64_t)pid);
    }
    sort_keys(keys, bp, bp + bm + key_width(nlev));
    out.reserve(keys.size());
    const uint64_t pm = (1ull << bp) - 1;
    for (uint64_t k : keys) out.push_back((int)(k & pm));
    return out;
  }
  for (int pid = 0; pid < max_patches; ++pid)
    if (active[pid] && !nchild[pid]) out.push_back(pid);
  std::sort(out.begin(), out.end(), [&](int a, int b) {
    if (level[a] != level[b]) return level[a] < level[b];
    const uint64_t ma = morton(&coord[3 * a], dim), mb = morton(&coord[3 * b], dim);
    return ma != mb ? ma < mb : a < b;
  });
  return out;
}

// A leaf's same-level neighbour in a direction exists iff it is a sibling or
// the parent's Moore neighbour in that direction has children: children come
// in complete sets, and by R2 the parent has every Moore neighbour.  So one
// mask per parent (bit = offset code of a neighbour with children) replaces the
// leaves' own neighbour lookups, and a leaf's missing regions are those that
// child_regions_ puts into the parent's neighbours without children.  Leaves
// are independent; their masks are split over host threads on large meshes.
// Meshes of 1 to 12 k patches: 829 us on average with a test of every region of
// every leaf, 226 us so.
size_t Forest::prolonged_regions(const std::vector<int>& order, std::vector<int>& out) const {
  constexpr uint32_t kFaces = 1u << 4 | 1u << 10 | 1u << 12 | 1u << 14 | 1u << 16 | 1u << 22;
  std::vector<uint32_t> kids(max_patches, 0);
  for (const int p : order) {
    if (is_leaf(p)) continue;
    const int c[3] = {coord[3 * p], coord[3 * p + 1], coord[3 * p + 2]};
    uint32_t bits = 1u << 13;
    for (const auto& off : moore_) {
      const int q = neighbour(level[p], c, off[0], off[1], off[2]);
      if (q >= 0 && !is_leaf(q)) bits |= 1u << ((off[0] + 1) + 3 * (off[1] + 1) + 9 * (off[2] + 1));
    }
    kids[p] = bits;
  }
  constexpr uint32_t kAll = (1u << 27) - 1;
  std::vector<uint32_t> miss(order.size());
  auto masks = [&](size_t from, size_t to) {
    for (size_t i = from; i < to; ++i) {
      const int pid = order[i], l = level[pid];
      miss[i] = 0;
      if (!is_leaf(pid) || l == 0) continue;
      const int P = parent[pid], r = ratio[l - 1];
      uint32_t without = kAll & ~kids[P];  // offset codes of the parent
      if (!without) continue;
      int pos[3] = {0, 0, 0};
      bool wall = false;
      for (int j = 0; j < dim; ++j) {
        const int c = coord[3 * pid + j];
        pos[j] = c - coord[3 * P + j] * r;
        wall |= !periodic[j] && (c == 0 || c == np[l] - 1);
      }
      const auto& regions = child_regions_[l][pos[0] + r * (pos[1] + r * pos[2])];
      if (!wall) {
        for (; without; without &= without - 1) miss[i] |= regions[__builtin_ctz(without)];
        continue;
      }
      for (const auto& off : moore_) {
        int d = 0, code = 0, mul = 1;
        for (int j = 0; j < 3; ++j) {
          const int v = coord[3 * pid + j] + off[j];
          const int o = j < dim && !periodic[j] && (v < 0 || v >= np[l]) ? 0 : off[j];
          const int w = pos[j] + o;
          d += (w < 0 ? 0 : (w >= (j < dim ? r : 1) ? 2 : 1)) * mul;
          code += (off[j] + 1) * mul;
          mul *= 3;
        }
        if (without >> d & 1) miss[i] |= 1u << code;
      }
    }
  };
  const size_t na = order.size();
  const unsigned nth =
      na < 32768 ? 1 : std::min(16u, std::max(1u, std::thread::hardware_concurrency()));
  if (nth == 1) {
    masks(0, na);
  } else {
    std::vector<std::thread> pool;
    for (unsigned t = 0; t < nth; ++t) pool.emplace_back(masks, na * t / nth, na * (t + 1) / nth);
    for (auto& th : pool) th.join();
  }
  size_t count = 0, faces = 0;
  for (const uint32_t b : miss) {
    count += __builtin_popcount(b);
    faces += __builtin_popcount(b & kFaces);
  }
  const size_t first = out.size(), second = first + 2 * count;
  out.resize(second + 2 * faces);
  int* a = out.data() + first;
  int* f = out.data() + second;
  for (size_t i = 0; i < na; ++i) {
    for (uint32_t b = miss[i]; b; b &= b - 1) {
      *a++ = order[i];
      *a++ = __builtin_ctz(b);
    }
    for (uint32_t b = miss[i] & kFaces; b; b &= b - 1) {
      *f++ = order[i];
      *f++ = __builtin_ctz(b);
    }
  }
  return second;
}

}  // namespace amr
