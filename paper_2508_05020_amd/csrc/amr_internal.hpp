// Internal structures shared by the host mesh manager, the kernels and the
// C-ABI layer of libamr.  Not part of the public interface (include/amr.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/amr.h"

namespace amr {

constexpr int kNG = AMR_GHOST;   // ghost layers (flux-form Eq. (9) + WENO5 need 4)
constexpr int kMaxLev = AMR_MAX_LEVELS;

// XCDs of the MI355X (gfx950): 8 dies of 32 compute units, one L2 each.
constexpr int kXcds = 8;
// A CFL-rate slot: the maximum is kept as kXcds parts (the blocks of each XCD
// raise their own, 128 bytes apart: atomics on one address are served one after
// the other), and the rate is the largest of them.
constexpr int kRateStride = 16;                  // 64-bit words between parts
constexpr int kRateWords = kXcds * kRateStride;  // words of a slot

// Per-level constants, mirrored on the device by value.
struct LevelC {
  int n;             // patch edge (cells)
  int full;          // n + 2 ng
  int np;            // patches per dimension on this level
  int cells;         // cells per dimension on this level
  int pid_base;      // first pid of this level's slot range
  int cap;           // slots of this level
  int map_off;       // offset of this level's patch map (np^dim ints)
  int ratio;         // children per dimension (2 n_l / n_{l+1}); 0 on the finest level
  long long pool_off;  // offset (doubles) of this level's pool in a state buffer
  long long stride;    // doubles per patch (nvar * full^dim)
  long long fr_off;    // offset (doubles) of this level's flux-register pool
  long long fr_stride; // doubles per patch of flux registers (2 dim nvar n^(dim-1))
  long long tag_off;   // offset (bytes) of this level's cell-tag pool
  double h, inv_h;
  // ceil(2^32 / n) and ceil(2^32 / full) where the high half of a product with
  // them is the exact quotient for every cell index of the level, of a patch's
  // interior (n_mul) or of its box (full_mul); else 0 (see div_by)
  unsigned n_mul, full_mul;
};

// Everything a kernel needs to address patch data, passed by value.
struct DevMesh {
  int dim, nvar, nlev, scheme;
  int tile;           // stage-kernel tile variant (index into Kernels::variant)
  int periodic[3];
  int max_patches, maxc;
  double gamma, gm1, igm1, eps, theta, cfl;
  int tag_buffer;
  LevelC lv[kMaxLev];
  const int* level;    // [max_patches]
  const int* coord;    // [max_patches * 3]
  const int* parent;   // [max_patches]
  const int* nchild;   // [max_patches]
  const int* child;    // [max_patches * maxc]
  const int* map;      // all levels' patch maps
};

// Work lists, all resident in one device int buffer.  `dir` (null for lists
// that no recordable call takes) is the list's entry {offset into the buffer,
// count} of the device list directory, which recorded launches read at run
// time, so that they stay valid across regrids as long as each list fits the
// grid it was recorded with.
struct ListView {
  const int* ptr;
  int count;
  const int* dir = nullptr;
};

// A list as a launch takes it: its entries; in a recorded launch the list
// buffer and the directory entry, and `count` only sizes the grid.
struct ListArg {
  const int* ptr = nullptr;
  int count = 0;
  const int* dir = nullptr;
};

// Work item of the stage kernel: a tile of a leaf, with what its block would
// else gather through the tables one dependent load after the other (level and
// position of the patch, then its neighbours, at the end the parent).  One
// 64-byte line per item, read by the scalar unit.
struct alignas(64) StageItem {
  int pid, level;
  int cf, regs;      // coarse/fine faces of the leaf; faces with flux registers
  int o[3];          // first cell of the tile in the patch
  int nb[6];         // same-level patch across each face (x-, x+, y-, ...): its pid,
                     // kNbNone, or kNbWall beyond a transmissive boundary
  int px;            // position of the patch along x (1D prolongation)
  long long parent;  // level >= 1: offset in a state buffer of the parent cell
                     // (first variable) that covers the tile's first cells
};
static_assert(sizeof(StageItem) == 64, "one line per item");
constexpr int kNbNone = -1, kNbWall = -2;

// Work item of the refluxing kernels, in the list buffer: a leaf with finer
// neighbours, with its level, position and parent cells (one load instead of
// two dependent ones before the fine patches can be looked up).
struct alignas(32) RefluxItem {
  int pid, mask, level;  // mask: faces 2 j + side with a finer patch across
  int pc[3];
  long long target;      // level >= 1: offset in a state buffer of the first
                         // parent cell it covers
};
static_assert(sizeof(RefluxItem) == 32, "eight ints in the list buffer");

// What a recording of the caller covers: dir[at] weighs `weight` in a sum that
// goes on with the next term where `cover` is negative, and else must not exceed
// it (see Kernels::check_covers).
struct CoverTerm {
  int at, weight, cover;
};
struct CoverTerms {
  static constexpr int kMax = 48;
  CoverTerm t[kMax];
  int n;
};

// Blocks of the 3D tag launch: patches and 8^3 tiles per patch of each level.
struct TagLevels {
  int count[kMaxLev], tiles[kMaxLev];
  // recorded launches: the counts are at dir[2 l] instead
  const int* dir = nullptr;
};

// Launch wrappers implemented in kernels.hip.
struct Kernels {
  // ghosts of the listed patches that have a same-level source (copies), and
  // the prolonged ones of the listed (pid, ghost region) pairs
  static void fill(const DevMesh& m, double* U, const ListArg& list, const ListArg& regions,
                   int* err, hipStream_t s);
  // Grids (blocks) of the batched launches for a list of `count` items, for
  // updating the launches of a recorded step graph after a regrid.
  static int fill_cf_grid(const DevMesh& m, int count);
  static int stage_grid(int count) { return ((count + kXcds - 1) / kXcds) * kXcds; }
  // prolonged ghost cells only, over (pid, ghost region) pairs
  static void fill_cf(const DevMesh& m, double* U, const ListArg& regions, int* err, hipStream_t s);
  // fuse = halo nodes outside the patch with a same-level source are read
  // from that source by the kernel itself; the others are prolonged by the
  // kernel too in 1D (into Uin's ghost layers; *err set where a source is
  // missing), in 2D and 3D they come from ghost layers filled before by fill_cf
  // dir (nullable, recorded launches): list directory entry whose count is read at
  // run time; `count` then only sizes the grid
  // lam_next (nullable, stage 3 only): accumulate the next step's CFL rate
  // over leaf cells not on coarse/fine faces
  // ev0/ev1 (optional): events stamped at the dispatch's own start and end.
  // lam_in (stage 1 only, optional): take dt = CFL / the rate in that slot instead of *dt,
  // write it to *dt_out and clear lam_next (the slot stage 3 accumulates in)
  // In the stage modes a tile of a leaf (level >= 1) also restricts its new
  // values into its parent patch; post corrects this where it refluxes.
  static void stage(const DevMesh& m, int mode, double* Uin, int* err, const double* Un,
                    double* out, double* fr, const StageItem* items, int count, const int* dir,
                    const double* dt, bool fuse, unsigned long long* lam_next, hipStream_t s,
                    hipEvent_t ev0 = nullptr,
                    hipEvent_t ev1 = nullptr, const unsigned long long* lam_in = nullptr,
                    double* dt_out = nullptr);
  // The stage kernel's items for a list of (pid, tile of variant m.tile) pairs;
  // cfmask: per pid the leaf's coarse/fine faces, then (from max_patches) the
  // faces with flux registers.  Built again whenever lists or tables change.
  static void stage_items(const DevMesh& m, const int* tiles, int count, const uint8_t* cfmask,
                          StageItem* items, hipStream_t s);
  // list: of RefluxItem, which start at a multiple of their size in the list buffer
  static void reflux(const DevMesh& m, int mode, double* out, const double* fr,
                     const ListArg& list, const double* dt, double w,
                     unsigned long long* lam_next, hipStream_t s);
  // refluxing with what it changes of the leaves' restriction, and the
  // restriction of the patches with children of level finest - 1 (plist) in one
  // launch; the stage kernel has restricted the leaves.  Recorded, plist's
  // directory entry follows rlist's.
  static void post(const DevMesh& m, int mode, double* out, const double* fr,
                   const ListArg& rlist, const ListArg& plist, const double* dt, double w,
                   unsigned long long* lam_next, hipStream_t s);
  static void restrict_level(const DevMesh& m, double* U, const ListArg& list, hipStream_t s);
  static void max_rate(const DevMesh& m, const double* U, const ListArg& list,
                       unsigned long long* lam_bits, hipStream_t s);
  static void zero_rate(unsigned long long* slot, hipStream_t s);
  // dt = cfl / rate; also clears the slot `clear` (nullable), the next accumulator
  static void dt_from_rate(const DevMesh& m, const unsigned long long* lam_bits,
                           double* dt, unsigned long long* clear, hipStream_t s);
  // fuse: halo cells read from same-level neighbours directly; ghost layers
  // hold only the prolonged cells (filled by fill_cf beforehand)
  static void tag(const DevMesh& m, const double* U, const ListArg& list,
                  uint8_t* has_tag, uint8_t* raw, bool fuse, hipStream_t s);
  // 3D, fused halo: tag flags of every active patch (`list` in level order,
  // level_count patches per level, recorded launches read them at level_dir[2 l];
  // prolonged regions filled before); mask:
  // scratch of max_patches ints; raw (nullable): the tag of each patch's own
  // cells and, in a leaf's ghost places, of the prolonged cells within tag_buffer
  static void tag_flags3(const DevMesh& m, const double* U, const ListArg& list,
                         const int* level_count, const int* level_dir, const ListArg& regions,
                         int* mask, uint8_t* has_tag, uint8_t* raw, hipStream_t s);
  // cells of the leaves with a tag within tag_buffer; shared: raw as tag_flags3
  // (3D) writes it, else as tag does; level_leaves (nullable): leaves per level,
  // the list in level order (recorded launches read them at level_dir[2 l])
  static void cell_tags(const DevMesh& m, const uint8_t* raw, const ListArg& leaves,
                        const int* level_leaves, const int* level_dir, bool shared, uint8_t* out,
                        hipStream_t s);
  static void requests(const DevMesh& m, const uint8_t* has_tag, const uint8_t* active_leaf,
                       int nslots, uint8_t* refine, uint8_t* coarsen, hipStream_t s);
  static void prolong_new(const DevMesh& m, double* U, const ListArg& list, int* err,
                          hipStream_t s);
  // sets the error flag when a list directory entry has outgrown a recording
  static void check_covers(const int* dir, const CoverTerms& c, int* err, hipStream_t s);
  // blocks per patch of edge n of the 3D tag launch and of the dilation
  static int tag_tiles(int n);
  static int cell_tiles(int dim, int n);
  static void scatter_int(int* dst, const int* pairs, int npairs, hipStream_t s);
  static void count_nonzero(const uint8_t* a, int n, int* out, hipStream_t s);
  static void check(const DevMesh& m, const double* U, const ListArg& list, int* bad,
                    hipStream_t s);
  // Tile variants of the stage kernel: extents (cells) and block size.
  struct TileVariant {
    int dim, tx, ty, tz, threads;
    int both = 0;  // 2D: x and y edges computed in one sweep
  };
  static int num_variants();
  static TileVariant variant(int v);
  // Whether variant v fits every level's patch edge.
  static bool variant_fits(int v, int dim, const int* n, int nlev);
  // First fitting variant of a dimension (the default), -1 when none fits.
  static int default_variant(int dim, const int* n, int nlev);
  static int tiles_per_patch(int v, int n);
};

// Stage modes of the fused RHS/combine kernel.
enum StageMode { kModeRHS = 0, kModeStage1 = 1, kModeStage2 = 2, kModeStage3 = 3 };

}  // namespace amr
