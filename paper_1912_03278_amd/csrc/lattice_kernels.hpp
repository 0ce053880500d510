// Launch interface of the fused lattice passes (lattice_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <utility>
#include <vector>

#include "ihmc_internal.hpp"

namespace ihmc {

// PASS_PAIR, PASS_FUSED: two middle steps in one launch, and as many as a round's launches
// take (2D groups; timing only).
enum PassMode : int {
  PASS_FIRST = 0,
  PASS_MIDDLE = 1,
  PASS_LAST = 2,
  PASS_MEASURE = 3,
  PASS_FORCE = 4,
  PASS_PAIR = 5,
  PASS_FUSED = 6
};

struct TileShape {
  int bx, by, bz;
};

// Built-in tile class of a lattice (row length L0, planes L2; L2 = 1 in 2D):
// the class that the context uses unless its tuning table has an entry for it.
int tile_class(int ndim, int L0, int L2);

// Number of tile classes of a dimension (2 or 3); classes are 0 .. n-1.
int tile_class_count(int ndim);

// Tile extents used for a state precision (4 or 8 bytes), dimension (2 or 3)
// and tile class.
TileShape tile_shape(int precision, int ndim, int cls);

// Chains small enough for one workgroup's LDS run whole trajectories per launch
// (lattice_resident): their launch group has this tile class, and one Tile
// entry per chain.
constexpr int RESIDENT_CLASS = -1;
// Chains of the inverse (phi) formulation run whole trajectories per launch
// too (lattice_resident_phi, FP64): their own launch group.
constexpr int RESIDENT_PHI_CLASS = -2;
// Largest phi-form chain (sites) that fits one workgroup's LDS.
int resident_phi_max_sites(bool site_field);
hipError_t launch_lattice_resident_phi(int ndim, const ChainDev* chains, const Tile* tiles, int n_chains, int n_traj,
                                       hipStream_t s);
// Largest chain (sites) of a state precision (4 or 8 bytes) that fits, with or
// without a per-site field.
int resident_max_sites(int precision, bool site_field);
// Largest members of a resident launch, which set its workgroup size and LDS:
// sites, site vectors (16 bytes each, rows padded to whole ones) and the values
// of one padded array.
struct ResidentShape {
  int max_sites = 0, max_vectors = 0, max_values = 0;
};
void resident_extend(ResidentShape& s, const ChainDev& c);
// n_traj trajectories of each of n_chains resident chains (tiles[b].chain is
// block b's chain); n_traj = 0 measures S and the estimator sums instead.
hipError_t launch_lattice_resident(int precision, int ndim, const ResidentShape& r, const ChainDev* chains,
                                   const Tile* tiles, int n_chains, int n_traj, hipStream_t s);

// Several middle steps per launch (2D): `steps` of them (2 or 4) on tiles of at most bx
// x by sites, threads that own H rows of a 4-site chunk column each, workgroups of
// `threads` threads (at most max_threads) and `rows` LDS rows per array.
struct StepShape {
  int steps = 0, bx = 0, by = 0, H = 0, max_threads = 0, threads = 0, rows = 0;
};
// max_middle: middle steps of the chain that has most.
StepShape choose_steps(int precision, const std::vector<std::pair<int, int>>& lattices, int max_middle);
void steps_tiles(const StepShape& g, int chain, int L0, int L1, std::vector<Tile>& out);
// Middle steps j .. j + max_steps - 1 (at most g.steps; each chain those that it
// has) as launch index k over n_tiles entries of steps_tiles.  full: on all rows
// of halo, whatever a chain has left (any choice gives the same values).
hipError_t launch_lattice_steps(int precision, const StepShape& g, const ChainDev* chains, const Tile* tiles,
                                int n_tiles, int j, int k, int max_steps, bool full, hipStream_t s);

// Launch one pass of kind `mode` (pass index j of the trajectory, which sets
// the kick and drift; launch index k, which sets the field buffers) over n_tiles
// consecutive entries of `tiles`; all tiles must belong to chains of the given
// precision, dimension and tile class.  A LAST launch with j < 0 runs every
// chain's own last pass (j = n_pass - 1), with the launch index that follows its
// middle steps when k != 0 (k per launch) or j when k == 0.  sole: no other
// 3D launches run beside a 3D one's; aligned: all chains' rows start at multiples of 32
// bytes (the kind of a 3D middle launch's stores, not its results, depends on them).
hipError_t launch_lattice_pass(int precision, int ndim, int cls, int mode, const ChainDev* chains,
                               const Tile* tiles, int n_tiles, int j, int k, hipStream_t s, bool sole = true,
                               bool aligned = true);

}  // namespace ihmc
