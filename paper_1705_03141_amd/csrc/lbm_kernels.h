// lbm_kernels.h -- launch-side view of the kernels (argument blocks and launchers).
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_cell.h"
#include "lbm_device.h"

namespace lbm {

// Thread layout of the step kernel: one thread per cell of a TX x TY tile; the first
// 2(TX+2) + 2TY threads also pull one cell of the ring around the tile.
template <int TX, int TY>
struct StepTile {
  static constexpr int kThreads = TX * TY;
  static constexpr int kRing = 2 * (TX + 2) + 2 * TY;
  static constexpr int SX = TX + 4, SY = TY + 4, kStaged = SX * SY;  // scalars, 2-cell halo
  static constexpr int DX = TX + 2, DY = TY + 2, kDense = DX * DY;   // densities, 1-cell ring
  static constexpr int kStagePerThread = (kStaged + kThreads - 1) / kThreads;
  static_assert(kThreads % 64 == 0, "tile must be whole waves");
  static_assert(kRing <= kThreads, "ring larger than the tile");
};

struct StepArgs {
  const void* g_in;      // populations written by the previous step (storage type)
  const float* sc_in;    // scalars written by the previous step
  void* g_out;
  float* sc_out;
  const float* init;     // init mode: rho_r, rho_b, ux, uy, uz planes of ncells floats
  const float* outlet;   // outlet record of the current time (outflow face only)
  long long step;
  int init_mode;
  int zchunk, tiles_x, tiles_y, nchunks;
  // with lateral walls: the tiles [tx_lo, tx_hi) x [ty_lo, ty_hi), none of whose cells and ring
  // cells lies on a wall
  int tx_lo, tx_hi, ty_lo, ty_hi;
  int* unstable;         // set to 1 by a cell whose density is NaN, infinite or <= 0
  int skip_unstable;     // 1: workgroups of a flagged lattice return at once (batches)
  Geo geo;
  PullConst pc;
  CollideParams cp;
  GroupRates rates;
};

// The step by bricks (lbm_brick.h).  8 x 4 x 4 cells while that gives every one of the 256 compute units at
// most one workgroup (32^3: 9.8 us against 11.0 with the larger brick), else 16 x 4 x 4, which pulls 2.5
// cells per cell instead of 2.8 (48^3: 19.4 against 22.3 us).
inline long long bricks_of(const Geo& g, int bx) {
  return (long long)((g.nx + bx - 1) / bx) * ((g.ny + 3) / 4) * ((g.nz + 3) / 4);
}
inline bool small_bricks(const Geo& g) { return bricks_of(g, 8) <= 256; }
inline long long brick_rounds(const Geo& g) { return small_bricks(g) ? 1 : (bricks_of(g, 16) + 255) / 256; }

// Blocks of a lattice's launch, or of its part of a batch's: a multiple of 8.
inline long long step_blocks(const StepArgs& a) { return ((long long)a.tiles_x * a.tiles_y * a.nchunks + 7) / 8 * 8; }

// Block L of the nb blocks of a lattice -> z chunk and tile; a chunk from nchunks on is a block of
// padding.  The hardware sends blocks x, x + 8, x + 16 ... to XCD x: that one takes a contiguous range,
// so that neighbouring tiles share an L2.  (With the blocks as they come, where their number is no
// multiple of 8: 85^3 80 against 57 us per step in FP32, 70^3 57 against 43, 150^3 323 against 269,
// 60^3 31.6 against 29.3.)
__host__ __device__ inline void place_of(const StepArgs& a, int L, int nb, int& chunk, int& tile) {
  L = (L & 7) * (nb >> 3) + (L >> 3);
  const int ntiles = a.tiles_x * a.tiles_y;
  chunk = L / ntiles;
  tile = L - chunk * ntiles;
}

// Whether a tile of a lattice with lateral walls takes the plain population loads: none of its
// cells and ring cells lies on a wall.  One launch covers all tiles; the others, the frame,
// branch to the loads that mirror at the walls.  (One launch per part of the frame, each with
// an instance that mirrors at its walls only, fetched the ring cells shared across launches from
// HBM again and cost up to 1.7 times the time of a step without walls.)
__host__ __device__ inline bool interior_tile(const StepArgs& a, int txi, int tyi) {
  return txi >= a.tx_lo && txi < a.tx_hi && tyi >= a.ty_lo && tyi < a.ty_hi;
}

// Arguments of the outlet and read-back kernels.
struct AuxArgs {
  const void* g_in;
  const float* sc_in;
  const float* init;
  const float* outlet_in;  // outlet record of the previous time
  float* outlet_out;       // outlet record of the current time
  long long step;
  int init_mode;
  Geo geo;
  PullConst pc;
  CollideParams cp;
};

struct DiagQuery {
  double xc, yc, zc, r_in, r_out;
};

// A pass over the lattice that hands every cell's macroscopic state to a consumer (lbm_scan.h):
// its split into 64 x 4 columns and z chunks, and the consumer's arguments.
enum ScanKind { kScanCoarse = 0, kScanDiag = 1 };

struct ScanArgs {
  int tiles_x, tiles_y, zchunk, nchunks;
  // coarse state: means over blocks of factor^3 cells, velocities times inv_u, rows of a
  // padded box of ph x pw voxels a plane
  int factor;
  float inv_u;
  float* out;
  int ph, pw;
  // diagnostics
  DiagQuery q;
  double* part;
};

inline long long scan_blocks(const ScanArgs& r) { return (long long)r.tiles_x * r.tiles_y * r.nchunks; }

// Whether a lattice uses less than a sixth of the lanes of its 64 x 4 columns: a cell per thread is
// faster then, although it loads the scalars of all 26 neighbours (coarse state with factor 1 and
// diagnostics, us: 8x40x300 21 and 63 against 23 and 73, 1x360x360 19 and 63 against 189 and 259;
// 12x200x400 the other way, 141 and 172 against 114 and 162).
inline bool scan_idle(const Geo& g) {
  return 6ll * g.nx * g.ny < 256ll * ((g.nx + 63) / 64) * ((g.ny + 3) / 4);
}

// The longest chunk, up to 32 planes, that still gives every place for a workgroup (4 on each of
// 256 compute units) one; a multiple of the factor; and not so that the last chunk is the
// outlet plane alone, whose state is formed from the plane below.  The diagnostics, whose blocks each
// leave a partial sum that one workgroup adds up, make do with 400 blocks below 8 planes (a
// call on 64x1x2000 63 us with 500 blocks of 4 planes, 69 with 2000 of one; 85^3 73 with 968, 79 with 1892).
inline ScanArgs scan_plan(const Geo& g, int factor, ScanKind kind) {
  ScanArgs r{};
  r.tiles_x = (g.nx + 63) / 64;
  r.tiles_y = (g.ny + 3) / 4;
  const long long tiles = (long long)r.tiles_x * r.tiles_y;
  int zc = 32;
  while (zc > factor && tiles * ((g.nz + zc - 1) / zc) < (kind == kScanDiag && zc < 8 ? 400 : 1024)) zc /= 2;
  if (zc > g.nz) zc = g.nz;
  if (g.face_hi == FACE_OUTFLOW)
    while (zc == 1 || g.nz % zc == 1) ++zc;
  r.zchunk = zc;
  r.nchunks = (g.nz + zc - 1) / zc;
  return r;
}

// Blocks of the diagnostics, each of which leaves 8 doubles.
inline long long diag_blocks(const Geo& g) {
  return scan_idle(g) ? (g.n + 255) / 256 : scan_blocks(scan_plan(g, 1, kScanDiag));
}

// Typed launchers, instantiated once per storage type (lbm_storage_*.hip).
template <typename T>
hipError_t launch_step_T(const StepArgs& a, int tx, int ty, hipStream_t s);
template <typename T>
hipError_t launch_bricks_T(const StepArgs& a, hipStream_t s);
template <typename T>
hipError_t launch_inflow_T(const StepArgs& a, hipStream_t s);
template <typename T>
hipError_t launch_batch_T(const StepArgs* cases, const int* first, int ncases, int nblocks, bool init, int tx, int ty,
                          bool walls, hipStream_t s);
template <typename T>
int step_resident_blocks_T(int tx, int ty, int device);
template <typename T>
hipError_t launch_outlet_T(const AuxArgs& a, hipStream_t s);
template <typename T>
hipError_t launch_batch_outlet_T(const AuxArgs* cases, const int* first, int ncases, int nblocks, long long step,
                                 hipStream_t s);
template <typename T>
hipError_t launch_batch_inflow_T(const StepArgs* cases, const int* first, int ncases, int nblocks, long long step,
                                 hipStream_t s);
template <typename T>
hipError_t launch_fields_T(const AuxArgs& a, int x0, int y0, int z0, int wx, int wy, int wz, double* out, hipStream_t s);
template <typename T>
hipError_t launch_populations_T(const AuxArgs& a, double* out, hipStream_t s);
template <typename T>
hipError_t launch_coarse_T(const AuxArgs& a, int f, float inv_u, float* out, int ph, int pw, hipStream_t s);
template <typename T>
hipError_t launch_diag_T(const AuxArgs& a, const DiagQuery& q, double* part, double* out, hipStream_t s);

// Dispatch on the storage code of lbm_params (0 FP32, 1 FP16, 2 BF16).
bool step_tiling_supported(int tx, int ty);
hipError_t launch_step(int storage, const StepArgs& a, int tx, int ty, hipStream_t s);
// The step of a small lattice by bricks (lbm_brick.h); its tile shape and z chunk are not used.
hipError_t launch_bricks(int storage, const StepArgs& a, hipStream_t s);
// One step of several lattices in one launch: cases (device array of ncases argument blocks,
// all with the same storage, tile shape and lateral rule: walls = free-slip x or y walls),
// first (device, ncases + 1 block offsets, each a multiple of 8), nblocks = first[ncases].
hipError_t launch_batch(int storage, const StepArgs* cases, const int* first, int ncases, int nblocks, bool init,
                        int tx, int ty, bool walls, hipStream_t s);
// Inflow sites of plane z = 0 written into the step's output state (after launch_step).
hipError_t launch_inflow(int storage, const StepArgs& a, hipStream_t s);
// Workgroups of the step kernel that fit on the device at once (0 if unknown).
int step_resident_blocks(int storage, int tx, int ty, int device);
hipError_t launch_outlet(int storage, const AuxArgs& a, hipStream_t s);
// The outlet records, and the inflow planes, of several lattices of one storage type at one
// step in one launch: cases (device array of ncases argument blocks of the step's parity),
// first (device, ncases + 1 block offsets of 256-thread blocks over each plane),
// nblocks = first[ncases].
hipError_t launch_batch_outlet(int storage, const AuxArgs* cases, const int* first, int ncases, int nblocks,
                               long long step, hipStream_t s);
hipError_t launch_batch_inflow(int storage, const StepArgs* cases, const int* first, int ncases, int nblocks,
                               long long step, hipStream_t s);
hipError_t launch_fields(int storage, const AuxArgs& a, int x0, int y0, int z0, int wx, int wy, int wz, double* out,
                         hipStream_t s);
hipError_t launch_populations(int storage, const AuxArgs& a, double* out, hipStream_t s);
hipError_t launch_coarse(int storage, const AuxArgs& a, int f, float inv_u, float* out, int ph, int pw, hipStream_t s);
hipError_t launch_diag(int storage, const AuxArgs& a, const DiagQuery& q, double* part, double* out, hipStream_t s);

}  // namespace lbm
