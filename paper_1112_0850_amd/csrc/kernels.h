// kernels.h -- launch interface between the C ABI glue and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "pair_plan.h"

namespace lbm {

// Launch geometry shared by every per-cell kernel.  A wavefront owns a
// 64-cell segment of one x-row; a 256-thread block owns 4 consecutive
// segments in (z, y, segment) order.  Blocks are remapped so that each of
// the 8 XCDs (which receive hardware block ids round-robin) works on one
// contiguous eighth of the domain, keeping neighbouring rows in one L2.
//
// Kernels receive Geo and no more than it.  With the fields that only the host
// reads ahead of yb and upw a wave waited for two more scalar loads before its
// first pull (graph replays, us a step: FP32 48^3 channel 6.23, now 6.01; 40^3
// 4.35, now 4.19), and a launch cost more host time (bursts of 40 steps, us a
// step: FP16 40^3 4.90 with 320 bytes of arguments, 4.09 with these 304).
struct Geo {
  int32_t nx, ny, nz;
  int32_t xs;       // x stride of a population row, in cells
  uint32_t plane;   // elements from one direction array to the next (nz * ny * xs + padding)
  int32_t nseg;     // 64-cell segments per row
  int32_t nrows;    // ny * nz
  int32_t upw;      // step kernel: the most 64-cell units of a row that a segment holds
  int32_t nb8;      // blocks launched, rounded down to a multiple of 8
  int32_t yb;       // step kernel: rows are visited in bands of yb rows of y, z fastest
};
static_assert(sizeof(Geo) == 40, "Geo grew: see above");

// The same with what the launchers need.
struct Plan : Geo {
  int32_t nblocks;  // blocks launched (4 segments each)
  int32_t xfill;    // columns of a row that a single step stores: nx, or more (zeros past nx)
  bool stream;      // non-temporal stores in the single step (see cached_stores),
  bool stream2;     //   and in the pair pass and the adjoint
  PairPlan pairs;   // the two-step pass (of the context's storage)
};

// Launch geometry of the two-step kernel: 64 x TY tiles in (x, y), z chunks.
struct Geo2 {
  int32_t nx, ny, nz;
  int32_t xs;      // x stride of a population row, in cells
  uint32_t plane;  // elements from one direction array to the next
  int32_t ntx, nty, zc, nblocks, nb8;
};

// Launch geometry of the two-step kernel on small boxes: 3-D tiles.
struct GeoT {
  int32_t nx, ny, nz;
  int32_t xs;      // x stride of a population row, in cells
  uint32_t plane;  // elements from one direction array to the next
  int32_t tx, ty, tz;
  int32_t ntx, nty, nblocks, nb8;
};

constexpr int kBlock = 256;
constexpr int kReduceBlocks = 1024;

struct PhysParams {
  double omega;      // 1 / tau (0 for tau = +inf)
  double F[3];       // body-force density
  double scale;      // FP16 storage scale 2^s (1 otherwise)
  double wall_u[3];  // velocity of the moving-wall cells
  bool moving;       // wall_u != 0 and the grid has flags: moving-wall markers are in use
  bool incomp;       // He-Luo incompressible equilibrium (u = j + F/2)
  bool split;        // bounce-back by the separate obstacle kernel (the paper's split design)
};

// Whether a row's 64-cell units nearly fill waves of four: the 16-bit step kernels
// then run four units per lane everywhere, some past the row end, instead of each
// wave's own count.  The branch to the count costs them 3 to 8% (FP16 1 x 329 x 960
// spheres, 15 units, 9.5 us against 10.3; 8 x 346 x 1472, 23 units, 68.8 against
// 71.1), the idle units of shorter rows more (300^3, 5 units, 540 against 456).
inline bool step_fours(int nx) {
  const int units = (nx + 63) / 64;
  return 5 * units >= 4 * ((units + 3) / 4 * 4);
}

Plan make_plan(int nx, int ny, int nz, int xs, uint64_t dir_stride);

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);
hipError_t launch_init(int storage, const Plan& g, const PhysParams& ph, void* grid,
                       const uint8_t* flags, const float* rho0, const float* u0, hipStream_t s);
hipError_t launch_mark_solids(int storage, const Plan& g, const PhysParams& ph, void* grid,
                              const uint8_t* flags, hipStream_t s);
hipError_t launch_step(int storage, bool solids, bool force, const Plan& g, const PhysParams& ph,
                       const void* src, void* dst, const uint8_t* flags, hipStream_t s);
// Two fused steps src = f*(t) -> dst = f*(t+2) (bit-identical to two launch_step calls;
// not for the split design).
// lmask: the link mask of launch_link_mask, or NULL (the walls then use the
// markers).
hipError_t launch_step2(int storage, bool solids, bool force, const Plan& g, const PhysParams& ph,
                        const void* src, void* dst, const uint8_t* flags, const uint32_t* lmask,
                        hipStream_t s);
// The same two steps storing the intermediate level too: mid = f*(t+1)
// (FP32 storage only: hipErrorInvalidValue otherwise).
hipError_t launch_step2_mid(int storage, bool solids, bool force, const Plan& g,
                            const PhysParams& ph, const void* src, void* mid, void* dst,
                            const uint8_t* flags, const uint32_t* lmask, hipStream_t s);
// One or two FP32 steps (not for the split design) that also store the moments
// of the pre-collision states: four arrays in the grid layout per state.  A
// null dst stores the moments only.
hipError_t launch_step_mom(bool solids, bool force, const Plan& g, const PhysParams& ph,
                           const float* src, float* dst, float* mom, const uint8_t* flags,
                           hipStream_t s);
hipError_t launch_step2_mom(bool solids, bool force, const Plan& g, const PhysParams& ph,
                            const float* src, float* dst, float* mom1, float* mom2,
                            const uint8_t* flags, const uint32_t* lmask, hipStream_t s);
// The two-step kernel's link mask of every cell ([nz][ny][nx] uint32) from the
// flags: bit i (1..18) for a blocked pull along c_i, bits 19 and 20 for the
// cell's own SOLID and NOFORCE flags; with moving walls bit 21 for a link to a
// moving wall and bit 22 for a moving-wall cell.
hipError_t launch_link_mask(const Plan& g, bool moving, const uint8_t* flags, uint32_t* mask,
                            hipStream_t s);
hipError_t launch_obstacle(int storage, const Plan& g, const PhysParams& ph, void* grid,
                           const uint8_t* flags, hipStream_t s);
hipError_t launch_macro(int storage, bool out_f64, const Plan& g, const PhysParams& ph,
                        const void* grid, const uint8_t* flags, void* rho, void* u, hipStream_t s);
hipError_t launch_reduce(int storage, const Plan& g, const PhysParams& ph, const void* grid,
                         const uint8_t* flags, double* scratch, double* out5, hipStream_t s);
// Discrete adjoint in pull form (nu = dL/df, the pre-collision adjoint):
// seed nu^T from dL/drho_T, dL/du_T and f*(T-1); step nu^{n+1} -> nu^n with
// f*(n-1); init dL/du0 from nu^1.
hipError_t launch_adj_seed(bool solids, const Plan& g, const PhysParams& ph, const float* fprev,
                           const uint8_t* flags, const float* dL_drho, const float* dL_du,
                           float* nu_T, double* partials, hipStream_t s);
hipError_t launch_adj_step(bool solids, const Plan& g, const PhysParams& ph, const float* fprev,
                           const uint8_t* flags, const float* nu_np1, float* nu_n,
                           double* partials, hipStream_t s);
// The seed (nu1 null) or one reverse step from stored moments.
hipError_t launch_adj_mom(bool solids, const Plan& g, const PhysParams& ph, const float* mom,
                          const uint8_t* flags, const float* dL_drho, const float* dL_du,
                          const float* nu1, float* nu0, double* partials, hipStream_t s);
// Two reverse steps from stored moments; lmask NULL when there are no solids.
bool adj_pair_fits(const Plan& g);
hipError_t launch_adj_pair(const Plan& g, const PhysParams& ph, const float* mom1, const float* mom2,
                           const float* nu2, float* nu0, const uint32_t* lmask, double* partials,
                           hipStream_t s);
hipError_t launch_adj_init(bool solids, const Plan& g, const PhysParams& ph, const uint8_t* flags,
                           const float* nu1, const float* rho0, const float* u0, float* dL_du0,
                           hipStream_t s);
hipError_t launch_adj_finish(const Plan& g, const double* partials, double* out3, hipStream_t s);
hipError_t launch_copy(void* c, const void* a, size_t n16, hipStream_t s);
// Copy variants for the bandwidth sweep: vec in {1, 2, 4} 16-byte elements per
// thread, non-temporal or not, `blocks` blocks (0 = one pass over the array).
hipError_t launch_copy_variant(void* c, const void* a, size_t n16, int vec, bool nt, size_t blocks,
                               hipStream_t s);
// Pull-copy probe: one pure-streaming pass dst_i(x) = src_i(x - c_i) (periodic,
// no geometry, no collision) with the step kernel's launch and access pattern.
hipError_t launch_pull_copy(int storage, const Plan& g, const void* src, void* dst, hipStream_t s);

}  // namespace lbm
