// Host-side launch interface between the C ABI and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mhd_device.hpp"

namespace mhd {

// Kernel identities for the optional per-kernel event timing.
enum KernelId : int { K_FACES = 0, K_EMF, K_UPDATE, K_CFL, K_CFL_FINAL, K_ADJ, K_PRIM, K_COUNT };

// Records a pair of HIP events around each launch on the launch stream.
struct Timer {
  virtual void begin(int kid, hipStream_t s) = 0;
  virtual void end(int kid, hipStream_t s) = 0;
  virtual ~Timer() = default;
};

// One RK stage (or the bare right-hand side).
struct StageArgs {
  int dim, limiter, riemann, precision;
  int emf;                // 0: upwind average with the HLL bounds; 1: UCT-HLLD
  bool glm;               // GLM divergence cleaning: nine cell-centred fields, no CT
  double glm_dmin;        // GLM: the smallest cell spacing (c_h = cfl dmin / dt)
  double glm_decay;       // GLM: damping factor of psi per step, exp(-alpha cfl)
  int stage;              // 0: out = L(U); 1: out = U + dt L; 2: out = (U0 + U + dt L)/2;
                          // 3: face/edge records only; SSP-RK3 stages 2 and 3:
                          // 4: out = (3 U0 + (U + dt L))/4; 5: out = (U0 + 2 (U + dt L))/3
  Geom g;
  const double* U;        // state the right-hand side is evaluated at
  const double* U0;       // stage 2: state at the start of the step
  double* out;
  double* FW;             // face records: dim * NSLOT * n doubles
  double* EW;             // edge EMFs: 3 * n doubles
  double* PW;             // 3D WENO-Z only: primitives of every cell, 8 (GLM: 9) * n doubles
  double dt;
  const double* dtp;      // device dt (nullptr: use dt)
  int* flag;              // sticky unphysical flag
  hipStream_t stream;
  Timer* timer;           // nullable
  // stage 1 only, optional: dt is the CFL bound of U, whose partials go to
  // cfl_partial (stage_cfl_blocks doubles in 3D, kInlineCfl2d in 2D); *dt_out =
  // cfl * min is written before anything reads dtp (which then must be dt_out)
  double* cfl_partial;
  double cfl;
  double* dt_out;
  // 3D with CT only: L(U) is left besides, of the five cell-averaged fields in FW
  // (n doubles each from its start, space no edge input uses), of the staggered
  // ones in EW
  bool keep_rhs;
  // 2D only: the stage's face records and E_z in FW and EW (the adjoint
  // reads them)
  bool records;
  // 2D only, optional: the stage also leaves the CFL partials of the state
  // it writes (stage_2d_tiles doubles; out must differ from U and U0), and a
  // first stage takes its dt from ncfl such partials in cfl_prev instead of
  // from a pass over U
  double* cfl_next;
  const double* cfl_prev;
  int ncfl;
};

// Column tiles in x, y and runs of lz planes along z.
struct MarchGrid {
  int ntx, nty, nzc, lz;
  unsigned nblocks;
};

struct CflArgs {
  int dim;
  bool glm;               // GLM: nine cell-centred fields
  Geom g;
  const double* U;
  double* partial;        // nblocks doubles
  int nblocks;
  double cfl;
  double* dt_out;         // device double
  int* flag;
  hipStream_t stream;
  Timer* timer;           // nullable
};

#define MHD_TIMED(args, kid, ...)                              \
  do {                                                         \
    if ((args).timer) (args).timer->begin((kid), (args).stream); \
    __VA_ARGS__;                                               \
    if ((args).timer) (args).timer->end((kid), (args).stream);   \
  } while (0)

hipError_t launch_stage(const StageArgs& a);
// number of CFL partials of a 3D stage (WENO-Z: one per block of the primitive
// kernel, else of a grid-stride pass)
size_t stage_cfl_blocks(const Geom& g, int limiter, bool glm);
constexpr size_t kCfl3d = 2048;
// 3D: on grids of at most this many workgroups of the face kernel each reduces the
// partials itself, if there are at most kCfl3d.
constexpr unsigned kInlineCfl3d = 1024;
// the CFL time step of U
hipError_t launch_cfl(const CflArgs& a);
// 3D face kernel (stage 3: edge inputs only; cflp: npart CFL partials, or null:
// a.dtp or a.dt), and with CT the EMFs and the update of the staggered field.
MarchGrid march_grid(const Geom& g, int limiter, double* turns = nullptr);
void launch_faces_march(const StageArgs& a, const double* cflp, int npart);
// The same cell by cell, from the primitives (dt: a.dtp or a.dt), and on which grids.
void launch_faces_cells(const StageArgs& a);
bool faces_by_cells(const Geom& g, int limiter, bool glm);
void launch_ct(const StageArgs& a);
// 2D stage in one kernel; cflp: npart CFL partials (null: a.dtp or a.dt).
void launch_stage_2d(const StageArgs& a, const double* cflp, int npart);
int stage_2d_tiles(const Geom& g, int limiter, int emf, int precision, bool glm);
// Grids of at most this many 32 x 8 tiles take 8 x 8 ones.
constexpr int64_t kSmallTiles2d = 256;
// 2D: most CFL partials that every workgroup of the stage reduces itself.
constexpr int kInlineCfl2d = 1024;
// Partials of the allocation-free CFL time step (a file-scope device array of
// that many doubles plus the flag; nblocks must not exceed it).
constexpr int kNoAllocPartials = 2048;
// The CFL time step with the partials and the flag in that array (a.partial
// and a.flag are ignored); flag_out (device int32, nullable) receives 1 if
// any cell was unphysical in this call, else 0.
hipError_t launch_cfl_noalloc(const CflArgs& a, int32_t* flag_out);

}  // namespace mhd
