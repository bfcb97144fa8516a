// The Newton-CG iteration as a device-side state machine ("march"): every
// instance advances by ticks of two launches whose kernels read what to do
// next from the instance's state, so the host takes no decision of a solve.
// One instance (small meshes of qe_solve) or many (qe_solve_batch) march in
// the same launches.
#pragma once

#include <vector>

#include "qe_runtime.h"

namespace qe {

enum MarchPhase : int { MARCH_RES = 0, MARCH_CG = 1, MARCH_DONE = 2 };
// LINEAR: the charge-free problem of the initial guess; INITIAL: the residual
// at the initial guess; NEWTON: the Newton steps.
enum MarchStage : int { MARCH_LINEAR = 0, MARCH_INITIAL = 1, MARCH_NEWTON = 2 };

// One instance's state between launches.  The two kernels of a tick each
// read the copy the other wrote and write their own, so no block of a launch
// can read what another block of it writes.
struct MarchState {
  int phase, stage;
  int status;      // qe_status once DONE
  int why;         // PcgStatus of the last CG
  int flags;       // validation flags of an instance that was not run
  int step;        // x + alpha p (x alone before the first iteration) is the current CG solution
  int iters;       // iterations of the current CG solve
  int newton, trial, kry, init_kry, halv, nres;
  int resident;    // 1: finished by the resident solve
  double rz, alpha, tol2, rtol, lam, nrm, res0;
};

// One instance's problem and work arrays.
struct MarchInst {
  Geom g;
  WaveMap wm;
  const double* eps;
  const uint8_t* semi;
  Doping dop;
  const int32_t* dir_id;
  const double* dir_val;
  double* phi;
  // r holds F while a residual is evaluated; c, eps_t, cflag tile-major
  double *x, *r, *z, *p, *y, *invdiag, *c, *eps_t, *rdz;
  uint8_t *mask, *cflag;
  unsigned int* cbits;
  double *part_a, *part_b;     // partials of the sweep (na) and of the vector kernel (nb)
  MarchState *sa, *sb;         // written by the sweep, by the vector kernel
  long N, E, nslots;
  int na, nb, n_dir;
};

struct MarchArgs {
  MarchInst one;               // n_inst = 1: the instance itself
  int n_inst;
  const MarchInst* inst;       // n_inst > 1: device arrays, and the (instance, block) of every block
  const int2 *blk_a, *blk_b;
  int na, nb;                  // blocks of the two kernels over all instances
  Charge ch;
  double atol, rtol_max, newton_rtol;
  int newton_maxit, ls_max, krylov_maxit;
  int lenient;                 // a failed CG of the initial guess is skipped, not an error
  int init;                    // the stage to start from
  int apply, zero_free;        // staging of phi (k_stage's)
  int* flags;                  // validation flags (nonzero: nothing is run); one per instance
  unsigned int* done;          // instances that have finished
  CgProgress* prog;            // host-coherent word posted when all have or NULL
};

int march_blocks_b(long N);
// The checks of every instance into flags[instance] (several instances).
void launch_march_validate(hipStream_t s, const MarchArgs& a);
void launch_march_stage(hipStream_t s, const MarchArgs& a);
void launch_march_tick(hipStream_t s, const MarchArgs& a);
void launch_march_count(hipStream_t s, const MarchArgs& a, const BoxSet& boxes, double* counts);
// Queues ticks until every instance has finished.
// ring: kEventRing events created on first use (not touched without hm->prog_dev).
qe_status march_run(hipStream_t s, MarchArgs& a, HostMirror& hm, hipEvent_t* ring, int ahead);

}  // namespace qe
