// Newton-CG with the mesh resident on the chip: one workgroup per box of
// nodes, every vector and coefficient in registers and LDS, and a barrier
// among the workgroups of an instance as the only wait.  For meshes of up to
// a few hundred thousand nodes; see qe_resident.hip.
#pragma once

#include "qe_march.h"

namespace qe {

constexpr int kResThreads = 512;     // threads of a workgroup, which has a compute unit to itself
constexpr int kResElemSlots = 3;     // elements of a box per thread, at most
constexpr int kResMaxWgs = 256;      // workgroups of one launch, at most (one per compute unit)

constexpr int kResCopies = 8;        // copies of the published sums

// How a mesh is cut: g boxes of t nodes along each axis (the last shorter).
struct ResPlan {
  int gx, gy, gz, tx, ty, tz;
  int nwg;
  float cost;   // us per CG iteration, by resident_plan's model
};
// The cut into at most max_wgs boxes that fit a workgroup with the shortest CG
// iteration or, where instances share the chip, the least workgroup time per
// iteration; false if there is none.
bool resident_plan(int nx, int ny, int nz, int max_wgs, bool share, ResPlan& p);
// Whether resident solves are taken (the QE_RESIDENT knob).
bool resident_on();
// The QE_RESIDENT_POLLS knob (0: the kernel's own limits).
int resident_polls();
// Workgroups that the current device holds at once, at most kResMaxWgs.
int resident_wgs();

struct ResInst {
  int nx, ny, nz, n_dir;
  const double *x, *y, *z;
  const double* eps;
  const uint8_t* semi;
  Doping dop;
  const int32_t* dir_id;
  const double* dir_val;
  double* phi;
  double* keep;             // [N] receives phi as it is before the solve; NULL: not needed
  // what neighbouring boxes read: two words per value, [2 N] each, in this
  // order one after the other
  unsigned long long *w0, *w1, *d;
  unsigned long long* part; // every box's sums, then the second buffer of d (resident_fit)
  ResPlan plan;
  const int* flags;         // validation flags (nonzero: not run), or NULL
  MarchState* out;          // written once, when the instance has finished
};

struct ResArgs {
  ResInst one;               // inst = NULL: the instance itself
  const ResInst* inst;
  int n_inst;
  const int2* seats;         // (instance, box) of every ticket, an instance's boxes in a row
  int n_seats;
  unsigned int* ticket;      // the next ticket; zeroed by the launch, like started and abort
  unsigned int* started;     // workgroups that have a compute unit
  unsigned long long* abort; // set when a wait ran out
  Charge ch;
  Quantum qm;                // eigenstates (one instance; n = 0: none)
  double atol, rtol_max, newton_rtol;
  int newton_maxit, ls_max, krylov_maxit;
  int lenient, init, apply, zero_free;
  int polls_first, polls_later;   // of one wait (set by the launch): while workgroups have not started; at all
};

// A launch wants every compute unit, and two that each had some would keep each
// other waiting, so of the calls of this process one at a time runs resident on
// a device: from the construction, which waits for its turn, until release or
// the end.  The wait is bounded (the holder's stream may be waiting for the
// caller's); a call that did not get its turn marches.
class ResidentTurn {
  int dev_ = -1;

 public:
  explicit ResidentTurn(bool wanted);
  ~ResidentTurn() { release(); }
  ResidentTurn(const ResidentTurn&) = delete;
  ResidentTurn& operator=(const ResidentTurn&) = delete;
  bool held() const { return dev_ >= 0; }
  void release();
};

// How the solves of this thread's last call went, in their order (a coarse start
// before the solve that it starts; a batch's instances), for the tests:
// qe_last_routes copies up to n of them and returns their number.
enum SolveRoute : uint8_t { ROUTE_OTHER = 0, ROUTE_RESIDENT = 1, ROUTE_LEFT = 2 };   // LEFT: tried resident, solved otherwise
void clear_routes();
void add_route(SolveRoute r);

// Boxes whose part fits `bytes`, at most wgs.
int resident_fit(size_t bytes, long nodes, int wgs);
// Zeroes the exchange buffers, then solves on at most wgs workgroups (a single
// instance: its plan's); plans: of every instance (nwg 0: not in this launch).
qe_status launch_resident(hipStream_t s, ResArgs a, const ResPlan* plans, int n_plans, int wgs);

}  // namespace qe
