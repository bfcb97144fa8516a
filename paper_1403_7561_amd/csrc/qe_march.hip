// Kernels and host loop of the march (qe_march.h): Newton with backtracking
// and Jacobi-CG for one or many instances, decided on the device.
//
// A tick is two launches: the sweep (wave tiles) and the vector kernel.
//   CG:        sweep: r^T z from the vector kernel's partials, the stopping
//              decision, beta, y = J z + beta y, p = z + beta p,
//              x += alpha p of the iteration before, p^T y partials;
//              vector: alpha, r -= alpha y, z = D^-1 r, r^T z partials.
//   residual:  sweep: F at phi + lam (x + alpha p), the Jacobian's diagonal
//              and Gauss-point coefficients, |F|^2 partials; vector: the line
//              search's decision and, when the point is accepted, phi, the
//              forcing term and the next CG's start r = -F, z = D^-1 r, x = 0.
// A sweep whose CG stops evaluates the residual in the same launch, so a
// Newton step costs one tick beyond its CG iterations and no host round trip
// (driven from the host, the same step took ~110 us of read-backs, small
// launches and idle CG launches; the 65x65x33 stack's 14 steps were 1.5 of
// its 7.2 ms).  Every block re-adds the partials it needs in the same fixed
// order and takes the same decision; block 0 of an instance records it.  With
// several instances each takes its own path through the states, and a launch
// holds blocks of all of them.
#include <algorithm>

#include "qe_march.h"
#include "qe_tiles.h"

namespace qe {

#define QE_LAUNCH(kernel, grid, block, stream, ...) \
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, (hipStream_t)(stream), __VA_ARGS__)

// The point of a residual: phi, or phi + lam (x + alpha p) with the CG's x
// before its last step (p is read only when a step is pending: before that it
// holds nothing).
struct TrialMarch {
  const double* x;
  const double* p;
  double lam, alpha;
  bool step, pending;
  __device__ __forceinline__ double operator()(double v, long n) const {
    if (!step) return v;
    double d = x[n];
    if (pending) d += alpha * p[n];
    return v + lam * d;
  }
};

__device__ __forceinline__ int2 march_block(const int2* __restrict__ blk, int b, int n) {
  // chunks of 16 blocks dealt to the XCDs, as wave_of_block does
  constexpr int C = 16;
  const int full = (n / (8 * C)) * 8 * C;
  if (b < full) b = (((b >> 3) / C) * 8 + (b & 7)) * C + (b >> 3) % C;
  return blk[b];
}

// A state is recorded field by field in global memory, from the one read (a
// local copy that is modified lands in scratch memory or LDS).
__device__ __forceinline__ void march_copy(MarchState* __restrict__ n, const MarchState* __restrict__ S) { *n = *S; }

// The record of a CG solve that has ended for the reason `why`; returns
// whether the instance has finished.
__device__ __forceinline__ bool march_cg_stop(MarchState* __restrict__ n, const MarchState* __restrict__ S, int why,
                                              bool lenient) {
  const bool failed = why == PCG_NONFINITE || why == PCG_BREAKDOWN;
  n->why = why;
  n->kry = S->kry + S->iters;
  if (S->stage == MARCH_LINEAR) n->init_kry = S->iters;
  if (failed && !(lenient && S->stage == MARCH_LINEAR)) {
    n->phase = MARCH_DONE;
    n->status = why == PCG_BREAKDOWN ? QE_ERR_KRYLOV_BREAKDOWN : QE_ERR_NONFINITE;
    return true;
  }
  n->phase = MARCH_RES;
  n->step = failed ? 0 : 1;
  if (S->stage == MARCH_LINEAR) n->stage = MARCH_INITIAL;
  n->lam = 1.0;
  n->trial = 0;
  return false;
}

template <bool kOne>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_march_sweep(MarchArgs A) {
  int lb = blockIdx.x;
  MarchInst I;
  if constexpr (kOne) {
    I = A.one;
  } else {
    const int2 e = march_block(A.blk_a, blockIdx.x, A.na);
    I = A.inst[__builtin_amdgcn_readfirstlane(e.x)];
    lb = __builtin_amdgcn_readfirstlane(e.y);
  }
  // the state's fields are read once each and never changed in place: a
  // state that the decision below could write through would live in scratch
  // memory (23 instead of 8 us per launch at 65x65x33)
  const MarchState* __restrict__ const S = I.sb;
  const int phase = S->phase;
  const bool first_thread = lb == 0 && threadIdx.x == 0;
  if (phase == MARCH_DONE) {
    if (first_thread) I.sa->phase = MARCH_DONE;
    return;
  }
  __shared__ double sred[4];
  constexpr int NT = 256;
  double rz_part[8];
  const bool rz_one = I.nb <= 8 * NT;
#pragma unroll
  for (int j = 0; j < 8; ++j) rz_part[j] = I.part_b[min((int)threadIdx.x + j * NT, I.nb - 1)];
  const int wid = __builtin_amdgcn_readfirstlane((kOne ? wave_of_block(lb, I.wm) : lb) * 4 + (threadIdx.x >> 6));
  const bool active = wid < I.wm.nwaves;
  int wx, wy, wz;
  wave_tile_of(wid, I.wm, wx, wy, wz);
  const WaveTile w(I.g, wx, wy, wz, I.wm.kz, threadIdx.x & 63, active);
  double acc = 0.0, rz_new = 0.0;
  int why = PCG_RUNNING;   // the stop of the CG this launch decides
  const int iters = S->iters, stage = S->stage;
  const double alpha = S->alpha;
  bool res = phase == MARCH_RES;
  if (!res) {
    const unsigned int cb = I.cbits[64L * min(wid, I.wm.nwaves - 1) + (threadIdx.x & 63)];
    double* const sp = sred;
    const int maxit = A.krylov_maxit;
    const double* const part_b = I.part_b;
    const int nb = I.nb;
    const double rz_old = S->rz, tol2 = S->tol2;
    auto decide = [=, &why, &rz_new]() -> JvGo<double> {
      double RZ;
      if (rz_one) {
        double a = 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) a += ((int)threadIdx.x + j * NT < nb) ? rz_part[j] : 0.0;
        RZ = uniform(block_sum_all<NT>(a, sp));
      } else {
        RZ = uniform(sum_partials(part_b, nb, 1, 0, sp));
      }
      const bool first = iters == 0;
      const bool bad = !isfinite(RZ), conv = !bad && (first ? RZ == 0.0 : RZ <= tol2), maxed = iters >= maxit;
      const double beta = uniform(first ? 0.0 : RZ / rz_old), al = first ? 0.0 : alpha;
      rz_new = RZ;
      why = bad ? PCG_NONFINITE : conv ? PCG_CONVERGED : maxed ? PCG_MAXIT : PCG_RUNNING;
      return {!(bad || conv || maxed), beta, first, al};
    };
    res = !jv_tile_cg<double>(I.g, w, I.wm.kz, I.eps_t, cb, I.c, I.z, I.y, I.p, I.x, acc, decide);
  }
  // a CG that failed has no step; outside a lenient linear start it ends the solve
  const bool failed = why == PCG_NONFINITE;
  const bool dead = failed && !(A.lenient && stage == MARCH_LINEAR);
  if (res && !dead) {
    Charge ch = A.ch;
    const bool stopped = phase == MARCH_CG;
    if (stage == MARCH_LINEAR && !stopped) ch = linear_charge(ch);
    const TrialMarch tr{I.x, I.p, stopped ? 1.0 : S->lam, alpha, stopped ? !failed : S->step != 0, iters > 0};
    residual_tile<false>(I.g, w, ch, I.eps, I.semi, I.dop, I.mask, I.phi, tr, nullptr, nullptr, I.r, I.invdiag, nullptr,
                         I.c, nullptr, I.cflag, active ? I.cbits + 64L * wid + (threadIdx.x & 63) : nullptr, nullptr,
                         acc);
  }
  if (first_thread) {
    march_copy(I.sa, S);
    if (phase == MARCH_CG) {
      I.sa->rz = rz_new;
      if (iters == 0) I.sa->tol2 = S->rtol * S->rtol * rz_new;
      if (why != PCG_RUNNING) march_cg_stop(I.sa, S, why, A.lenient != 0);
    }
  }
  if (dead) return;
  const double d = wave_sum(acc);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sred[threadIdx.x >> 6] = d;
  __syncthreads();
  if (threadIdx.x == 0) I.part_a[lb] = sred[0] + sred[1] + sred[2] + sred[3];
}

// What a residual norm decides: whether phi takes the step, and what is next.
struct MarchNext {
  bool accept;
  int phase, status;   // MARCH_CG: start a solve to rtol
  double rtol;
};

// Newton's convergence test at a point with residual norm nrm, and the
// forcing term of the next CG solve (Eisenstat-Walker).
__device__ __forceinline__ MarchNext march_newton_check(bool accept, double nrm, double prev, double res0, int newton,
                                                        const MarchArgs& A) {
  if (nrm <= A.atol || nrm <= A.newton_rtol * res0) return {accept, MARCH_DONE, QE_OK, 0.0};
  if (newton >= A.newton_maxit) return {accept, MARCH_DONE, QE_ERR_NOT_CONVERGED, 0.0};
  const double q = nrm / prev;
  double eta = prev < 0.0 ? A.rtol_max : fmin(A.rtol_max, QE_EW_GAMMA * q * q);
  eta = fmax(eta, 0.5 * A.atol / nrm);
  eta = fmin(eta, A.rtol_max);
  return {accept, MARCH_CG, QE_OK, fmax(eta, 1e-13)};
}

__device__ __forceinline__ MarchNext march_next(const MarchState* __restrict__ S, double sum, double nt,
                                                const MarchArgs& A) {
  const bool fin = isfinite(nt);
  const int stage = S->stage;
  if (stage == MARCH_LINEAR) {
    if (sum > 0.0 && fin) return {false, MARCH_CG, QE_OK, QE_INIT_RTOL};
    if (!fin && !A.lenient) return {false, MARCH_DONE, QE_ERR_NONFINITE, 0.0};
    return {false, MARCH_RES, QE_OK, 0.0};   // the residual of the full problem at phi
  }
  if (stage == MARCH_INITIAL) {
    if (!fin) return {S->step != 0, MARCH_DONE, QE_ERR_NONFINITE, 0.0};
    return march_newton_check(S->step != 0, nt, -1.0, nt, 0, A);
  }
  if (fin && nt <= (1.0 - 1e-4 * S->lam) * S->nrm) return march_newton_check(true, nt, S->nrm, S->res0, S->newton + 1, A);
  if (S->trial + 1 > A.ls_max) return {false, MARCH_DONE, QE_ERR_LINESEARCH, 0.0};
  return {false, MARCH_RES, QE_OK, 0.0};     // half the step
}

// The state after that decision.
__device__ __forceinline__ void march_record(MarchState* __restrict__ n, const MarchState* __restrict__ S,
                                             const MarchNext& m, double nt) {
  const int stage = S->stage;
  if (stage != MARCH_LINEAR) n->nres = S->nres + 1;
  if (stage == MARCH_LINEAR) {
    if (m.phase == MARCH_RES) {
      n->stage = MARCH_INITIAL;
      n->step = 0;
    }
  } else if (stage == MARCH_INITIAL) {
    n->nrm = n->res0 = nt;
    if (m.status != QE_ERR_NONFINITE) n->stage = MARCH_NEWTON;
  } else if (m.accept) {
    n->nrm = nt;
    n->newton = S->newton + 1;
  } else {
    n->lam = 0.5 * S->lam;
    n->halv = S->halv + 1;
    n->trial = S->trial + 1;
  }
  n->phase = m.phase;
  n->status = m.status;
  if (m.phase == MARCH_CG) {
    n->rtol = m.rtol;
    n->iters = 0;
  }
}

// Counts an instance that has finished; the last one posts the host's word.
__device__ __forceinline__ void march_count_done(const MarchArgs& A) {
  if (atomicAdd(A.done, 1u) == (unsigned int)A.n_inst - 1u && A.prog)
    __hip_atomic_store(&A.prog->word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <bool kOne>
__global__ __launch_bounds__(kVecThreads) void k_march_vec(MarchArgs A) {
  int lb = blockIdx.x;
  MarchInst I;
  if constexpr (kOne) {
    I = A.one;
  } else {
    const int2 e = march_block(A.blk_b, blockIdx.x, A.nb);
    I = A.inst[__builtin_amdgcn_readfirstlane(e.x)];
    lb = __builtin_amdgcn_readfirstlane(e.y);
  }
  const MarchState* __restrict__ const S = I.sa;
  const int phase = S->phase;
  const bool first_thread = lb == 0 && threadIdx.x == 0;
  if (phase == MARCH_DONE) {
    // the sweep ended the solve (a launch after the end changes nothing)
    if (first_thread && I.sb->phase != MARCH_DONE) {
      march_copy(I.sb, S);
      march_count_done(A);
    }
    return;
  }
  __shared__ double sred[kVecThreads / 64];
  constexpr int NT = kVecThreads;
  double part[8];
  const bool one_pass = I.na <= 8 * NT;
#pragma unroll
  for (int j = 0; j < 8; ++j) part[j] = I.part_a[min((int)threadIdx.x + j * NT, I.na - 1)];
  const long N = I.N, nc = (N + 3) / 4, stride = (long)I.nb * NT;
  long c = (long)lb * NT + threadIdx.x;
  const bool cg = phase == MARCH_CG;
  Quad<double> qr, qy, qd;
  if (c < nc) {
    qr = ld4(I.r, c, N);
    if (cg) qy = ld4(I.y, c, N);
    qd = ld4(I.invdiag, c, N);
  }
  const double rz_old = S->rz, alpha_old = S->alpha, lam = S->lam;
  double sum;
  if (one_pass) {
    double a = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) a += ((int)threadIdx.x + j * NT < I.na) ? part[j] : 0.0;
    sum = block_sum_all<NT>(a, sred);
  } else {
    sum = sum_partials(I.part_a, I.na, 1, 0, sred);
  }
  double rz = 0.0;
  if (cg) {
    if (!(sum > 0.0) || !isfinite(sum)) {
      if (first_thread) {
        march_copy(I.sb, S);
        if (march_cg_stop(I.sb, S, PCG_BREAKDOWN, A.lenient != 0)) march_count_done(A);
      }
      return;
    }
    const double alpha = rz_old / sum;
    while (c < nc) {
      Quad<double> qz;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        qr.v[j] -= alpha * qy.v[j];
        qz.v[j] = qd.v[j] * qr.v[j];
        rz += qr.v[j] * qz.v[j];
      }
      st4(I.r, c, N, qr);
      st4(I.z, c, N, qz);
      c += stride;
      if (c < nc) {
        qr = ld4(I.r, c, N);
        qy = ld4(I.y, c, N);
        qd = ld4(I.invdiag, c, N);
      }
    }
    if (first_thread) {
      march_copy(I.sb, S);
      I.sb->alpha = alpha;
      I.sb->iters = S->iters + 1;
    }
  } else {
    const double nt = sqrt(sum);
    const MarchNext m = march_next(S, sum, nt, A);
    const bool pending = S->iters > 0, start = m.phase == MARCH_CG, accept = m.accept;
    if (accept || start) {
      while (c < nc) {
        if (accept) {
          const Quad<double> qx = ld4(I.x, c, N);
          Quad<double> qp = qx;
          if (pending) qp = ld4(I.p, c, N);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (4 * c + j < N) I.phi[4 * c + j] += lam * (pending ? qx.v[j] + alpha_old * qp.v[j] : qx.v[j]);
        }
        if (start) {
          Quad<double> qz, q0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            qr.v[j] = -qr.v[j];
            qz.v[j] = qd.v[j] * qr.v[j];
            q0.v[j] = 0.0;
            rz += qr.v[j] * qz.v[j];
          }
          st4(I.r, c, N, qr);
          st4(I.z, c, N, qz);
          st4(I.x, c, N, q0);
        }
        c += stride;
        if (c < nc) {
          qr = ld4(I.r, c, N);
          qd = ld4(I.invdiag, c, N);
        }
      }
    }
    if (first_thread) {
      march_copy(I.sb, S);
      march_record(I.sb, S, m, nt);
      if (m.phase == MARCH_DONE) march_count_done(A);
    }
  }
  const double s1 = block_sum(rz, sred);
  if (threadIdx.x == 0) I.part_b[lb] = s1;
}

// ---------------------------------------------------------------------------
// Before a march of several instances: the checks of each instance's arrays,
// with k_validate's flag bits.  (An axis's first value and the Dirichlet
// values are not checked here, as the batch never has: such an instance
// reports a residual that is not finite.)
__global__ __launch_bounds__(kVecThreads) void k_march_validate(MarchArgs A) {
  const int2 b = A.blk_b[blockIdx.x];
  const int id = __builtin_amdgcn_readfirstlane(b.x);
  const MarchInst I = A.inst[id];
  const long t0 = (long)__builtin_amdgcn_readfirstlane(b.y) * kVecThreads + threadIdx.x;
  const long stride = (long)I.nb * kVecThreads;
  int f = 0;
  for (long e = t0; e < I.E; e += stride) {
    const double v = I.eps[e];
    if (!(v > 0.0) || !isfinite(v)) f |= 1;
    if (I.dop.net && !isfinite(I.dop.net[e])) f |= 2;
    if (I.dop.donors && !(I.dop.donors[e] >= 0.0 && isfinite(I.dop.donors[e]))) f |= 2;
    if (I.dop.acceptors && !(I.dop.acceptors[e] >= 0.0 && isfinite(I.dop.acceptors[e]))) f |= 2;
  }
  for (long n = t0; n < I.N; n += stride) {
    const int d = I.dir_id[n];
    if (d < -1 || d >= I.n_dir) f |= 4;
  }
  const int n[3] = {I.g.nx, I.g.ny, I.g.nz};
  const double* co[3] = {I.g.x, I.g.y, I.g.z};
#pragma unroll
  for (int a = 0; a < 3; ++a)
    for (long i = t0 + 1; i < n[a]; i += stride) {
      const double v = co[a][i];
      if (!isfinite(v) || !(v > co[a][i - 1])) f |= 128 << a;
    }
  if (f) atomicOr(A.flags + id, f);
}

// The Dirichlet mask, phi's Dirichlet values, the tile-major permittivity,
// the z spacings and the first state of an instance whose checks found
// nothing; one with validation flags set is finished without being touched,
// and of several, those that a resident solve has finished are left as they
// are.
template <bool kOne>
__global__ __launch_bounds__(kVecThreads) void k_march_stage(MarchArgs A) {
  int lb = blockIdx.x, id = 0;
  MarchInst I;
  if constexpr (kOne) {
    I = A.one;
  } else {
    const int2 e = A.blk_b[blockIdx.x];
    id = __builtin_amdgcn_readfirstlane(e.x);
    I = A.inst[id];
    lb = __builtin_amdgcn_readfirstlane(e.y);
  }
  if (!kOne && I.sb->phase == MARCH_DONE) {
    if (lb == 0 && threadIdx.x == 0) {
      *I.sa = *I.sb;
      march_count_done(A);
    }
    return;
  }
  const bool bad = A.flags && A.flags[id] != 0;
  if (lb == 0 && threadIdx.x == 0) {
    MarchState S = {};
    S.phase = bad ? MARCH_DONE : MARCH_RES;
    S.stage = A.init;
    S.status = bad ? QE_ERR_INVALID_ARG : QE_OK;
    S.flags = bad ? A.flags[id] : 0;
    S.lam = 1.0;
    *I.sa = S;
    *I.sb = S;
    if (bad) march_count_done(A);
  }
  if (bad) return;
  const long t0 = (long)lb * kVecThreads + threadIdx.x, stride = (long)I.nb * kVecThreads;
  for (long k = t0; k < I.g.nz - 1; k += stride) {
    const double h = I.g.z[k + 1] - I.g.z[k];
    I.rdz[k] = 1.0 / h;
    I.rdz[I.g.nz - 1 + k] = h;
  }
  for (long n = t0; n < I.N; n += stride) {
    const int d = I.dir_id[n];
    I.mask[n] = d >= 0 ? 1 : 0;
    if (A.apply) {
      if (d >= 0)
        I.phi[n] = I.dir_val[d];
      else if (A.zero_free)
        I.phi[n] = 0.0;
    }
  }
  const int gx = (I.g.nx + 6) / 7, gy = (I.g.ny + 6) / 7;
  for (long sl = t0; sl < I.nslots; sl += stride) {
    const int j = (int)(sl % 49);
    const long blk = sl / 49;
    const int tx = (int)(blk % gx), ty = (int)((blk / gx) % gy), L = (int)(blk / ((long)gx * gy));
    const int ex = 7 * tx + j % 7, ey = 7 * ty + j / 7;
    double v = 0.0;
    if (ex < I.g.nx - 1 && ey < I.g.ny - 1)
      v = I.eps[(long)ex + (long)(I.g.nx - 1) * ((long)ey + (long)(I.g.ny - 1) * L)];
    I.eps_t[sl] = v;
  }
}

// After the march: electrons per box.  One partial per block and box (into z,
// free by then: nb boxes.n <= N / 64 + 16 values), then one block per instance
// adds them in a fixed order into counts[instance][box].
__global__ __launch_bounds__(kVecThreads) void k_march_count(MarchArgs A, BoxSet boxes) {
  __shared__ double sred[kVecThreads / 64];
  const int2 e = A.blk_b[blockIdx.x];
  const MarchInst I = A.inst[__builtin_amdgcn_readfirstlane(e.x)];
  const int lb = __builtin_amdgcn_readfirstlane(e.y);
  const long ex = I.g.nx - 1, ey = I.g.ny - 1;
  double acc[kMaxBoxes];
#pragma unroll
  for (int r = 0; r < kMaxBoxes; ++r) acc[r] = 0.0;
  for (long el = (long)lb * kVecThreads + threadIdx.x; el < I.E; el += (long)I.nb * kVecThreads) {
    if (!I.semi[el]) continue;
    const int i = (int)(el % ex), j = (int)((el / ex) % ey), k = (int)(el / (ex * ey));
    const double xc = 0.5 * (I.g.x[i] + I.g.x[i + 1]), yc = 0.5 * (I.g.y[j] + I.g.y[j + 1]),
                 zc = 0.5 * (I.g.z[k] + I.g.z[k + 1]);
    bool any = false;
    for (int r = 0; r < boxes.n; ++r) any |= boxes.b[r].contains(xc, yc, zc);
    if (!any) continue;
    const long n0 = (long)i + (long)I.g.nx * ((long)j + (long)I.g.ny * k);
    const long sy = I.g.nx, sz = (long)I.g.nx * I.g.ny;
    double ve[8] = {I.phi[n0], I.phi[n0 + 1], I.phi[n0 + sy], I.phi[n0 + sy + 1],
                    I.phi[n0 + sz], I.phi[n0 + sz + 1], I.phi[n0 + sz + sy], I.phi[n0 + sz + sy + 1]};
    gauss_interp(ve);
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) s += electron_density_only(A.ch, ve[q]);
    s *= (I.g.x[i + 1] - I.g.x[i]) * (I.g.y[j + 1] - I.g.y[j]) * (I.g.z[k + 1] - I.g.z[k]) * 0.125;
#pragma unroll
    for (int r = 0; r < kMaxBoxes; ++r)
      if (r < boxes.n && boxes.b[r].contains(xc, yc, zc)) acc[r] += s;
  }
#pragma unroll
  for (int r = 0; r < kMaxBoxes; ++r)
    if (r < boxes.n) {
      const double s = block_sum(acc[r], sred);
      if (threadIdx.x == 0) I.z[(long)lb * boxes.n + r] = s;
    }
}

__global__ __launch_bounds__(64) void k_march_count_sum(MarchArgs A, int n_boxes, double* __restrict__ counts) {
  const MarchInst I = A.inst[blockIdx.x];
  if ((int)threadIdx.x >= n_boxes) return;
  double s = 0.0;
  for (int b = 0; b < I.nb; ++b) s += I.z[(long)b * n_boxes + threadIdx.x];
  counts[(long)blockIdx.x * n_boxes + threadIdx.x] = s;
}

// ------------------------------------------------------------ host side
// Blocks of the vector kernel: the CG's, one 4-entry chunk per thread.
int march_blocks_b(long N) { return cg_blocks(N); }

void launch_march_validate(hipStream_t s, const MarchArgs& a) {
  QE_LAUNCH(k_march_validate, a.nb, kVecThreads, s, a);
}

void launch_march_stage(hipStream_t s, const MarchArgs& a) {
  if (a.n_inst == 1 && !a.inst)
    QE_LAUNCH(k_march_stage<true>, a.nb, kVecThreads, s, a);
  else
    QE_LAUNCH(k_march_stage<false>, a.nb, kVecThreads, s, a);
}

void launch_march_tick(hipStream_t s, const MarchArgs& a) {
  if (a.n_inst == 1 && !a.inst) {
    QE_LAUNCH(k_march_sweep<true>, a.na, 256, s, a);
    QE_LAUNCH(k_march_vec<true>, a.nb, kVecThreads, s, a);
  } else {
    QE_LAUNCH(k_march_sweep<false>, a.na, 256, s, a);
    QE_LAUNCH(k_march_vec<false>, a.nb, kVecThreads, s, a);
  }
}

void launch_march_count(hipStream_t s, const MarchArgs& a, const BoxSet& boxes, double* counts) {
  QE_LAUNCH(k_march_count, a.nb, kVecThreads, s, a, boxes);
  QE_LAUNCH(k_march_count_sum, a.n_inst, 64, s, a, boxes.n, counts);
}

}  // namespace qe
