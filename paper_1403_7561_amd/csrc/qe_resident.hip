// The resident solve: Newton with backtracking and Jacobi-CG in one launch.
//
// A mesh is cut into boxes of tx x ty x tz nodes, one workgroup each, at most
// one workgroup per compute unit.  A workgroup keeps its box with a one-node
// halo for the whole solve: a thread holds up to two of its nodes (neighbours
// in z) and two of the halo (phi, x, r, s, p, D^-1) and, for its own nodes, the
// 27 entries of the assembled Jacobian row, all in registers; the vector a
// product is applied to goes through LDS.  So a CG iteration moves no vector
// and no coefficient through memory; what it costs is the wait for the other
// workgroups.
//
// One wait per iteration: CG in the form with a single reduction (Chronopoulos
// and Gear, 1989: r^T u and u^T J u together, J p by recurrence), and the
// updates of r, s, p and x repeated on the halo, whose only missing value,
// w = J u, the neighbouring boxes publish together with the sums.
//
// Exchange between workgroups: a published double is two 64-bit words, each
// half of it with the number of the exchange, written and read with relaxed
// atomic accesses at agent scope, which reach the memory that all XCDs share.
// A reader polls the word it needs until the number is there, so a value's
// arrival is its own signal: no counter, no fence, no second round trip.
// (Measured with counters instead, waiting for the stores, counting arrivals
// and then reading: 2.0 us per exchange for 8 workgroups, 3.7 us for 256; with
// release fences at agent scope, which write back an XCD's whole L2, 9.8 us.)
// Buffers alternate by the exchange's parity: a workgroup publishes into a
// buffer again only after it has the sums of the exchange in between, which
// every reader of the buffer sent after reading it.
//
// Several instances: a free workgroup takes the next ticket, and the tickets
// run through the instances' boxes one instance after another.  An instance
// runs once all its tickets are taken; the workgroups of those that run take
// the tickets that are missing when they finish, so there is always one that
// can run, whatever the boxes' numbers.
//
// Waiting: an instance needs all its workgroups at once.  A launch has at most
// one per compute unit, so on a device without other work they all run (this
// process's launches take turns: ResidentTurn); when other work keeps some out
// for too long, every wait ends after a bounded number of polls, much fewer
// while some have not started; then the workgroups leave, the instance's state
// says that it is not finished, and the host takes the tick-by-tick march
// instead, from the caller's phi: workgroups that had the last exchange in time
// have written their part by then, so a warm start is kept and put back.
//
// Measured, whole solves, with the host-driven launches of one kernel per CG
// step / the march / resident: 17x17x9 3.2 / 2.5 / 0.85 ms, a junction of
// 33x29x41 11.7 / 10.7 / 3.4, 65x65x33 7.4 / 6.4 / 3.3; 256 instances of 33x33x17
// to 65x65x33 in one call 505 / 251 / 245.  A CG iteration at 65x65x33 in 169
// boxes takes ~6 us: product and updates 1.9, sums of the workgroup 0.9,
// publishing 0.5, waiting 2.6, sums of all 0.5.
#include <algorithm>
#include <chrono>
#include <mutex>
#include <vector>

#include "qe_resident.h"
#include "qe_tiles.h"

namespace qe {

// Polls of one wait (each a round trip to memory, ~0.5 us or more): an
// instance's first while some workgroups of the launch still have no compute
// unit, and any.  (With all of them running, the first wait of one of several
// instances may last as long as other instances' solves.)  QE_RESIDENT_POLLS
// sets both (tests of the fallback).
constexpr int kResPollsFirst = 20000, kResPollsLater = 2000000;

// MarchState::phase of an instance that is not finished: one of its workgroups
// gave up, or all of them left it to the march
constexpr int kResGaveUp = -1;

typedef unsigned long long res_word;

__device__ __forceinline__ res_word agent_load(const res_word* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned int agent_load(const unsigned int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(res_word* p, res_word v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Word pairs are addressed by a uniform base and a 32-bit byte offset per lane.
__device__ __forceinline__ res_word* res_at(res_word* base, unsigned int bytes) {
  return reinterpret_cast<res_word*>(reinterpret_cast<char*>(base) + bytes);
}
__device__ __forceinline__ void publish(res_word* base, unsigned int bytes, double v, unsigned int tag) {
  const res_word b = (res_word)__double_as_longlong(v);
  agent_store(res_at(base, bytes), (b << 32) | tag);
  agent_store(res_at(base, bytes) + 1, (b & 0xffffffff00000000ull) | tag);
}
__device__ __forceinline__ double published(res_word lo, res_word hi) {
  return __longlong_as_double((long long)((hi & 0xffffffff00000000ull) | (lo >> 32)));
}

// Sum over the wave, the same in every lane (fixed order; DPP row shifts and
// broadcasts, which cost no trip through LDS as shuffles do).
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, kRows, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRows, 0xf, false);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_total(double v) {
  v = dpp_add<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: lane 15 of each row holds its sum
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);   // row_bcast15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);   // row_bcast31 into rows 2 and 3
  return lane_value(v, 63);
}

// rho and drho/dphi at one Gauss point.  Not inlined: the polynomial
// constants of its exponentials and logarithms would be held in registers
// through the whole solve, and eight copies of it do not fit the instruction
// cache.
struct ResCharge {
  double rho, drho;
};
__device__ __attribute__((noinline)) ResCharge res_charge(const Charge* ch, double phi, double net, double nd,
                                                           double na) {
  ResCharge q;
  space_charge(*ch, phi, net, nd, na, q.rho, q.drho);
  return q;
}

// The same for given electrons.
__device__ __attribute__((noinline)) ResCharge res_charge_n(const Charge* ch, double phi, double n, double dn,
                                                             double net, double nd, double na) {
  ResCharge q;
  space_charge_n(*ch, phi, n, dn, net, nd, na, q.rho, q.drho);
  return q;
}

// kQ: electrons from eigenstates (one instance), summed per element like the
// wave-tiled residual's (pc_states).  65x65x33 nodes with 16 states: 406 CG
// iterations and 12 residuals in 4.1 ms, against 8.4 with host-driven launches.
template <bool kOne, bool kQ>
__global__ __launch_bounds__(kResThreads) void k_resident(ResArgs A) {
  extern __shared__ double lds[];
  constexpr int NT = kResThreads, ES = kResElemSlots, kResWaves = NT / 64;
  __shared__ double sred_own[2 * kResWaves], sred_all[2 * kResWaves];
  __shared__ int s_dead;
  __shared__ Charge s_ch;
  __shared__ Quantum s_qm;
  // kQ: the order in which the elements are dealt to the threads, those in a
  // state's support box first, so that few waves run the loop over the states
  // (in the mesh's order every wave of a box that holds a dot does)
  __shared__ unsigned short s_order[kQ ? kResElemSlots * kResThreads : 1];
  __shared__ int s_ticket;
  const int t = threadIdx.x, wave = t >> 6;
  unsigned int epoch = 0;   // exchanges of the instance so far; their tags are 1, 2, ...
  // The abort word is read by one thread for the workgroup: another workgroup
  // may set it at any time, and waves that read it apart could part ways.
  if (t == 0) {
    s_dead = agent_load(A.abort) != 0u ? 1 : 0;
    __hip_atomic_fetch_add(A.started, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_ch = A.ch;
    if constexpr (kQ) s_qm = A.qm;
  }
  __syncthreads();
  if (s_dead) return;

  // After a poll: whether the wave's wait is over (everything `here`, or the
  // wait ran out and s_dead is set); k counts the polls.
  auto waited = [&](bool here, int& k) -> bool {
    if (__builtin_amdgcn_ballot_w64(!here) == 0) return true;
    ++k;
    if (k >= A.polls_later ||
        ((k & 255) == 255 &&
         (agent_load(A.abort) != 0u || (epoch <= 1u && k >= A.polls_first && agent_load(A.started) < gridDim.x)))) {
      agent_store(A.abort, 1u);
      s_dead = 1;
      return true;
    }
    if (k > 64) __builtin_amdgcn_s_sleep(16);   // a long wait: leave the memory to those that work
    return false;
  };

  for (int turn = 0;; ++turn) {
    // the next box
    ResInst I;
    int wg = blockIdx.x;
    if constexpr (kOne) {
      if (turn > 0) return;
      I = A.one;
    } else {
      __syncthreads();
      if (t == 0)   // (after an abort none is taken)
        s_ticket = agent_load(A.abort) != 0u
                       ? A.n_seats
                       : (int)__hip_atomic_fetch_add(A.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      const int k = __builtin_amdgcn_readfirstlane(s_ticket);
      if (k >= A.n_seats) return;
      const int2 seat = A.seats[k];
      I = A.inst[__builtin_amdgcn_readfirstlane(seat.x)];
      wg = __builtin_amdgcn_readfirstlane(seat.y);
      epoch = 0;
    }
    if (I.flags && *I.flags != 0) {
      if (wg == 0 && t == 0) {
        MarchState S = {};
        S.phase = MARCH_DONE;
        S.status = QE_ERR_INVALID_ARG;
        S.flags = *I.flags;
        *I.out = S;
      }
      return;   // (one instance: several are checked before they are launched)
    }
    const ResPlan P = I.plan;
    const int nwg = P.nwg;
    const int nx = I.nx, ny = I.ny, nz = I.nz;
    const int ex = P.tx + 2, ey = P.ty + 2, exy = ex * ey;
    const int fx = P.tx + 1, fy = P.ty + 1, fxy = fx * fy, nel = fxy * (P.tz + 1);
    const int planes = 2 * ((P.tz + 1) / 2) + 2;
    double* const su = lds;                       // [planes * exy] a vector on the box and its halo
    double* const so = su + planes * exy;         // [8][nel] element values, or [27][NT] matrix rows
    double* const se = so + max(8 * nel, 27 * NT);   // [nel] permittivity, 0 outside the mesh
    double* const sh = se + nel;                  // spacings (hx, hy, hz) and their inverses
    // then [nel] bytes: the element has nonzero coefficients
    const int bx = wg % P.gx, by = (wg / P.gx) % P.gy, bz = wg / (P.gx * P.gy);
    const int i0 = bx * P.tx - 1, j0 = by * P.ty - 1, k0 = bz * P.tz - 1;   // the halo's first node

    // this thread's nodes: 0 and 1 its own (neighbours in z), 2 and 3 of the halo
    enum { IN = 1, FACE = 2, FREE = 4 };
    unsigned int nid[4];   // byte offset of the node's word pair (16 bytes a node)
    int nfl[4], un[4];
    double phi[4], x[4], r[4], s[4], p[4], dinv[4];
    int e0_;   // the element whose last corner is node 0
    {
      const int a = t % P.tx + 1, b = (t / P.tx) % P.ty + 1, c = 2 * (t / (P.tx * P.ty)) + 1;
      e0_ = (a - 1) + fx * (b - 1) + fxy * (c - 1);
      const int per = 2 * ex + 2 * P.ty, nh = 2 * exy + per * P.tz;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        int na = a, nb = b, nc = c + q;
        bool ok = true;
        if (q < 2) {
          ok = nc <= P.tz;
        } else {
          int h = t + NT * (q - 2);
          ok = h < nh;
          if (h < 2 * exy) {
            nc = h < exy ? 0 : P.tz + 1;
            h = h < exy ? h : h - exy;
            na = h % ex;
            nb = h / ex;
          } else {
            h -= 2 * exy;
            nc = 1 + h / per;
            h -= (nc - 1) * per;
            if (h < 2 * ex) {
              nb = h < ex ? 0 : P.ty + 1;
              na = h < ex ? h : h - ex;
            } else {
              h -= 2 * ex;
              na = h < P.ty ? 0 : P.tx + 1;
              nb = 1 + (h < P.ty ? h : h - P.ty);
            }
          }
        }
        un[q] = ok ? na + ex * nb + exy * nc : 0;
        const int i = i0 + na, j = j0 + nb, k = k0 + nc;
        nid[q] = 0;
        nfl[q] = ok ? 8 : 0;   // bit 8: the thread writes su[un]
        phi[q] = x[q] = r[q] = s[q] = p[q] = dinv[q] = 0.0;
        if (ok && i >= 0 && i < nx && j >= 0 && j < ny && k >= 0 && k < nz) {
          const int n = i + nx * (j + ny * k);
          nid[q] = 16u * (unsigned int)n;
          int f = 8 | IN;
          if (q < 2 && (na == 1 || na == P.tx || nb == 1 || nb == P.ty || nc == 1 || nc == P.tz)) f |= FACE;
          const int d = I.dir_id[n];
          if (d < 0) f |= FREE;
          if (d >= 0 && A.apply)
            phi[q] = I.dir_val[d];
          else if (!(A.apply && A.zero_free))
            phi[q] = I.phi[n];
          nfl[q] = f;
        }
      }
      // spacings along the axes (1 outside the mesh) and the elements' eps
      for (int m = t; m < fx + fy + P.tz + 1; m += NT) {
        const double* co = m < fx ? I.x : m < fx + fy ? I.y : I.z;
        const int g = m < fx ? i0 + m : m < fx + fy ? j0 + (m - fx) : k0 + (m - fx - fy);
        const int n = m < fx ? nx : m < fx + fy ? ny : nz;
        const double h = (g >= 0 && g < n - 1) ? co[g + 1] - co[g] : 1.0;
        sh[m] = h;
        sh[fx + fy + P.tz + 1 + m] = 1.0 / h;
      }
      for (int e = t; e < nel; e += NT) {
        const int i = i0 + e % fx, j = j0 + (e / fx) % fy, k = k0 + e / fxy;
        se[e] = (i >= 0 && i < nx - 1 && j >= 0 && j < ny - 1 && k >= 0 && k < nz - 1)
                    ? I.eps[(long)i + (long)(nx - 1) * ((long)j + (long)(ny - 1) * k)]
                    : 0.0;
      }
    }
    if constexpr (kQ) {
      __syncthreads();   // s_qm
      unsigned char* const near = reinterpret_cast<unsigned char*>(sh + 2 * (fx + fy + P.tz + 1));
      for (int e = t; e < nel; e += NT) {
        const int i = i0 + e % fx, j = j0 + (e / fx) % fy, k = k0 + e / fxy;
        bool in = false;
        for (int m = 0; m < s_qm.n; ++m) {
          const int* b = s_qm.sbox + 6 * m;
          in = in || (i + 1 >= b[0] && i <= b[1] && j + 1 >= b[2] && j <= b[3] && k + 1 >= b[4] && k <= b[5]);
        }
        near[e] = in ? 1 : 0;
      }
      __syncthreads();
      if (wave == 0) {   // (in a fixed order: which elements share a wave may change their last bits)
        int first = 0, last = nel;
        for (int e0 = 0; e0 < nel; e0 += 64) {
          const int e = e0 + t;
          const bool in = e < nel && near[e] != 0, out = e < nel && near[e] == 0;
          const unsigned long long bi = __builtin_amdgcn_ballot_w64(in), bo = __builtin_amdgcn_ballot_w64(out);
          const unsigned long long before = (1ull << t) - 1;
          if (in) s_order[first + __popcll(bi & before)] = (unsigned short)e;
          if (out) s_order[last - 1 - __popcll(bo & before)] = (unsigned short)e;
          first += __popcll(bi);
          last -= __popcll(bo);
        }
      }
      __syncthreads();
    }
    // the assembled Jacobian's rows of this thread's own nodes: the second in
    // registers, the first in LDS where the element values were (both in
    // registers leave too few for the rest: the compiler spills a row to
    // memory and the product takes 6 instead of 1 us)
    double J1[27];

    // Publishes the workgroup's sums of (a, b) and waits for everybody's;
    // `mine` publishes the thread's own values, `theirs` polls the halo's.
    // false: a wait ran out (uniform).
    auto exchange = [&](double& a, double& b, auto mine, auto theirs) -> bool {
      ++epoch;
      mine();
      a = wave_total(a);
      b = wave_total(b);
      if ((t & 63) == 0) {
        sred_own[wave] = a;
        sred_own[kResWaves + wave] = b;
      }
      __syncthreads();
      // [2][kResCopies][nwg][4]: every workgroup publishes its sums once per
      // copy and reads one copy, so that no line is polled by all of them
      res_word* const pb = I.part + (long)(epoch & 1u) * 4 * kResCopies * nwg;
      if (wave == 0) {
        double ta = 0.0, tb = 0.0;
#pragma unroll
        for (int w = 0; w < kResWaves; ++w) {
          ta += sred_own[w];
          tb += sred_own[kResWaves + w];
        }
        // lanes (copy, sum)
        if (t < 2 * kResCopies)
          publish(pb, 32u * (unsigned int)(nwg * (t >> 1) + wg) + 16u * (t & 1), (t & 1) ? tb : ta, epoch);
      }
      a = b = 0.0;
      for (int k = 0;;) {
        bool here = theirs();
        if (t < nwg) {
          const res_word* const q = res_at(pb, 32u * (unsigned int)(nwg * (wg & (kResCopies - 1)) + t));
          const res_word w0 = agent_load(q), w1 = agent_load(q + 1), w2 = agent_load(q + 2), w3 = agent_load(q + 3);
          here = here && (unsigned int)w0 == epoch && (unsigned int)w1 == epoch && (unsigned int)w2 == epoch &&
                 (unsigned int)w3 == epoch;
          a = published(w0, w1);
          b = published(w2, w3);
        }
        if (waited(here, k)) break;
      }
      a = wave_total(a);
      b = wave_total(b);
      if ((t & 63) == 0) {
        sred_all[wave] = a;
        sred_all[kResWaves + wave] = b;
      }
      __syncthreads();
      a = b = 0.0;
#pragma unroll
      for (int w = 0; w < kResWaves; ++w) {
        a += sred_all[w];
        b += sred_all[kResWaves + w];
      }
      return s_dead == 0;
    };
    auto wbuf = [&](unsigned int e) { return (e & 1u) ? I.w1 : I.w0; };
    // A workgroup that gives up says so in the state, whether or not another
    // has finished the instance in the meantime (it may have seen the last
    // exchange in time): the state of an instance with a part missing is
    // never MARCH_DONE.
    auto give_up = [&]() {
      if (t == 0) __hip_atomic_exchange(&I.out->phase, kResGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    // |F|^2 at phi + lam x (has_x): r = F and D^-1 on the box and its halo,
    // the Jacobian's rows of the box there.  false: a wait ran out.
    auto residual = [&](bool linear, bool has_x, double lam, double& n2) -> bool {
      // Copies that the compiler cannot see through: the element indices and
      // addresses below are formed here, where they are used, instead of once
      // before the Newton loop, where holding them pushes the Jacobian's rows
      // out of the registers.
      int t = threadIdx.x, e0 = e0_, fx = P.tx + 1, fxy = fx * (P.ty + 1), ex = P.tx + 2, exy = ex * (P.ty + 2);
      asm volatile("" : "+v"(t), "+v"(e0));
      asm volatile("" : "+s"(fx), "+s"(fxy), "+s"(ex), "+s"(exy));
      const int fy = P.ty + 1, nel = fxy * (P.tz + 1), hinv = fx + fy + P.tz + 1;
      double* const so = su + planes * exy;
      double* const se = so + max(8 * nel, 27 * NT);
      double* const sh = se + nel;
      unsigned char* const sf = reinterpret_cast<unsigned char*>(sh + 2 * hinv);
      auto weights = [&](int a, int b, int c, double e, double& sx, double& sy, double& sz) {
        const double hx = sh[a], hy = sh[fx + b], hz = sh[fx + fy + c];
        sx = e * (hy * sh[hinv + a] * hz);
        sy = e * (hx * sh[hinv + fx + b] * hz);
        sz = e * (hx * hy * sh[hinv + fx + fy + c]);
      };
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (nfl[q]) su[un[q]] = has_x ? phi[q] + lam * x[q] : phi[q];
      __syncthreads();
      // kQ: the thread's nodes go to memory for the loop over the states, which
      // needs their registers; left to itself the compiler spills them through
      // the CG as well (65x65x33, 16 states: 3.3 instead of 1.6 us of work per iteration)
      volatile double parked[kQ ? 16 : 1];
      volatile unsigned int parked_id[kQ ? 12 : 1];
      if constexpr (kQ)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          parked[q] = phi[q];
          parked[4 + q] = x[q];
          parked[8 + q] = r[q];
          parked[12 + q] = dinv[q];
          parked_id[q] = nid[q];
          parked_id[4 + q] = (unsigned int)nfl[q];
          parked_id[8 + q] = (unsigned int)un[q];
        }
      double c8[ES][8];
#pragma unroll
      for (int q = 0; q < ES; ++q)
#pragma unroll
        for (int m = 0; m < 8; ++m) c8[q][m] = 0.0;
#pragma unroll 1
      for (int q = 0; q < ES; ++q) {
        int e = t + NT * q;
        if (e >= nel) break;
        if constexpr (kQ) e = s_order[e];
        double out[8], cc[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) out[m] = cc[m] = 0.0;
        const double ee = se[e];
        bool nonzero = false;
        if (ee != 0.0) {
          const int a = e % fx, b = (e / fx) % fy, c = e / fxy;
          double sx, sy, sz, ve[8];
          weights(a, b, c, ee, sx, sy, sz);
          const int u = a + ex * b + exy * c;
          ve[0] = su[u];
          ve[1] = su[u + 1];
          ve[2] = su[u + ex];
          ve[3] = su[u + ex + 1];
          ve[4] = su[u + exy];
          ve[5] = su[u + exy + 1];
          ve[6] = su[u + exy + ex];
          ve[7] = su[u + exy + ex + 1];
          jv_element(ve, sx, sy, sz, cc, false, out);
          const long el = (long)(i0 + a) + (long)(nx - 1) * ((long)(j0 + b) + (long)(ny - 1) * (k0 + c));
          if (I.semi[el]) {
            const double kw = A.ch.kappa * (sh[a] * sh[fx + b]) * sh[fx + fy + c] * 0.125;
            double net = 0.0, ndo = 0.0, nac = 0.0;
            if (A.ch.incomplete && !linear) {
              ndo = I.dop.donors[el];
              nac = I.dop.acceptors[el];
            } else if (I.dop.net) {
              net = I.dop.net[el];
            } else if (I.dop.donors) {
              net = I.dop.donors[el] - I.dop.acceptors[el];
            }
            gauss_interp(ve);
            bool states = false;   // electrons from the eigenstates
            double nq[8], dnq[8];
            if constexpr (kQ) {
              states = !s_qm.region || s_qm.region[el];
              if (states) {
#pragma unroll
                for (int m = 0; m < 8; ++m) nq[m] = dnq[m] = 0.0;
                // states whose support box holds the element of some lane; in
                // the other lanes all their |psi_i|^2 are exactly 0
                const int gi = i0 + a, gj = j0 + b, gk = k0 + c;
                unsigned int act = 0;
                for (int i = 0; i < s_qm.n; ++i) {
                  const int* bx = s_qm.sbox + 6 * i;
                  const bool in = gi + 1 >= bx[0] && gi <= bx[1] && gj + 1 >= bx[2] && gj <= bx[3] && gk + 1 >= bx[4] &&
                                  gk <= bx[5];
                  if (__builtin_amdgcn_ballot_w64(in)) act |= 1u << i;
                }
                if (act) {
                  const long n0 = (long)gi + (long)nx * ((long)gj + (long)ny * gk), sxy = (long)nx * ny;
                  auto corners = [&](const double* __restrict__ v, double o[8]) {
                    o[0] = v[0];
                    o[1] = v[1];
                    o[2] = v[nx];
                    o[3] = v[nx + 1];
                    o[4] = v[sxy];
                    o[5] = v[sxy + 1];
                    o[6] = v[sxy + nx];
                    o[7] = v[sxy + nx + 1];
                  };
                  double u8[8];
                  corners(s_qm.phik + n0, u8);
                  pc_states(s_qm, act, ve, u8,
                            [&](int i, double s2[8]) { corners(s_qm.psi2 + s_qm.N * i + n0, s2); }, nq, dnq);
                }
              }
            }
#pragma unroll
            for (int m = 0; m < 8; ++m) {
              ResCharge q{net, 0.0};   // the initial guess: doping alone, and the states' electrons
              if (kQ && states && linear)
                q = ResCharge{net - nq[m], -dnq[m]};
              else if (kQ && states)
                q = res_charge_n(&s_ch, ve[m], nq[m], dnq[m], net, ndo, nac);
              else if (!linear)
                q = res_charge(&s_ch, ve[m], net, ndo, nac);
              ve[m] = kw * q.rho;
              cc[m] = -kw * q.drho;
              nonzero |= cc[m] != 0.0;
            }
            gauss_interp(ve);
#pragma unroll
            for (int m = 0; m < 8; ++m) out[m] -= ve[m];
          }
        }
        sf[e] = nonzero ? 1 : 0;
#pragma unroll
        for (int m = 0; m < 8; ++m) so[m * nel + e] = out[m];
#pragma unroll
        for (int v = 0; v < ES; ++v)
          if (q == v)
#pragma unroll
            for (int m = 0; m < 8; ++m) c8[v][m] = cc[m];
      }
      if constexpr (kQ)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          phi[q] = parked[q];
          x[q] = parked[4 + q];
          r[q] = parked[8 + q];
          dinv[q] = parked[12 + q];
          nid[q] = parked_id[q];
          nfl[q] = (int)parked_id[4 + q];
          un[q] = (int)parked_id[8 + q];
        }
      __syncthreads();
      double acc = 0.0, zero = 0.0;
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (nfl[q] & IN) {
          const int e = e0 + q * fxy;   // eight elements in a fixed order
          double v = so[7 * nel + e];
          v += so[6 * nel + e + 1];
          v += so[5 * nel + e + fx];
          v += so[4 * nel + e + fx + 1];
          v += so[3 * nel + e + fxy];
          v += so[2 * nel + e + fxy + 1];
          v += so[1 * nel + e + fxy + fx];
          v += so[0 * nel + e + fxy + fx + 1];
          r[q] = (nfl[q] & FREE) ? v : 0.0;
          acc += r[q] * r[q];
        }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < ES; ++q) {
        int e = t + NT * q;
        if (e < nel) {
          if constexpr (kQ) e = s_order[e];
#pragma unroll
          for (int m = 0; m < 8; ++m) so[m * nel + e] = c8[q][m];
        }
      }
      __syncthreads();
      // row of node q: each of its eight elements gives the entries between
      // the node's local corner and the element's eight corners
      auto assemble = [&](int q, double* __restrict__ J) {
#pragma unroll
        for (int m = 0; m < 27; ++m) J[m] = 0.0;
        if (!(nfl[q] & FREE)) return;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
          constexpr double k18 = 1.0 / 18.0;
          const int da = d & 1, db = (d >> 1) & 1, dc = d >> 2;   // element offset; the node is its corner (1-da, 1-db, 1-dc)
          const int e = e0 + q * fxy + da + fx * db + fxy * dc;
          const int a = e % fx, b = (e / fx) % fy, c = e / fxy;
          const double ee = se[e];
          double sx, sy, sz, v[8];
          weights(a, b, c, ee, sx, sy, sz);
#pragma unroll
          for (int m = 0; m < 8; ++m) v[m] = 0.0;
          if (sf[e]) {
#pragma unroll
            for (int m = 0; m < 8; ++m) {
              // weight of the node's corner at Gauss point m
              const double wq = ((m & 1) == 1 - da ? kG1 : kG0) * (((m >> 1) & 1) == 1 - db ? kG1 : kG0) *
                                ((m >> 2) == 1 - dc ? kG1 : kG0);
              v[m] = wq * so[m * nel + e];
            }
            gauss_interp(v);
          }
#pragma unroll
          for (int m = 0; m < 8; ++m) {
            const int ox = da + (m & 1) - 1, oy = db + ((m >> 1) & 1) - 1, oz = dc + (m >> 2) - 1;
            // 1/36 of (1 | -1 along the weight's axis) (4 | 2 | 1 over the others)
            const double mx = ox == 0 ? 2.0 : 1.0, my = oy == 0 ? 2.0 : 1.0, mz = oz == 0 ? 2.0 : 1.0;
            const double kx = (ox == 0 ? 0.5 : -0.5) * my * mz * k18, ky = (oy == 0 ? 0.5 : -0.5) * mx * mz * k18,
                         kz = (oz == 0 ? 0.5 : -0.5) * mx * my * k18;
            double& j = J[(ox + 1) + 3 * (oy + 1) + 9 * (oz + 1)];
            j += sx * kx + sy * ky + sz * kz + v[m];
            // added here, not with the other elements' at the end, which would
            // keep all 64 terms in registers until then
            asm volatile("" : "+v"(j));
          }
        }
      };
      assemble(1, J1);
      {
        double J0[27];
        assemble(0, J0);
        dinv[0] = J0[13] > 0.0 ? 1.0 / J0[13] : 0.0;
        dinv[1] = J1[13] > 0.0 ? 1.0 / J1[13] : 0.0;
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 27; ++m) so[m * NT + t] = J0[m];
      }
      res_word* const wb = wbuf(epoch + 1u);
      // (by the exchange's parity like w: two residuals may follow each other)
      res_word* const db = ((epoch + 1u) & 1u) ? I.d : I.part + (size_t)nwg * 8 * kResCopies;
      const bool ok = exchange(
          acc, zero,
          [&]() {
#pragma unroll
            for (int q = 0; q < 2; ++q)
              if (nfl[q] & FACE) {
                publish(wb, nid[q], r[q], epoch);
                publish(db, nid[q], dinv[q], epoch);
              }
          },
          [&]() {
            bool here = true;
#pragma unroll
            for (int q = 2; q < 4; ++q)
              if (nfl[q] & IN) {
                const res_word *fp = res_at(wb, nid[q]), *dp = res_at(db, nid[q]);
                const res_word f0 = agent_load(fp), f1 = agent_load(fp + 1), d0 = agent_load(dp), d1 = agent_load(dp + 1);
                here = here && (unsigned int)f0 == epoch && (unsigned int)f1 == epoch && (unsigned int)d0 == epoch &&
                       (unsigned int)d1 == epoch;
                r[q] = published(f0, f1);
                dinv[q] = published(d0, d1);
              }
            return here;
          });
      n2 = acc;
      return ok;
    };

    // CG on J x = -F from x = 0 after residual() at the linearisation point.
    // Returns the reason it stopped, or -1 when a wait ran out.
    int iters = 0;
    auto cg = [&](double rtol) -> int {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        r[q] = -r[q];
        x[q] = p[q] = s[q] = 0.0;
        if (nfl[q]) su[un[q]] = dinv[q] * r[q];
      }
      double gam_old = 1.0, alpha = 1.0, tol2 = 0.0;
      for (iters = 0;; ++iters) {
        __syncthreads();
        double w[4] = {0.0, 0.0, 0.0, 0.0}, gam = 0.0, del = 0.0;
        if (nfl[0]) {
          // (row addresses formed here: see residual)
          int rx = ex, rxy = exy;
          asm volatile("" : "+s"(rx), "+s"(rxy));
          const double* const u0 = su + (un[0] - rxy - rx - 1);
          const double* const j0 = so + t;
#pragma unroll
          for (int l = 0; l < 4; ++l) {
            double v[9], c[9];
#pragma unroll
            for (int m = 0; m < 9; ++m) {
              v[m] = u0[l * rxy + (m / 3) * rx + m % 3];
              if (l < 3) c[m] = j0[(9 * l + m) * NT];
            }
#pragma unroll
            for (int m = 0; m < 9; ++m) {
              if (l < 3) w[0] += c[m] * v[m];
              if (l > 0) w[1] += J1[9 * (l - 1) + m] * v[m];
            }
          }
          // an absent or Dirichlet node's row is zero, but the plane above
          // the box may hold anything
          if (!(nfl[1] & FREE)) w[1] = 0.0;
          const double a = dinv[0] * r[0], b = dinv[1] * r[1];
          gam = r[0] * a + r[1] * b;
          del = w[0] * a + w[1] * b;
        }
        res_word* const wb = wbuf(epoch + 1u);
        const bool ok = exchange(
            gam, del,
            [&]() {
#pragma unroll
              for (int q = 0; q < 2; ++q)
                if (nfl[q] & FACE) publish(wb, nid[q], w[q], epoch);
            },
            [&]() {
              bool here = true;
#pragma unroll
              for (int q = 2; q < 4; ++q)
                if (nfl[q] & IN) {
                  const res_word* fp = res_at(wb, nid[q]);
                  const res_word f0 = agent_load(fp), f1 = agent_load(fp + 1);
                  here = here && (unsigned int)f0 == epoch && (unsigned int)f1 == epoch;
                  w[q] = published(f0, f1);
                }
              return here;
            });
        if (!ok) return -1;
        if (!isfinite(gam)) return PCG_NONFINITE;
        if (iters == 0) {
          if (gam == 0.0) return PCG_CONVERGED;
          tol2 = rtol * rtol * gam;
        } else if (gam <= tol2) {
          return PCG_CONVERGED;
        }
        if (iters >= A.krylov_maxit) return PCG_MAXIT;
        const double beta = iters == 0 ? 0.0 : gam / gam_old;
        const double pap = iters == 0 ? del : del - beta * gam / alpha;   // p^T J p
        if (!(pap > 0.0) || !isfinite(pap)) return PCG_BREAKDOWN;
        alpha = gam / pap;
        gam_old = gam;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          p[q] = dinv[q] * r[q] + beta * p[q];
          s[q] = w[q] + beta * s[q];
          x[q] += alpha * p[q];
          r[q] -= alpha * s[q];
          if (nfl[q]) su[un[q]] = dinv[q] * r[q];
        }
      }
    };

    // Newton, with the decisions of march_next: a residual, then the line
    // search's or the convergence test's verdict, then a CG solve
    int status = QE_OK, why = PCG_RUNNING, stage = A.init, newton = 0, kry = 0, init_kry = 0, halv = 0, nres = 0;
    int trial = 0;
    double nrm = 0.0, res0 = 0.0, prev = -1.0, lam = 1.0;
    bool step = false;
    // This form of the CG takes p^T J p and J p from recurrences, which lose
    // digits to cancellation where the direct form does not.  A CG that breaks
    // down and a line search that fails are therefore not the last word: the
    // instance is left unfinished, and the march solves it from its start.
    bool handed = false;
    for (;;) {
      double n2;
      if (!residual(stage == MARCH_LINEAR, step, lam, n2)) {
        give_up();
        return;
      }
      const double nt = sqrt(n2);
      const bool fin = isfinite(nt);
      double rtol;
      if (stage == MARCH_LINEAR) {
        if (!(n2 > 0.0 && fin)) {
          if (!fin && !A.lenient) {
            status = QE_ERR_NONFINITE;
            break;
          }
          stage = MARCH_INITIAL;   // the residual of the full problem at phi
          continue;
        }
        rtol = QE_INIT_RTOL;
      } else {
        ++nres;
        const bool accept = stage == MARCH_INITIAL || (fin && nt <= (1.0 - 1e-4 * lam) * nrm);
        if (!accept) {
          lam *= 0.5;
          ++halv;
          if (++trial <= A.ls_max) continue;
          handed = true;
          break;
        }
        if (step)
#pragma unroll
          for (int q = 0; q < 4; ++q) phi[q] += lam * x[q];
        if (stage == MARCH_INITIAL) {
          res0 = nt;
        } else {
          prev = nrm;
          ++newton;
        }
        nrm = nt;
        if (!fin) {
          status = QE_ERR_NONFINITE;
          break;
        }
        stage = MARCH_NEWTON;
        if (nrm <= A.atol || nrm <= A.newton_rtol * res0) break;
        if (newton >= A.newton_maxit) {
          status = QE_ERR_NOT_CONVERGED;
          break;
        }
        const double qn = nrm / prev;
        rtol = prev < 0.0 ? A.rtol_max : fmin(A.rtol_max, QE_EW_GAMMA * qn * qn);
        rtol = fmax(rtol, 0.5 * A.atol / nrm);
        rtol = fmin(rtol, A.rtol_max);
        rtol = fmax(rtol, 1e-13);
      }
      why = cg(rtol);
      if (why < 0) {
        give_up();
        return;
      }
      kry += iters;
      if (stage == MARCH_LINEAR) init_kry = iters;
      handed = why == PCG_BREAKDOWN || why == PCG_NONFINITE;
      if (handed) break;
      step = true;
      if (stage == MARCH_LINEAR) stage = MARCH_INITIAL;
      lam = 1.0;
      trial = 0;
    }
    if (handed) {   // (every workgroup alike: the sums are the same in all)
      give_up();
      __syncthreads();
      continue;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (nfl[q] & IN) I.phi[nid[q] >> 4] = phi[q];
    if (wg == 0 && t == 0) {
      // (field by field: the others may have set the phase)
      MarchState* const S = I.out;
      S->stage = stage;
      S->status = status;
      S->why = why;
      S->flags = 0;
      S->newton = newton;
      S->kry = kry;
      S->init_kry = init_kry;
      S->halv = halv;
      S->nres = nres;
      S->resident = 1;
      S->nrm = nrm;
      S->res0 = res0;
      int expected = MARCH_RES;
      __hip_atomic_compare_exchange_strong(&S->phase, &expected, (int)MARCH_DONE, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------ host side
int resident_wgs() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  return std::min(cus, kResMaxWgs);
}

constexpr int kMaxRoutes = 4096;
static thread_local uint8_t t_routes[kMaxRoutes];
static thread_local int t_n_routes = 0;
void clear_routes() { t_n_routes = 0; }
void add_route(SolveRoute r) {
  if (t_n_routes < kMaxRoutes) t_routes[t_n_routes++] = r;
}

// As long as several single solves; a launch's first wait is no shorter.
constexpr std::chrono::milliseconds kResTurn(20);
constexpr int kResDevices = 64;
static std::timed_mutex& resident_mutex(int dev) {
  static std::timed_mutex m[kResDevices];
  return m[dev];
}
ResidentTurn::ResidentTurn(bool wanted) {
  int dev = -1;
  if (wanted && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kResDevices &&
      resident_mutex(dev).try_lock_for(kResTurn))
    dev_ = dev;
}
void ResidentTurn::release() {
  if (dev_ >= 0) resident_mutex(dev_).unlock();
  dev_ = -1;
}

static size_t resident_lds(const ResPlan& p) {
  const size_t nel = (size_t)(p.tx + 1) * (p.ty + 1) * (p.tz + 1);
  const size_t planes = 2 * ((p.tz + 1) / 2) + 2;
  return sizeof(double) * (planes * (p.tx + 2) * (p.ty + 2) + std::max(8 * nel, (size_t)27 * kResThreads) + nel +
                           2 * (p.tx + p.ty + p.tz + 3)) + ((nel + 7) & ~size_t(7));
}

// The cuts of one axis: g boxes of t nodes, every t once.
struct ResCut {
  int g, t;
};
static std::vector<ResCut> res_cuts(int n, int most) {
  std::vector<ResCut> c;
  for (int g = 1; g <= std::min(n, most); ++g) {
    const int t = (n + g - 1) / g;
    if ((n + t - 1) / t == g) c.push_back({g, t});
  }
  return c;
}

// The cost of a CG iteration in us, fitted to measurements over 17x17x9 (8 to
// 32 boxes), 33x29x41 (63 to 150) and 65x65x33 (150 to 245) nodes: the
// exchange grows with the workgroups (their sums are read by all) and the
// halo, the rest with the box's node pairs.  4.0 us for 17x17x9 in 32 boxes,
// 4.4 us for 33x29x41 in 126, 7.0 us for 65x65x33 in 180.
bool resident_plan(int nx, int ny, int nz, int max_wgs, bool share, ResPlan& best) {
  double cost = 1e300;
  const std::vector<ResCut> cx = res_cuts(nx, max_wgs), cy = res_cuts(ny, max_wgs), cz = res_cuts(nz, max_wgs);
  for (const ResCut& a : cx)
    for (const ResCut& b : cy) {
      if (a.g * b.g > max_wgs) break;
      for (const ResCut& d : cz) {
        const int nwg = a.g * b.g * d.g;
        if (nwg > max_wgs) break;
        const long pairs = (long)a.t * b.t * ((d.t + 1) / 2), el = (long)(a.t + 1) * (b.t + 1) * (d.t + 1);
        const long halo = (long)(a.t + 2) * (b.t + 2) * (d.t + 2) - (long)a.t * b.t * d.t;
        if (pairs > kResThreads || halo > 2 * kResThreads || el > (long)kResElemSlots * kResThreads) continue;
        const double c = 3.1 + 0.004 * nwg + 2e-5 * nwg * nwg + 0.0036 * pairs + (halo > kResThreads ? 0.5 : 0.0);
        const double v = share ? c * nwg : c;
        if (v < cost) {
          cost = v;
          best = ResPlan{a.g, b.g, d.g, a.t, b.t, d.t, nwg, (float)c};
        }
      }
    }
  return cost < 1e300;
}

// An instance's part: the published sums of every box, then the second buffer
// of D^-1 (2 words a node).
static size_t res_part_bytes(int nwg, long nodes) {
  return ((size_t)nwg * 8 * kResCopies + 2 * (size_t)nodes) * sizeof(res_word);
}
int resident_fit(size_t bytes, long nodes, int wgs) {
  const size_t box = res_part_bytes(1, 0), rest = 2 * (size_t)nodes * sizeof(res_word);
  return bytes < rest ? 0 : (int)std::min<size_t>(wgs, (bytes - rest) / box);
}

// Zeroes the buffers between the boxes of every instance (w0, w1 and d are
// six vectors that follow each other; then the part) and the launch's
// counters, sets the state's phase, and keeps phi where that is asked for.
__global__ __launch_bounds__(256) void k_resident_zero(ResArgs A) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    *A.ticket = 0u;
    *A.started = 0u;
    *A.abort = 0ull;
  }
  for (int k = blockIdx.y; k < A.n_inst; k += gridDim.y) {
    const ResInst I = A.inst ? A.inst[k] : A.one;
    if (I.plan.nwg == 0) continue;
    if (blockIdx.x == 0 && threadIdx.x == 0) I.out->phase = MARCH_RES;
    const long n = (long)I.nx * I.ny * I.nz, t0 = (long)blockIdx.x * 256 + threadIdx.x, stride = (long)gridDim.x * 256;
    ulonglong2* const p = reinterpret_cast<ulonglong2*>(I.w0);
    const long words = reinterpret_cast<ulonglong2*>(I.d) - p + n;
    for (long i = t0; i < words; i += stride) p[i] = make_ulonglong2(0, 0);
    if (I.keep)
      for (long i = t0; i < n; i += stride) I.keep[i] = I.phi[i];
    ulonglong2* const q = reinterpret_cast<ulonglong2*>(I.part);
    for (long i = t0; i < (long)I.plan.nwg * 4 * kResCopies + n; i += stride) q[i] = make_ulonglong2(0, 0);
  }
}

template <bool kOne, bool kQ>
static qe_status resident_launch(hipStream_t s, const ResArgs& a, int grid, size_t lds) {
  const void* fn = reinterpret_cast<const void*>(k_resident<kOne, kQ>);
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return fail(QE_ERR_HIP, "resident solve: %zu bytes of LDS refused", lds);
  hipLaunchKernelGGL((k_resident<kOne, kQ>), dim3(grid), dim3(kResThreads), lds, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(QE_ERR_HIP, "resident solve launch failed: %s", hipGetErrorString(e));
  return QE_OK;
}

qe_status launch_resident(hipStream_t s, ResArgs a, const ResPlan* plans, int n_plans, int wgs) {
  size_t lds = 0;
  for (int i = 0; i < n_plans; ++i)
    if (plans[i].nwg > 0) lds = std::max(lds, resident_lds(plans[i]));
  const int polls = resident_polls();
  a.polls_first = polls > 0 ? polls : kResPollsFirst;
  a.polls_later = polls > 0 ? polls : kResPollsLater;
  const int gy = std::min(a.n_inst, 32768);
  hipLaunchKernelGGL(k_resident_zero, dim3(std::max(1, std::min(256, 4096 / a.n_inst)), gy), dim3(256), 0, s, a);
  if (a.inst) return resident_launch<false, false>(s, a, std::min(wgs, a.n_seats), lds);
  return a.qm.n > 0 ? resident_launch<true, true>(s, a, a.one.plan.nwg, lds)
                    : resident_launch<true, false>(s, a, a.one.plan.nwg, lds);
}

}  // namespace qe

extern "C" int qe_last_routes(uint8_t* out, int n) {
  for (int i = 0; i < std::min(n, qe::t_n_routes); ++i) out[i] = qe::t_routes[i];
  return qe::t_n_routes;
}
