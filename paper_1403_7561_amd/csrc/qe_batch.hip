// Batched solve of many independent devices (a gate-voltage sweep over
// uneven meshes).  Instances that fit are solved resident on the chip
// (qe_resident.h), as many at a time as their boxes fit the compute units.
// The others, and any that its workgroups left unfinished, march
// together (qe_march.h): every launch advances all of them, so their number
// bounds nothing but the traffic.
//
// The host checks the instances, lays out the workspace, cuts the meshes,
// picks the march's chunk height (recorded in the tune cache) and queues the
// launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <map>
#include <numeric>
#include <sstream>
#include <string>
#include <vector>

#include "qe_resident.h"

namespace qe {

static size_t al256(size_t v) { return (v + 255) & ~size_t(255); }

// Chunk heights of the wave tiles, as make_wavemap's: the tallest that still
// gives kMinWaves waves over all instances.
static const int kMinKz = 3, kMaxKz9 = 9;
static const long kMinWaves = 2048;

static size_t inst_bytes(const qe_problem& p) {
  const long N = (long)p.nx * p.ny * p.nz;
  const long S = tile_slots(p.nx, p.ny, p.nz);
  const long tiles = make_wavemap(p.nx, p.ny, p.nz, kMinKz).nwaves;
  return 6 * al256(N * 8) + al256(S * 64) + al256(S * 8) + al256(S) + al256(N) + al256(2 * (p.nz - 1) * 8) +
         al256(tiles * 64 * 4) + al256((tiles + 3) / 4 * 8) + al256(march_blocks_b(N) * 8);
}

// Per-instance results, read back in one copy.
struct BatchHead {
  size_t inst, res, seats, blk_a, blk_b, state_a, state_b, counts, flags, done, total;
};

static BatchHead batch_head(int n, const qe_problem* probs) {
  BatchHead h;
  size_t off = 0, na = 0, nb = 0, ns = 0;
  for (int i = 0; i < n; ++i) {
    na += make_wavemap(probs[i].nx, probs[i].ny, probs[i].nz, kMinKz).nblocks;
    const long N = (long)probs[i].nx * probs[i].ny * probs[i].nz;
    nb += march_blocks_b(N);
    ns += std::min<long>(kResMaxWgs, N);
  }
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = al256(off + bytes);
    return o;
  };
  h.inst = take(sizeof(MarchInst) * n);
  h.res = take(sizeof(ResInst) * n);
  h.seats = take(sizeof(int2) * ns);
  h.blk_a = take(sizeof(int2) * na);
  h.blk_b = take(sizeof(int2) * nb);
  h.state_a = take(sizeof(MarchState) * n);
  h.state_b = take(sizeof(MarchState) * n);
  h.counts = take(sizeof(double) * kMaxBoxes * n);
  h.flags = take(sizeof(int) * n);
  h.done = take(256);
  h.total = off;
  return h;
}

static size_t batch_bytes(int n, const qe_problem* probs) {
  size_t t = batch_head(n, probs).total;
  for (int i = 0; i < n; ++i) t += inst_bytes(probs[i]);
  return t;
}

static int device_cus() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
  return cus;
}

static std::string tune_key(int n, const std::vector<long>& sizes) {
  int dev = 0;
  hipDeviceProp_t prop;
  std::string arch = "gpu";
  if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) arch = prop.gcnArchName;
  const long tot = std::accumulate(sizes.begin(), sizes.end(), 0L);
  const long mx = sizes.empty() ? 0 : *std::max_element(sizes.begin(), sizes.end());
  // bucket the workload: instance count and mean / max size to ~powers of two
  auto b2 = [](long v) {
    int k = 0;
    while ((1L << k) < v) ++k;
    return k;
  };
  std::ostringstream os;
  os << "march;" << arch << ";cu=" << device_cus() << ";n=" << b2(n) << ";mean=" << b2(n ? tot / n : 0) << ";max=" << b2(mx);
  std::string k = os.str();
  for (auto& ch : k)
    if (ch == ' ' || ch == '\n') ch = '_';
  return k;
}

static bool read_cache(const char* path, const std::string& key, int& kz) {
  if (!path) return false;
  std::ifstream f(path);
  std::string line;
  while (std::getline(f, line)) {
    std::istringstream is(line);
    std::string k;
    int v;
    if (is >> k >> v && k == key && v >= kMinKz && v <= kMaxKz9) {
      kz = v;
      return true;
    }
  }
  return false;
}

static void write_cache(const char* path, const std::string& key, int kz) {
  if (!path) return;
  std::ofstream f(path, std::ios::app);
  f << key << " " << kz << "\n";
}

// Zeroes the flags, the states' phases and the count of finished instances.
__global__ __launch_bounds__(256) void k_batch_begin(int* flags, MarchState* sb, int n, unsigned int* done) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    flags[i] = 0;
    sb[i].phase = MARCH_RES;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *done = 0;
}

// The cuts of all instances (nwg 0: does not fit), each mesh's found once.
// When the batch fills the chip, the cuts with the least workgroup time;
// otherwise each instance gets its share of the chip.
static void batch_plans(int n, const qe_problem* probs, int wgs, std::vector<ResPlan>& plans) {
  std::map<std::array<int, 3>, ResPlan> seen;
  // (most: workgroups an instance may have; what its boxes exchange fits the
  // room of the march's coefficients)
  auto cut = [&](int most, bool share) {
    seen.clear();
    long total = 0;
    for (int i = 0; i < n; ++i) {
      const qe_problem& p = probs[i];
      const std::array<int, 3> dims{p.nx, p.ny, p.nz};
      auto it = seen.find(dims);
      if (it == seen.end()) {
        ResPlan q{};
        const int fit = resident_fit((size_t)tile_slots(p.nx, p.ny, p.nz) * 64, (long)p.nx * p.ny * p.nz, wgs);
        if (!resident_plan(p.nx, p.ny, p.nz, std::min(fit, most), share, q) &&
            !resident_plan(p.nx, p.ny, p.nz, fit, share, q))
          q.nwg = 0;
        it = seen.emplace(dims, q).first;
      }
      plans[i] = it->second;
      total += plans[i].nwg;
    }
    return total;
  };
  if (cut(wgs, true) < wgs) cut(std::max(1, wgs / n), false);
}

// The order of the instances: first fit decreasing into rows of wgs boxes, so
// that the instances that are next to each other fill the chip.  us: time of
// a CG iteration of all of them, each row as long as its slowest.
static std::vector<int> batch_order(const std::vector<ResPlan>& plans, int wgs, double& us) {
  std::vector<int> by(plans.size());
  std::iota(by.begin(), by.end(), 0);
  std::stable_sort(by.begin(), by.end(), [&](int l, int r) { return plans[l].nwg > plans[r].nwg; });
  std::vector<std::vector<int>> rows;
  std::vector<int> room;
  size_t open = 0;   // rows before this one are full
  for (int i : by) {
    if (plans[i].nwg == 0) continue;
    size_t r = open;
    while (r < rows.size() && room[r] < plans[i].nwg) ++r;
    if (r == rows.size()) {
      rows.emplace_back();
      room.push_back(wgs);
    }
    rows[r].push_back(i);
    room[r] -= plans[i].nwg;
    while (open < rows.size() && room[open] == 0) ++open;
  }
  std::vector<int> order;
  us = 0.0;
  for (const auto& row : rows) {
    float slowest = 0.0f;
    for (int i : row) slowest = std::max(slowest, plans[i].cost);
    us += slowest;
    order.insert(order.end(), row.begin(), row.end());
  }
  return order;
}

// Which instances are solved resident: those of up to a number of nodes, the
// rest march; the number with the least time per CG iteration.  A tick of the
// march costs its two launches and its traffic over all instances (measured
// 12 us + 24 us per million nodes), so large instances are better marched
// together than solved one or two at a time.  Measured, resident / march: 40
// of 17x17x9 1.5 / 4.6 ms, 256 of 33x33x17 33 / 44, 64 of 49x49x25 66 / 49, 8
// and 256 of 65x65x33 30 / 20 and 856 / 443.
static std::vector<int> batch_split(const std::vector<long>& sizes, std::vector<ResPlan>& plans, int wgs) {
  std::vector<long> most(sizes);
  std::sort(most.begin(), most.end());
  most.erase(std::unique(most.begin(), most.end()), most.end());
  if (most.size() > 16) {   // (one in so many, and the largest)
    std::vector<long> some;
    for (size_t k = 1; k <= 16; ++k) some.push_back(most[k * most.size() / 16 - 1]);
    most.swap(some);
  }
  auto split = [&](long m, std::vector<ResPlan>& q) {
    double march = 0.0, us = 0.0;
    q = plans;
    for (size_t i = 0; i < q.size(); ++i) {
      if (sizes[i] > m) q[i].nwg = 0;
      if (q[i].nwg == 0) march += 24e-6 * sizes[i];
    }
    std::vector<int> order = batch_order(q, wgs, us);
    return std::make_pair(us + (march > 0.0 ? 12.0 + march : 0.0), order);
  };
  std::vector<ResPlan> q, best(plans.size(), ResPlan{});
  std::vector<int> order;
  double least = split(-1, q).first;   // all marched
  for (long m : most) {
    const auto r = split(m, q);
    if (r.first < least) {
      least = r.first;
      order = r.second;
      best = q;
    }
  }
  plans = best;
  return order;
}

struct EventRing {
  hipEvent_t e[kEventRing] = {};
  ~EventRing() {
    for (hipEvent_t v : e)
      if (v) (void)hipEventDestroy(v);
  }
};

}  // namespace qe

using namespace qe;

extern "C" {

size_t qe_batch_workspace_bytes(int32_t n_inst, const qe_problem* probs, const qe_options* o) {
  (void)o;
  if (n_inst < 1 || !probs) return 0;
  for (int i = 0; i < n_inst; ++i)
    if (check_problem(&probs[i]) != QE_OK) return 0;
  return batch_bytes(n_inst, probs);
}

qe_status qe_solve_batch(int32_t n_inst, const qe_problem* probs, const qe_physics* ph, const qe_options* o,
                         double* const* phi, int32_t n_boxes, const double* boxes, double* counts,
                         const char* tune_cache, void* ws_, size_t ws_bytes, void* stream, qe_report* reps) {
  clear_error();
  clear_routes();
  if (n_inst < 1 || !probs || !phi) return fail(QE_ERR_INVALID_ARG, "need n_inst >= 1, probs and phi");
  qe_status st;
  if ((st = check_options(o)) != QE_OK) return st;
  if (o->precision != QE_PREC_FP64) return fail(QE_ERR_INVALID_ARG, "the batched solve runs in FP64");
  // every instance starts from the linear guess (a coarse-mesh sequence is
  // for meshes far larger than the sweep's)
  if (o->init_guess == 1) return fail(QE_ERR_INVALID_ARG, "the batched solve starts from the linear guess");
  Charge ch;
  if ((st = make_charge(ph, ch)) != QE_OK) return st;
  if (n_boxes < 0 || n_boxes > kMaxBoxes) return fail(QE_ERR_INVALID_ARG, "n_boxes must be in [0, %d]", kMaxBoxes);
  if (n_boxes > 0 && (!boxes || !counts)) return fail(QE_ERR_INVALID_ARG, "boxes/counts is NULL");
  BoxSet bs;
  bs.n = n_boxes;
  for (int r = 0; r < n_boxes; ++r) {
    const double* b = boxes + 6 * r;
    for (int k = 0; k < 6; ++k)
      if (std::isnan(b[k])) return fail(QE_ERR_INVALID_ARG, "box %d has NaN", r);
    bs.b[r] = Box{b[0], b[1], b[2], b[3], b[4], b[5]};
  }
  for (int i = 0; i < n_inst; ++i) {
    if ((st = check_problem(&probs[i])) != QE_OK) return fail(st, "instance %d: %s", i, qe_last_error());
    if (!phi[i]) return fail(QE_ERR_INVALID_ARG, "phi[%d] is NULL", i);
    if (probs[i].quantum)
      return fail(QE_ERR_INVALID_ARG, "instance %d: predictor-corrector states are not supported by the batch", i);
    if (probs[i].n_sheets > 0)
      return fail(QE_ERR_INVALID_ARG, "instance %d: interface / Robin sheets are not supported by the batch", i);
    if (ch.incomplete && !probs[i].donors)
      return fail(QE_ERR_INVALID_ARG, "instance %d: incomplete ionization needs donors and acceptors", i);
  }
  const size_t need = batch_bytes(n_inst, probs);
  if (!ws_) return fail(QE_ERR_WORKSPACE, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(ws_) & 255) return fail(QE_ERR_WORKSPACE, "workspace not 256-byte aligned");
  if (ws_bytes < need) return fail(QE_ERR_WORKSPACE, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  hipStream_t s = (hipStream_t)stream;
  HostMirror& hm = mirror();
  if (!hm.ok) return fail(QE_ERR_HIP, "pinned host buffer allocation failed");
  char* ws = reinterpret_cast<char*>(ws_);
  const BatchHead H = batch_head(n_inst, probs);
  std::vector<long> sizes(n_inst);
  for (int i = 0; i < n_inst; ++i) sizes[i] = (long)probs[i].nx * probs[i].ny * probs[i].nz;
  const std::string key = tune_key(n_inst, sizes);
  int kz = kMaxKz9;
  if (!read_cache(tune_cache, key, kz)) {
    for (; kz > kMinKz; --kz) {
      long waves = 0;
      for (int i = 0; i < n_inst; ++i) waves += make_wavemap(probs[i].nx, probs[i].ny, probs[i].nz, kz).nwaves;
      if (waves >= kMinWaves) break;
    }
    write_cache(tune_cache, key, kz);
  }
  // the instances and the block tables, staged on the host as they lie in the
  // workspace
  std::vector<char> head(H.state_a);
  MarchInst* hinst = reinterpret_cast<MarchInst*>(head.data() + H.inst);
  ResInst* hres = reinterpret_cast<ResInst*>(head.data() + H.res);
  int2* seats = reinterpret_cast<int2*>(head.data() + H.seats);
  std::vector<ResPlan> plans(n_inst);
  const int wgs = resident_on() ? resident_wgs() : 0;
  int n_seats = 0, placed = 0;
  if (wgs > 0) {
    batch_plans(n_inst, probs, wgs, plans);
    for (int i : batch_split(sizes, plans, wgs)) {
      ++placed;
      for (int b = 0; b < plans[i].nwg; ++b) seats[n_seats++] = make_int2(i, b);
    }
  }
  int2* blk_a = reinterpret_cast<int2*>(head.data() + H.blk_a);
  int2* blk_b = reinterpret_cast<int2*>(head.data() + H.blk_b);
  MarchArgs a;
  std::memset(&a, 0, sizeof(a));
  size_t off = H.total;
  for (int i = 0; i < n_inst; ++i) {
    const qe_problem& p = probs[i];
    MarchInst& I = hinst[i];
    const long N = sizes[i], S = tile_slots(p.nx, p.ny, p.nz);
    const long tiles = make_wavemap(p.nx, p.ny, p.nz, kMinKz).nwaves;
    auto tk = [&](size_t bytes) {
      char* q = ws + off;
      off = al256(off + bytes);
      return q;
    };
    I.wm = make_wavemap(p.nx, p.ny, p.nz, kz);
    I.eps = p.eps_r;
    I.semi = p.semi;
    I.dop = Doping{p.net_doping, p.donors, p.acceptors};
    I.dir_id = p.dir_id;
    I.dir_val = p.dir_val;
    I.phi = phi[i];
    I.x = reinterpret_cast<double*>(tk(N * 8));
    I.r = reinterpret_cast<double*>(tk(N * 8));
    I.z = reinterpret_cast<double*>(tk(N * 8));
    I.p = reinterpret_cast<double*>(tk(N * 8));
    I.y = reinterpret_cast<double*>(tk(N * 8));
    I.invdiag = reinterpret_cast<double*>(tk(N * 8));
    I.c = reinterpret_cast<double*>(tk(S * 64));
    I.eps_t = reinterpret_cast<double*>(tk(S * 8));
    I.cflag = reinterpret_cast<uint8_t*>(tk(S));
    I.mask = reinterpret_cast<uint8_t*>(tk(N));
    I.rdz = reinterpret_cast<double*>(tk(2 * (p.nz - 1) * 8));
    I.cbits = reinterpret_cast<unsigned int*>(tk(tiles * 64 * 4));
    I.part_a = reinterpret_cast<double*>(tk((tiles + 3) / 4 * 8));
    I.nb = march_blocks_b(N);
    I.part_b = reinterpret_cast<double*>(tk(I.nb * 8));
    I.sa = reinterpret_cast<MarchState*>(ws + H.state_a) + i;
    I.sb = reinterpret_cast<MarchState*>(ws + H.state_b) + i;
    I.g = Geom{p.nx, p.ny, p.nz, p.x, p.y, p.z, I.rdz, I.rdz + (p.nz - 1)};
    I.N = N;
    I.E = (long)(p.nx - 1) * (p.ny - 1) * (p.nz - 1);
    I.nslots = S;
    I.na = I.wm.nblocks;
    I.n_dir = p.n_dir;
    ResInst& R = hres[i];
    R.nx = p.nx;
    R.ny = p.ny;
    R.nz = p.nz;
    R.n_dir = p.n_dir;
    R.x = p.x;
    R.y = p.y;
    R.z = p.z;
    R.eps = p.eps_r;
    R.semi = p.semi;
    R.dop = I.dop;
    R.dir_id = p.dir_id;
    R.dir_val = p.dir_val;
    R.phi = phi[i];
    R.keep = nullptr;   // (every start is the linear guess)
    // two vectors' room each
    R.w0 = reinterpret_cast<unsigned long long*>(I.x);
    R.w1 = reinterpret_cast<unsigned long long*>(I.z);
    R.d = reinterpret_cast<unsigned long long*>(I.y);
    R.part = reinterpret_cast<unsigned long long*>(I.c);
    R.plan = plans[i];
    R.flags = nullptr;
    R.out = I.sb;
    for (int b = 0; b < I.na; ++b) blk_a[a.na++] = make_int2(i, b);
    for (int b = 0; b < I.nb; ++b) blk_b[a.nb++] = make_int2(i, b);
  }
  a.n_inst = n_inst;
  a.inst = reinterpret_cast<const MarchInst*>(ws + H.inst);
  a.blk_a = reinterpret_cast<const int2*>(ws + H.blk_a);
  a.blk_b = reinterpret_cast<const int2*>(ws + H.blk_b);
  a.ch = ch;
  a.atol = o->newton_atol;
  a.rtol_max = o->krylov_rtol_max;
  a.newton_maxit = o->newton_maxit;
  a.ls_max = o->ls_max_halvings;
  a.krylov_maxit = o->krylov_maxit;
  a.lenient = 1;
  a.init = MARCH_LINEAR;
  a.apply = a.zero_free = 1;
  a.flags = reinterpret_cast<int*>(ws + H.flags);
  a.done = reinterpret_cast<unsigned int*>(ws + H.done);
  auto hip_ok = [](hipError_t e) { return e == hipSuccess; };
  if (!hip_ok(hipMemcpyAsync(ws, head.data(), head.size(), hipMemcpyHostToDevice, s)))
    return fail(QE_ERR_HIP, "descriptor upload failed");
  hipLaunchKernelGGL(k_batch_begin, dim3((n_inst + 255) / 256), dim3(256), 0, s, a.flags,
                     reinterpret_cast<MarchState*>(ws + H.state_b), n_inst, a.done);
  launch_march_validate(s, a);
  // nothing is solved unless every instance is valid
  std::vector<int> flags(n_inst);
  if (!hip_ok(hipGetLastError()) ||
      !hip_ok(hipMemcpyAsync(flags.data(), a.flags, n_inst * sizeof(int), hipMemcpyDeviceToHost, s)) ||
      !hip_ok(hipStreamSynchronize(s)))
    return fail(QE_ERR_HIP, "validation failed to run");
  for (int i = 0; i < n_inst; ++i)
    for (int ax = 0; ax < 3; ++ax)
      if (flags[i] & (128 << ax))
        return fail(QE_ERR_INVALID_ARG, "instance %d: coordinates %c not strictly increasing", i, "xyz"[ax]);
  int f = 0;
  for (int i = 0; i < n_inst; ++i) f |= flags[i];
  if (f & 1) return fail(QE_ERR_INVALID_ARG, "eps_r must be finite and > 0");
  if (f & 2) return fail(QE_ERR_NONFINITE, "net_doping not finite or donors / acceptors not finite and >= 0");
  if (f & 4) return fail(QE_ERR_INVALID_ARG, "dir_id outside [-1, n_dir)");
  std::vector<char> res(H.flags - H.state_b);
  const MarchState* hs = reinterpret_cast<const MarchState*>(res.data());
  auto read_back = [&]() {
    return hip_ok(hipGetLastError()) &&
           hip_ok(hipMemcpyAsync(res.data(), ws + H.state_b, res.size(), hipMemcpyDeviceToHost, s)) &&
           hip_ok(hipStreamSynchronize(s));
  };
  ResidentTurn turn(placed > 0);
  if (turn.held()) {
    ResArgs ra;
    std::memset(&ra, 0, sizeof(ra));
    ra.inst = reinterpret_cast<const ResInst*>(ws + H.res);
    ra.n_inst = n_inst;
    ra.seats = reinterpret_cast<const int2*>(ws + H.seats);
    ra.n_seats = n_seats;
    ra.ticket = a.done + 16;
    ra.started = a.done + 17;
    ra.abort = reinterpret_cast<unsigned long long*>(a.done + 32);
    ra.ch = ch;
    ra.atol = a.atol;
    ra.rtol_max = a.rtol_max;
    ra.newton_maxit = a.newton_maxit;
    ra.ls_max = a.ls_max;
    ra.krylov_maxit = a.krylov_maxit;
    ra.lenient = 1;
    ra.init = MARCH_LINEAR;
    ra.apply = ra.zero_free = 1;
    if ((st = launch_resident(s, ra, plans.data(), n_inst, wgs)) != QE_OK) return st;
  }
  const bool tried = turn.held();
  bool all = turn.held() && placed == n_inst;
  if (n_boxes > 0 && all) launch_march_count(s, a, bs, reinterpret_cast<double*>(ws + H.counts));
  if (all) {
    if (!read_back()) return fail(QE_ERR_HIP, "batch kernel failed");
    for (int i = 0; i < n_inst; ++i) all = all && hs[i].phase == MARCH_DONE;
  }
  if (!all) {
    if (turn.held() && !hip_ok(hipStreamSynchronize(s))) return fail(QE_ERR_HIP, "batch kernel failed");
    turn.release();   // (the march takes as long as it takes)
    hm.prog->word = 0;
    a.prog = hm.prog_dev;
    launch_march_stage(s, a);
    EventRing ring;
    if ((st = march_run(s, a, hm, ring.e, 0)) != QE_OK) return st;
    if (n_boxes > 0) launch_march_count(s, a, bs, reinterpret_cast<double*>(ws + H.counts));
    if (!read_back()) return fail(QE_ERR_HIP, "batch kernel failed");
  }
  const double* hc = reinterpret_cast<const double*>(res.data() + (H.counts - H.state_b));
  qe_status worst = QE_OK;
  for (int i = 0; i < n_inst; ++i) {
    if (reps) {
      qe_report& r = reps[i];
      std::memset(&r, 0, sizeof(r));
      r.status = hs[i].status;
      r.newton_iters = hs[i].newton;
      r.krylov_iters = hs[i].kry;
      r.ls_halvings = hs[i].halv;
      r.init_krylov_iters = hs[i].init_kry;
      r.n_residual_evals = hs[i].nres;
      r.res0 = hs[i].res0;
      r.res_final = hs[i].nrm;
    }
    for (int b = 0; b < n_boxes; ++b) counts[(long)i * n_boxes + b] = hc[(long)i * n_boxes + b];
    add_route(hs[i].resident ? ROUTE_RESIDENT : tried && plans[i].nwg > 0 ? ROUTE_LEFT : ROUTE_OTHER);
    if (hs[i].status != QE_OK && worst == QE_OK) worst = (qe_status)hs[i].status;
  }
  if (worst != QE_OK) return fail(worst, "at least one instance did not converge (see the reports)");
  return QE_OK;
}

}  // extern "C"
