// Host runtime of libshellhom: validation, slot layout and setup, and the
// batched PCG driver shared by the single-design entry points, the batch
// entry points and the serving engine.
#include "runtime.hpp"
#include "sel.hpp"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>

#include "kernels.hpp"

namespace shh {

#define SHH_HIP(call)                                \
  do {                                               \
    hipError_t e_ = (call);                          \
    if (e_ != hipSuccess) return SHH_HIP_ERROR;      \
  } while (0)

namespace {
std::atomic<bool> g_prof_on{false};
std::mutex g_prof_mu;
long long g_prof_launches[SHH_PROF_NKIND] = {};
double g_prof_ms[SHH_PROF_NKIND] = {};
}  // namespace

void profile_enable(bool on) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  g_prof_on = on;
  if (on) {
    for (int k = 0; k < SHH_PROF_NKIND; ++k) {
      g_prof_launches[k] = 0;
      g_prof_ms[k] = 0.0;
    }
  }
}
bool profile_on() { return g_prof_on.load(); }
int profile_read(int kind, long long *launches, double *ms) {
  if (kind < 0 || kind >= SHH_PROF_NKIND) return SHH_INVALID_ARG;
  std::lock_guard<std::mutex> lk(g_prof_mu);
  if (launches) *launches = g_prof_launches[kind];
  if (ms) *ms = g_prof_ms[kind];
  return SHH_OK;
}
void profile_add(int kind, double ms) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  g_prof_launches[kind] += 1;
  g_prof_ms[kind] += ms;
}

double now_ms() {
  using namespace std::chrono;
  return duration<double, std::milli>(steady_clock::now().time_since_epoch()).count();
}

static bool finite(double v) { return std::isfinite(v); }

int sym_images(int sym) { return sym == SHH_SYM_MIRROR ? 8 : (sym == SHH_SYM_CUBIC ? 48 : 1); }

// Image g of a point under the fundamental volume's group: the axes permuted
// (permutation g / 8 of six, cubic only), then reflected x_d -> 1 - x_d for
// the bits of g % 8.
static const int kPerm[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};

void sym_image(int g, const double *p, double *v) {
  const int *pm = kPerm[g / 8];
  for (int d = 0; d < 3; ++d) {
    v[d] = p[pm[d]];
    if ((g >> d) & 1) v[d] = 1.0 - v[d];
  }
}

// dL/dp of a given charge accumulates dL/dv of its image g (the transpose of
// the image map's linear part)
void sym_fold(int g, const double *gv, double *gp) {
  const int *pm = kPerm[g / 8];
  for (int d = 0; d < 3; ++d) gp[pm[d]] += ((g >> d) & 1) ? -gv[d] : gv[d];
}

int charge_count(const shh_design *d) { return d->num_charges * sym_images(d->symmetry); }

int validate_design(const shh_design *d) {
  if (!d) return SHH_INVALID_ARG;
  if (d->n < 2 || d->n > 512) return SHH_INVALID_ARG;  // 32-bit byte offsets per vector
  if (d->num_charges < 1 || !d->pos || !d->q) return SHH_INVALID_ARG;
  if (d->symmetry < SHH_SYM_NONE || d->symmetry > SHH_SYM_CUBIC) return SHH_INVALID_ARG;
  if ((long long)d->num_charges * sym_images(d->symmetry) > 4096) return SHH_INVALID_ARG;
  if (d->K < 1 || d->K > MAXK) return SHH_INVALID_ARG;
  for (int j = 0; j < d->num_charges; ++j) {
    if (!finite(d->pos[3 * j]) || !finite(d->pos[3 * j + 1]) || !finite(d->pos[3 * j + 2]) ||
        !finite(d->q[j]))
      return SHH_INVALID_ARG;
  }
  if (d->alpha) {
    const int K1 = d->K + 1;
    for (int i = 0; i < K1 * K1 * K1; ++i)
      if (!finite(d->alpha[i])) return SHH_INVALID_ARG;
  }
  if (!finite(d->iso)) return SHH_INVALID_ARG;
  if (!finite(d->thickness)) return SHH_INVALID_ARG;
  if (d->thickness < 0 && !(d->target_vf > 0.0 && d->target_vf < 1.0)) return SHH_INVALID_ARG;
  if (!(d->kappa >= 0.0) || !finite(d->kappa)) return SHH_INVALID_ARG;
  if (d->dist_mode != 0 && d->dist_mode != 1) return SHH_INVALID_ARG;
  if (!(d->E > 0.0) || !finite(d->E)) return SHH_INVALID_ARG;
  if (!(d->nu > -1.0 && d->nu < 0.5)) return SHH_INVALID_ARG;
  if (!(d->E_void >= 0.0 && d->E_void <= d->E)) return SHH_INVALID_ARG;
  return SHH_OK;
}

int normalize_opts(const shh_opts *in, shh_opts *out) {
  if (!in) return SHH_INVALID_ARG;
  *out = *in;
  if (out->precision != SHH_PREC_FP64 && out->precision != SHH_PREC_MIXED) return SHH_INVALID_ARG;
  if (!(out->rtol > 0.0 && out->rtol < 1.0)) return SHH_INVALID_ARG;
  if (out->max_iter < 0 || out->recompute_every < 0 || out->check_every < 0) return SHH_INVALID_ARG;
  if (out->solver != SHH_SOLVER_JACOBI && out->solver != SHH_SOLVER_MG && out->solver != SHH_SOLVER_AUTO &&
      !is_selective(out->solver))
    return SHH_INVALID_ARG;
  // the selective multigrid solve replaces its FP32 residual five times as
  // often: its V-cycle puts large components along the culled operator's
  // (near-)null modes, which the FP32 recursion turns into residual drift
  if (out->recompute_every == 0 && out->precision == SHH_PREC_MIXED)
    out->recompute_every = out->solver == SHH_SOLVER_SELECTIVE ? 10 : 50;
  return SHH_OK;
}

// Iterations until the next look at the slots' states where the caller set no
// period: until the last load case is due at its rate of convergence (since the
// last look, or from the start), at least 2 and at most 16 -- 64 in a solve of
// hundreds of iterations while the end is far (an early estimate says little: the
// residual of the first iterations hardly falls).  A fixed 16 ran up to 15 empty
// iterations after the last load case stopped: a twentieth of a 48^3 solve.  The
// arithmetic does not depend on it.
int next_poll(const std::vector<Slot *> &slots, int fixed) {
  if (fixed > 0) return fixed;
  double left = 0.0;
  int done = 0;
  for (Slot *s : slots) {
    const CgState &c = s->state;
    int it = 0;
    double v = -1e300;
    for (int k = 0; k < NRHS; ++k) {
      if (!c.active[k]) continue;
      it = std::max(it, c.iters[k]);
      v = std::max(v, c.rel[k] > 0.0 && std::isfinite(c.rel[k]) ? std::log(c.rel[k] / s->host.rtol) : 0.0);
    }
    if (it <= 0 || v <= 0.0) {  // not started, or about to stop
      left = std::max(left, it <= 0 ? 16.0 : 2.0);
      continue;
    }
    done = std::max(done, it);
    const double all = (std::log(1.0 / s->host.rtol) - v) / it;
    const double recent = it > s->polled_at ? (s->polled_log - v) / (it - s->polled_at) : 0.0;
    const double rate = s->polled_at > 0 && recent > 0.0 ? recent : all;
    left = std::max(left, rate > 0.0 ? v / rate : 16.0);
    s->polled_at = it;
    s->polled_log = v;
  }
  return std::max(2, std::min(left > 128.0 && done > 128 ? 64 : 16, int(std::min(left, 1e6)) + 1));
}

static size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// The tiling of a slot's operator passes.  FP64: 32 x 14 nodes keep eight waves on
// a CU (one workgroup; the passes' registers allow no more), 32 x 8 five, or ten
// where two workgroups fit.  The tall tile pays where it needs no more waves in all
// than the flat one, since more of them share a halo (ms, flat and tall: multigrid
// 28^3 5.8 and 5.3, 64^3 17.2 and 14.6, 96^3 34.1 and 27.5; Jacobi 25^3 9.2 and
// 7.4, 101^3 703 and 674), and in the multigrid, whose passes stage more, up to a
// tenth more: 48^3 (7 % more waves) 10.3 and 9.1, 32^3 (20 % more) 5.1 and 5.2.
// The Jacobi CG is even there (7 % more: 45^3 35.5 and 34.8, 71^3 162 and 179; as
// many: 57^3 69.6 and 72.3).  Below 25^3 a pass is as long as one workgroup, and
// the flat tile's is the shorter (multigrid 16^3 4.8 and 4.9, 24^3 4.1 and 4.2).
// It depends on the grid, precision and solver alone.
static int tile_x(int tiling) { return tiling == TILING_F32 ? Tile<float>::X : Tile<double>::X; }
static int tile_y(int tiling) {
  return tiling == TILING_F32 ? Tile<float>::Y : (tiling == TILING_F64 ? Tile<double>::Y : Tile<double, true>::Y);
}
static int tile_count(int n, int tiling) {
  return ((n + tile_x(tiling) - 1) / tile_x(tiling)) * ((n + tile_y(tiling) - 1) / tile_y(tiling));
}
static int tiling_for(int n, int prec, int solver) {
  if (prec != SHH_PREC_FP64) return TILING_F32;
  const int tall = tile_count(n, TILING_F64_TALL) * (Tile<double, true>::THREADS / 64);
  const int flat = tile_count(n, TILING_F64) * (Tile<double>::THREADS / 64);
  return n >= 25 && (solver == SHH_SOLVER_MG ? 10 * tall <= 11 * flat : tall <= flat) ? TILING_F64_TALL : TILING_F64;
}

// z planes per stencil workgroup (the z-march length) of an n^3 grid.  One
// design's six load cases are tiles x runs x 6 workgroups on 512 places (two
// workgroups on each of 256 CUs; 256 with the tall FP64 tile); a workgroup of tz planes takes about tz + 3
// layer times (two planes of halo and the pipeline's start).  The length is the
// even one, at most 64, with the smallest sum of the time of one design alone
// (whole rounds over the places) and twice that in a large batch (rounds
// shared): short runs where the grid would leave the chip idle (FP32, 48^3: 6
// planes, where 32 ran 96 workgroups: a Jacobi pass at 45^3 61 -> 27 us; a design
// at 24^3 in FP64 27.6 -> 19.9 ms), balanced rounds on larger grids (FP32, 128^3:
// 26, where 32 left the third round at 6 %).  It depends on the grid, precision and
// solver alone, so a design's result does not depend on its batch.
static int tz_for(int n, int tiling) {
  // the tall FP64 tile's LDS leaves one workgroup on a CU
  const long long places = tiling == TILING_F32 ? 256 * (1024 / Tile<float>::THREADS) : (tiling == TILING_F64 ? 512 : 256);
  const long long tiles = (long long)tile_count(n, tiling) * NRHS;
  int best = 2;
  double best_cost = -1.0;
  for (int tz = 2; tz <= n + 1 && tz <= 64; tz += 2) {
    const long long groups = tiles * ((n + tz - 1) / tz);
    const double cost = (double((groups + places - 1) / places) + 2.0 * double(groups) / places) * (tz + 3);
    if (best_cost < 0.0 || cost <= best_cost) {  // of equal costs the longer run: less halo
      best = tz;
      best_cost = cost;
    }
  }
  return best;
}

Layout make_layout(int n, int N, int K, int prec, bool save, bool vectors, int solver) {
  Layout L{};
  L.vectors = vectors;
  const long long nn = (long long)n * n * n;
  const int nb = 2 * K + 1;
  // room for the runs of either solver's tiling: an adjoint call may name another
  // solver than its forward, so nothing before the multigrid region depends on it
  int runs = 0, tiles = 0;
  for (int sv : {SHH_SOLVER_JACOBI, SHH_SOLVER_MG}) {
    const int tz = tz_for(n, tiling_for(n, prec, sv));
    runs = std::max(runs, (n + tz - 1) / tz);
  }
  for (int w = 0; w < NTILING; ++w) tiles = std::max(tiles, tile_count(n, w) * runs);
  const int chunks = int((nn + CHUNK - 1) / CHUNK);
  L.maxparts = std::max(std::max(tiles, chunks), 1024);
  const size_t ts = prec == SHH_PREC_FP64 ? 8 : 4;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align256(off + bytes);
    return o;
  };
  L.slotdev = take(sizeof(SlotDev));
  L.state = take(sizeof(CgState));
  L.charges = take(sizeof(double) * 4 * (size_t)N);
  L.alpha = take(sizeof(double) * (size_t)(K + 1) * (K + 1) * (K + 1));
  L.coef = take(sizeof(double) * (size_t)nb * nb * nb);
  L.partials = take(sizeof(double) * (size_t)NRHS * L.maxparts * PSTRIDE);
  L.segs = take(4096);
  L.E64 = take(sizeof(double) * nn);
  L.E32 = prec == SHH_PREC_MIXED ? take(sizeof(float) * nn) : 0;
  L.Dinv = take(ts * nn);
  if (!vectors) {  // the operator calls bring their own vectors
    L.total = off;
    return L;
  }
  L.x64 = prec == SHH_PREC_MIXED ? take(sizeof(double) * NRHS * 3 * nn) : 0;
  L.vec_bytes = align256(ts * NRHS * 3 * nn);
  L.vec = take(7 * L.vec_bytes);  // r[2], p[2], q[2], x
  // after a forward with save, the adjoint takes r[0] for dL/dE and p[0], p[1],
  // q[0], q[1] as scratch -- or a region of its own on grids too small for
  // that, so that the solution (x, or x64) survives for further calls
  if (save) {
    const size_t adj = align256(adjoint_scratch_bytes(n, K));
    L.adj = adj <= 4 * L.vec_bytes ? L.vec + 2 * L.vec_bytes : take(adj);
  }
  L.field = save ? take(sizeof(double) * 5 * nn) : L.vec;  // F, G[3], d (aliased unless saved)
  // the selective solve takes the same multigrid region for its coarse levels
  if (solver == SHH_SOLVER_MG || solver == SHH_SOLVER_SELECTIVE) L.mg = take(mg_region_bytes(n, prec));
  L.total = off;
  return L;
}

void copy_design(const shh_design *src, DesignCopy &dst) {
  dst.d = *src;
  const int N = src->num_charges, G = sym_images(src->symmetry);
  dst.sym = src->symmetry;
  dst.nfbv = N;
  // the fundamental volume's charges and their images, charge by charge
  dst.pos.resize(3 * (size_t)N * G);
  dst.q.resize((size_t)N * G);
  for (int j = 0; j < N; ++j)
    for (int g = 0; g < G; ++g) {
      sym_image(g, src->pos + 3 * j, &dst.pos[3 * ((size_t)j * G + g)]);
      dst.q[(size_t)j * G + g] = src->q[j];
    }
  dst.d.num_charges = N * G;
  dst.d.symmetry = SHH_SYM_NONE;
  if (src->alpha) {
    const int K1 = src->K + 1;
    dst.alpha.assign(src->alpha, src->alpha + K1 * K1 * K1);
    dst.d.alpha = dst.alpha.data();
  } else {
    dst.alpha.clear();
    dst.d.alpha = nullptr;
  }
  dst.d.pos = dst.pos.data();
  dst.d.q = dst.q.data();
}

static void element_operator(double nu, double kop[KOP_N]) {
  const double lam = nu / ((1.0 + nu) * (1.0 - 2.0 * nu));
  const double mu = 1.0 / (2.0 * (1.0 + nu));
  const double Mh[2] = {1.0, 1.0 / 3.0}, Sh[2] = {0.0, 4.0};
  // diagonal entry of component c at mode m depends on s_c and s_o1 + s_o2 only
  for (int sc = 0; sc < 2; ++sc)
    for (int so = 0; so < 3; ++so) {
      const int s1 = so > 0 ? 1 : 0, s2 = so > 1 ? 1 : 0;
      kop[sc * 3 + so] = ((lam + 2.0 * mu) * Sh[sc] * Mh[s1] * Mh[s2] +
                          mu * Mh[sc] * (Sh[s1] * Mh[s2] + Mh[s1] * Sh[s2])) / 64.0;
    }
  for (int mk = 0; mk < 2; ++mk) {
    kop[6 + mk] = 4.0 * lam * Mh[mk] / 64.0;
    kop[8 + mk] = 4.0 * mu * Mh[mk] / 64.0;
  }
}

int slot_init(Slot &s, char *base, hipStream_t st, const std::function<void(SlotDev &)> &adjust,
              const OperatorSegment *op) {
  const shh_design &d = s.design.d;
  const int prec = s.opts.precision;
  s.base = base;
  const Layout &L = s.lay;
  SlotDev &h = s.host;
  std::memset(&h, 0, sizeof(h));
  const int n = d.n;
  h.n = n;
  h.prec = prec;
  h.nn = (long long)n * n * n;
  h.wt = tiling_for(n, prec, s.opts.solver);
  h.wr = prec == SHH_PREC_FP64 ? h.wt : TILING_F64_TALL;  // (mixed, 128^3: a solve 1 % faster than with the flat tile)
  h.tz = tz_for(n, h.wt);
  h.tiles_z = (n + h.tz - 1) / h.tz;
  for (int w = 0; w < NTILING; ++w) {
    h.tiles_x[w] = (n + tile_x(w) - 1) / tile_x(w);
    h.tiles_y[w] = (n + tile_y(w) - 1) / tile_y(w);
    h.ntiles[w] = h.tiles_x[w] * h.tiles_y[w] * h.tiles_z;
  }
  h.nchunks = int((h.nn + CHUNK - 1) / CHUNK);
  h.K = d.K;
  h.nb = 2 * d.K + 1;
  h.N = d.num_charges;
  h.dist_mode = d.dist_mode;
  h.maxparts = L.maxparts;
  h.mode_t = d.thickness >= 0 ? 0 : (d.kappa == 0.0 ? 1 : 2);
  h.lam = d.nu / ((1.0 + d.nu) * (1.0 - 2.0 * d.nu));
  h.mu = 1.0 / (2.0 * (1.0 + d.nu));
  h.E = d.E;
  h.E_void = is_selective(s.opts.solver) ? 0.0 : d.E_void;  // the culled system has no floor: E_e = E beta
  h.iso = d.iso;
  h.kappa = d.kappa;
  h.t_given = d.thickness;
  h.target_vf = d.target_vf;
  h.rtol = s.opts.rtol;
  h.max_iter = s.opts.max_iter;
  h.ffloor = 1e-12 * d.E * std::sqrt(3.0 * double(h.nn));
  h.cull = is_selective(s.opts.solver) ? SEL_EPS : 0.0;
  element_operator(d.nu, h.kop64);
  for (int i = 0; i < KOP_N; ++i) h.kop32[i] = (float)h.kop64[i];
  h.charges = (double *)(base + L.charges);
  h.alpha = d.alpha ? (double *)(base + L.alpha) : nullptr;
  h.coef = (double *)(base + L.coef);
  h.F = L.vectors ? (double *)(base + L.field) : nullptr;
  h.G = L.vectors ? h.F + h.nn : nullptr;
  h.d = L.vectors ? h.F + 4 * h.nn : nullptr;
  h.E64 = (double *)(base + L.E64);
  h.E32 = prec == SHH_PREC_MIXED ? (float *)(base + L.E32) : nullptr;
  h.Dinv = base + L.Dinv;
  if (L.vectors) {
    for (int b = 0; b < 2; ++b) {
      h.r[b] = base + L.vec + (0 + b) * L.vec_bytes;
      h.p[b] = base + L.vec + (2 + b) * L.vec_bytes;
      h.q[b] = base + L.vec + (4 + b) * L.vec_bytes;
    }
    h.x = base + L.vec + 6 * L.vec_bytes;
    h.x64 = prec == SHH_PREC_MIXED ? (double *)(base + L.x64) : (double *)h.x;
  }  // else: left null; each operator call sets the vectors it uses
  h.partials = (double *)(base + L.partials);
  h.st = (CgState *)(base + L.state);
  s.d_slot = (SlotDev *)(base + L.slotdev);
  s.d_state = h.st;
  CgState init;
  std::memset(&init, 0, sizeof(init));
  init.t = d.thickness;
  if (adjust) adjust(h);
  // descriptor, state, charges and alpha lie one after the other at the
  // region's start: one copy (four and a wait took 40 us of a call)
  const size_t K13 = (size_t)(d.K + 1) * (d.K + 1) * (d.K + 1);
  if (!s.upload.empty()) SHH_HIP(hipStreamSynchronize(s.upload_stream));
  s.upload.assign(L.alpha + (d.alpha ? sizeof(double) * K13 : (op ? sizeof(Segment) : 0)), 0);
  s.upload_stream = st;
  char *up = s.upload.data();
  std::memcpy(up + L.slotdev, &h, sizeof(SlotDev));
  std::memcpy(up + L.state, &init, sizeof(CgState));
  double *ch = (double *)(up + L.charges);
  for (int j = 0; j < h.N; ++j) {
    ch[4 * j] = d.pos[3 * j];
    ch[4 * j + 1] = d.pos[3 * j + 1];
    ch[4 * j + 2] = d.pos[3 * j + 2];
    ch[4 * j + 3] = d.q[j];
  }
  if (d.alpha) {
    std::memcpy(up + L.alpha, d.alpha, sizeof(double) * K13);
  } else if (op) {
    static_assert(sizeof(Segment) <= 8 * sizeof(double), "fits the weights of the smallest K");
    Segment g;
    std::memset(&g, 0, sizeof(g));
    g.slot = s.d_slot;
    g.nrhs = op->nrhs;
    for (int r = 0; r < op->nrhs; ++r) g.rhs[r] = r;
    g.flag = op->flag;
    g.nblocks = h.ntiles[op->residual ? h.wr : h.wt] * op->nrhs;
    std::memcpy(up + L.alpha, &g, sizeof(g));
  }
  SHH_HIP(hipMemcpyAsync(base, up, s.upload.size(), hipMemcpyHostToDevice, st));
  return SHH_OK;
}

int slot_setup_field(Slot &s, double *beta_out, hipStream_t st, bool solve) {
  const SlotDev &h = s.host;
  SHH_HIP(launch_field(s.d_slot, h.n, h.nb, (long long)NRHS * h.maxparts * PSTRIDE, st));
  if (h.mode_t == 1) {
    const long long k = (long long)std::floor(h.target_vf * double(h.nn) + 0.5);
    SHH_HIP(launch_select_hard(s.d_slot, h.nn, k, st));
  } else if (h.mode_t == 2) {
    SHH_HIP(launch_bisect(s.d_slot, h.nn, st));
  }
  SHH_HIP(launch_occupancy(s.d_slot, h.nn, beta_out, st));
  if (solve) SHH_HIP(launch_dinv(s.d_slot, h.nn, h.prec, st));
  return SHH_OK;
}

int slot_setup_moduli(Slot &s, const void *d_E, int e_dtype, double Es, double Ev, hipStream_t st) {
  const SlotDev &h = s.host;
  SHH_HIP(launch_moduli(s.d_slot, h.nn, d_E, e_dtype, Es, Ev, h.prec, st));
  return SHH_OK;
}

// ---------------------------------------------------------------------------
// batched solver
// ---------------------------------------------------------------------------

size_t Solver::seg_bytes(int max_slots) {
  return align256(sizeof(Segment) * (size_t)std::max(max_slots, 1)) * SEG_TABLES;
}

void Solver::set_segment_memory(char *d_mem, size_t bytes) {
  seg_mem_ = d_mem;
  seg_cap_ = bytes / SEG_TABLES;
  for (auto &v : host_segs_) v.clear();
}

// Divide the workgroups among the XCDs in order, each taking its share of the
// cost: grids of different sizes march z-runs of different lengths, and equal
// counts left the XCDs of the long runs behind (a batch of 64^3, 96^3 and 128^3
// designs ran 5 to 7 % slower).
static void split_by_cost(const std::vector<Segment> &segs, const std::vector<int> &cost, LaunchArgs &la) {
  long long all = 0;
  for (size_t i = 0; i < segs.size(); ++i) all += (long long)segs[i].nblocks * cost[i];
  la.per = 0;
  la.start[0] = 0;
  size_t i = 0;
  long long before = 0;  // cost of the segments before i
  for (int x = 1; x <= NXCD; ++x) {
    const long long upto = (all * x + NXCD - 1) / NXCD;
    while (i < segs.size() && before + (long long)segs[i].nblocks * cost[i] < upto)
      before += (long long)segs[i].nblocks * cost[i], ++i;
    la.start[x] = i < segs.size() ? segs[i].first + int((upto - before + cost[i] - 1) / cost[i]) : la.total;
    la.start[x] = std::min(la.start[x], la.total);
    la.per = std::max(la.per, la.start[x] - la.start[x - 1]);
  }
}

// The launch of kind k over the slots' live load cases.  With `tall`, a per-tile
// kind's FP64 slots of the tall tiling make a launch of their own, its segments
// behind the others' in the kind's table.
int Solver::build(Kind k, const std::vector<Slot *> &slots, int flag, bool all_rhs, LaunchArgs &la,
                  LaunchArgs *tall) {
  std::vector<Segment> segs[2];
  std::vector<int> cost[2];  // of one workgroup of each segment
  int first[2] = {0, 0};
  for (Slot *s : slots) {
    Segment g;
    std::memset(&g, 0, sizeof(g));
    g.slot = s->d_slot;
    g.flag = flag;
    const bool per_tile = (k == K_STENCIL || k == K_RESID || k == K_MG_DIR || k == K_MG_PRE || k == K_MG_POST);
    const bool scalar = (k == K_SCAL_IT || k == K_SCAL_RES);
    // the CG pass and the operator compute in the vector precision, the residual always in FP64
    const int tiling = k == K_RESID ? s->host.wr : s->host.wt;
    const int t = tall && s->host.prec == SHH_PREC_FP64 && tiling == TILING_F64_TALL;
    const int units = scalar ? 1 : (per_tile ? s->host.ntiles[tiling] : s->host.nchunks);
    if (k == K_FOLD || k == K_ZERO) {
      g.nrhs = 1;
      g.rhs[0] = 0;
    } else {
      g.nrhs = 0;
      for (int r = 0; r < NRHS; ++r) {
        // skip load cases known (from the last read-back) to be finished, unless asked for all
        const bool live = all_rhs || s->state.active[r];
        if (live) g.rhs[g.nrhs++] = r;
      }
      if (g.nrhs == 0) continue;
    }
    g.first = first[t];
    g.nblocks = units * g.nrhs;
    first[t] += g.nblocks;
    segs[t].push_back(g);
    cost[t].push_back(per_tile ? std::min(s->host.tz, s->host.n) + 3 : 1);
  }
  const size_t flat = segs[0].size(), bytes = sizeof(Segment) * (flat + segs[1].size());
  if (bytes > seg_cap_) return SHH_WORKSPACE_TOO_SMALL;
  Segment *dst = (Segment *)(seg_mem_ + (size_t)k * seg_cap_);
  for (int t = 0; t < (tall ? 2 : 1); ++t) {
    LaunchArgs &l = t ? *tall : la;
    l.segs = dst + (t ? flat : 0);
    l.nseg = int(segs[t].size());
    l.total = first[t];
    split_by_cost(segs[t], cost[t], l);
  }
  std::vector<Segment> &cur = segs[0];
  cur.insert(cur.end(), segs[1].begin(), segs[1].end());
  if (cur.empty()) return SHH_OK;
  auto &prev = host_segs_[k];
  const bool same = prev.size() == cur.size() && std::memcmp(prev.data(), cur.data(), bytes) == 0;
  if (!same) {
    SHH_HIP(hipMemcpyAsync(dst, cur.data(), bytes, hipMemcpyHostToDevice, st_));
    SHH_HIP(hipStreamSynchronize(st_));
    prev = cur;
  }
  return SHH_OK;
}

// Residual f - K x in FP64 (mode RES_INIT: x = 0), mean projection and the
// scalar update for the given slots.
int Solver::residual(const std::vector<Slot *> &slots, int mode) {
  if (slots.empty()) return SHH_OK;
  const int prec = slots[0]->host.prec;
  const bool all = mode != RES_RECOMPUTE;
  LaunchArgs la;
  int rc;
  if (mode != RES_INIT) {
    // apply the pending x update (and, mixed, move x into the FP64 accumulator)
    if ((rc = build(K_FOLD, slots, mode, true, la))) return rc;
    SHH_HIP(launch_fold(la, prec, st_));
  }
  LaunchArgs lr[2];
  if ((rc = build(K_RESID, slots, mode, all, lr[0], &lr[1]))) return rc;
  hipEvent_t e0 = nullptr;
  if (lr[0].total + lr[1].total > 0 && (rc = timed_begin(&e0))) return rc;
  SHH_HIP(launch_stencil_resid(lr[0], prec, prec == SHH_PREC_FP64 ? TILING_F64 : TILING_F64_TALL, st_));
  SHH_HIP(launch_stencil_resid(lr[1], prec, TILING_F64_TALL, st_));
  if ((rc = timed_end(e0, SHH_PROF_RESID64))) return rc;
  LaunchArgs ls;
  if ((rc = build(K_SCAL_RES, slots, mode, all, ls))) return rc;
  SHH_HIP(launch_scalar(ls, PH_MEAN, st_));
  if ((rc = build(K_FINISH, slots, mode, all, la))) return rc;
  SHH_HIP(launch_finish_resid(la, prec, st_));
  SHH_HIP(launch_scalar(ls, PH_RESID, st_));
  // a multigrid-preconditioned CG takes z = V r of the new residual: a
  // restart after the first and the final residual, the direction kept after
  // a replacement (reliable updates)
  for (Slot *s : slots) {
    s->mg_restart = true;
    s->mg_keep_dir = mode == RES_RECOMPUTE;
  }
  return SHH_OK;
}

int Solver::start(const std::vector<Slot *> &in, std::vector<Slot *> *failed) {
  if (in.empty()) return SHH_OK;
  const int prec = in[0]->host.prec;
  LaunchArgs la;
  int rc;
  // multigrid hierarchies first: their setup borrows the CG vector region
  std::vector<Slot *> mgs;
  for (Slot *s : in)
    if (s->opts.solver == SHH_SOLVER_MG) mgs.push_back(s);
  std::vector<int> rcs;
  if ((rc = mg_setup(mgs, st_, failed ? &rcs : nullptr))) return rc;
  std::vector<Slot *> slots;
  for (Slot *s : in) {
    bool ok = true;
    for (size_t i = 0; i < rcs.size(); ++i)
      if (mgs[i] == s && rcs[i] != SHH_OK) {
        s->finished = true;
        s->status = rcs[i];
        failed->push_back(s);
        ok = false;
      }
    if (ok) slots.push_back(s);
  }
  if (slots.empty()) return SHH_OK;
  if ((rc = build(K_ZERO, slots, 0, true, la))) return rc;
  SHH_HIP(launch_zero_vectors(la, prec, st_));
  for (Slot *s : slots) if (s->ev[1]) SHH_HIP(hipEventRecord(s->ev[1], st_));
  if ((rc = residual(slots, RES_INIT))) return rc;
  for (Slot *s : slots) {
    if (s->ev[2]) SHH_HIP(hipEventRecord(s->ev[2], st_));
    for (int r = 0; r < NRHS; ++r) s->state.active[r] = 1;  // refreshed at the next read-back
    s->launched = 0;
  }
  return SHH_OK;
}

Solver::~Solver() {
  resolve_events();
  for (hipEvent_t e : ev_pool_) (void)hipEventDestroy(e);
}

hipEvent_t Solver::get_event() {
  if (!ev_pool_.empty()) {
    hipEvent_t e = ev_pool_.back();
    ev_pool_.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Call only after the stream has been synchronized.
void Solver::resolve_events() {
  for (auto &tk : ev_timed_) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, tk.e0, tk.e1) == hipSuccess) profile_add(tk.kind, ms);
    ev_pool_.push_back(tk.e0);
    ev_pool_.push_back(tk.e1);
  }
  ev_timed_.clear();
}

int Solver::iterate(const std::vector<Slot *> &all, int iters) {
  if (all.empty()) return SHH_OK;
  std::vector<Slot *> slots, mgs;
  for (Slot *s : all) (s->opts.solver == SHH_SOLVER_MG ? mgs : slots).push_back(s);
  int rc;
  if (!mgs.empty() && (rc = iterate_mg(mgs, iters))) return rc;
  if (slots.empty()) return SHH_OK;
  const int prec = slots[0]->host.prec;
  LaunchArgs la_s[2];
  if ((rc = build(K_STENCIL, slots, 0, false, la_s[0], &la_s[1]))) return rc;
  LaunchArgs la_c;
  if ((rc = build(K_SCAL_IT, slots, 0, false, la_c))) return rc;
  for (int it = 0; it < iters; ++it) {
    hipEvent_t e0 = nullptr;
    if (la_s[0].total + la_s[1].total > 0 && (rc = timed_begin(&e0))) return rc;
    SHH_HIP(launch_stencil_pcg(la_s[0], prec, st_));  // the precision's first tiling has its index
    SHH_HIP(launch_stencil_pcg(la_s[1], TILING_F64_TALL, st_));
    if ((rc = timed_end(e0, SHH_PROF_CG_PASS))) return rc;
    SHH_HIP(launch_scalar(la_c, PH_ITER, st_));
    std::vector<Slot *> due;
    for (Slot *s : slots) {
      s->launched += 1;
      if (s->R > 0 && s->launched % s->R == 0) due.push_back(s);
    }
    if (!due.empty()) {
      if ((rc = residual(due, RES_RECOMPUTE))) return rc;
    }
  }
  return SHH_OK;
}

// Multigrid-preconditioned CG: one launch sequence per slot and iteration.
int Solver::iterate_mg(const std::vector<Slot *> &slots, int iters) {
  int rc;
  // voxel-level operator over all the given slots, one launch
  MgApply0 apply0 = [this](const std::vector<Slot *> &ss, int op) -> int {
    static const Kind kinds[3] = {K_MG_DIR, K_MG_PRE, K_MG_POST};
    static const int prof[3] = {SHH_PROF_MG_DIR, SHH_PROF_MG_STEP1, SHH_PROF_MG_LAST};
    if (op < SMG_DIR || op > SMG_POST) return SHH_INVALID_ARG;
    LaunchArgs la[2];
    int r;
    // segments of the load cases still running at the last read-back; the
    // kernels also skip those that stopped since
    if ((r = build(kinds[op], ss, 0, false, la[0], &la[1]))) return r;
    if (la[0].total + la[1].total == 0) return SHH_OK;
    hipEvent_t e0 = nullptr;
    if ((r = timed_begin(&e0))) return r;
    SHH_HIP(launch_stencil_mg(la[0], ss[0]->host.prec, op, st_));
    SHH_HIP(launch_stencil_mg(la[1], TILING_F64_TALL, op, st_));
    return timed_end(e0, prof[op]);
  };
  for (int it = 0; it < iters; ++it) {
    if ((rc = mg_iterate(slots, st_, this, apply0))) return rc;
    std::vector<Slot *> due;
    for (Slot *s : slots) {
      s->launched += 1;
      if (s->R > 0 && s->launched % s->R == 0) due.push_back(s);
    }
    if (!due.empty() && (rc = residual(due, RES_RECOMPUTE))) return rc;
  }
  return SHH_OK;
}

int Solver::timed_begin(hipEvent_t *e0) {
  *e0 = nullptr;
  if (!timing_ || !profile_on()) return SHH_OK;
  *e0 = get_event();
  if (*e0) SHH_HIP(hipEventRecord(*e0, st_));
  return SHH_OK;
}

int Solver::timed_end(hipEvent_t e0, int kind) {
  if (!e0) return SHH_OK;
  hipEvent_t e1 = get_event();
  if (!e1) {
    ev_pool_.push_back(e0);
    return SHH_OK;
  }
  SHH_HIP(hipEventRecord(e1, st_));
  ev_timed_.push_back({e0, e1, kind});
  return SHH_OK;
}

int Solver::read_states(const std::vector<Slot *> &slots) {
  for (Slot *s : slots)
    SHH_HIP(hipMemcpyAsync(&s->state, s->d_state, sizeof(CgState), hipMemcpyDeviceToHost, st_));
  SHH_HIP(hipStreamSynchronize(st_));
  resolve_events();
  return SHH_OK;
}

int Solver::sync() {
  SHH_HIP(hipStreamSynchronize(st_));
  resolve_events();
  return SHH_OK;
}

static bool all_inactive(const CgState &c) {
  for (int r = 0; r < NRHS; ++r)
    if (c.active[r]) return false;
  return true;
}

int Solver::final_check(const std::vector<Slot *> &slots) {
  if (slots.empty()) return SHH_OK;
  int rc;
  if ((rc = residual(slots, RES_FINAL))) return rc;
  for (Slot *s : slots) s->finals += 1;
  return read_states(slots);
}

int Solver::poll(const std::vector<Slot *> &slots, std::vector<Slot *> &done) {
  int rc;
  if ((rc = read_states(slots))) return rc;
  std::vector<Slot *> cand;
  for (Slot *s : slots)
    if (!s->finished && all_inactive(s->state)) cand.push_back(s);
  if (cand.empty()) return SHH_OK;
  for (Slot *s : cand) if (s->ev[3]) SHH_HIP(hipEventRecord(s->ev[3], st_));
  if ((rc = final_check(cand))) return rc;
  std::vector<Slot *> fin;
  for (Slot *s : cand) {
    if (!all_inactive(s->state) && s->finals < 8) {
      // true residual above rtol: resume.  Align the recompute schedule with
      // the device iteration count so that a design's arithmetic does not
      // depend on when the host happened to poll it.
      int m = 0;
      for (int r = 0; r < NRHS; ++r) m = std::max(m, s->state.iters[r]);
      s->launched = m;
      continue;
    }
    fin.push_back(s);
  }
  for (Slot *s : fin) {
    SHH_HIP(launch_energy(s->d_slot, s->host.nn, st_));
    if (s->ev[4]) SHH_HIP(hipEventRecord(s->ev[4], st_));
  }
  if (!fin.empty()) {
    if ((rc = read_states(fin))) return rc;
  }
  for (Slot *s : fin) {
    s->finished = true;
    int status = SHH_OK;
    for (int r = 0; r < NRHS; ++r) {
      if (s->state.status[r] == ST_BREAKDOWN) status = SHH_BREAKDOWN;
      else if (status == SHH_OK && s->state.status[r] != ST_CONVERGED) status = SHH_NOT_CONVERGED;
    }
    s->status = status;
    float a = 0.f;
    if (s->ev[0] && hipEventElapsedTime(&a, s->ev[0], s->ev[1]) == hipSuccess) s->ms[0] = a;
    if (s->ev[1] && hipEventElapsedTime(&a, s->ev[1], s->ev[2]) == hipSuccess) s->ms[1] = a;
    if (s->ev[2] && hipEventElapsedTime(&a, s->ev[2], s->ev[3]) == hipSuccess) s->ms[2] = a;
    if (s->ev[3] && hipEventElapsedTime(&a, s->ev[3], s->ev[4]) == hipSuccess) s->ms[3] = a;
    if (s->ev[0] && hipEventElapsedTime(&a, s->ev[0], s->ev[4]) == hipSuccess) s->ms[4] = a;
    done.push_back(s);
  }
  return SHH_OK;
}

void fill_result(const Slot &s, shh_result *out) {
  std::memset(out, 0, sizeof(*out));
  for (int i = 0; i < 36; ++i) out->CH[i] = s.state.C[i];
  out->vol_frac = s.state.V;
  out->t_used = s.state.t;
  for (int r = 0; r < NRHS; ++r) {
    out->iters[r] = s.state.iters[r];
    out->rel_res[r] = s.state.rel_true[r];
  }
  for (int i = 0; i < 5; ++i) out->ms[i] = s.ms[i];
  out->status = s.status;
  out->active_nodes = is_selective(s.opts.solver) ? s.sel_active_nodes : int32_t(s.host.nn);
}

}  // namespace shh
