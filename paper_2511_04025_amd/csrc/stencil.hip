// Matrix-free periodic stiffness operator q = K p, K = sum_e E_e P_e^T K_0 P_e
// (Sec. 4.1, Eq. (7)-(8)), for one load case per workgroup.
//
// A workgroup owns a TX x TY tile of nodes in the x-y plane (64 x 6 for FP32
// compute, 32 x 8 or 32 x 14 for FP64) and marches up a run of tz planes in z.  Per
// element layer it
//   1. stages the next node plane (tile + one-node periodic halo) in LDS,
//   2. forms, for each of the (TX+1)(TY+1) element columns, the Hadamard
//      coefficients of the element's 24 nodal values (x-y from the 2x2 node
//      block in LDS, z from the previous plane kept in registers),
//   3. applies E_e K_0 in that basis (hexop.hpp) and transforms back along z
//      (the half for the lower node plane completes it; the upper half is
//      carried to the next layer in registers),
//   4. transforms the lower node plane's share back to the four x-y corners,
//      exchanges them through LDS and sums four per output node.
// Thread t < TX*TY both stages and outputs interior node (t % TX, t / TX) of
// the tile; the ring of halo nodes around the tile is staged by the remaining
// threads (and, past those, by a second slot of the first threads).  Every
// global access is a coalesced x-row of one buffer resource; the periodic
// wrap is an index map on the halo only.
//
// Modes
//   PCG   : one whole Jacobi-PCG iteration of the load case per pass.  Pass j
//           reads r_{j-1}, q_{j-1}, p_{j-1} (set pcur) and, at every staged
//           node, forms
//             r_j = r_{j-1} - alpha q_{j-1},  z_j = D^-1 r_j,
//             p_j = z_j + beta p_{j-1}
//           with the alpha, beta left by the scalar kernel after pass j-1.
//           At owned nodes it writes r_j, p_j (other set) and
//           x_j = x_{j-1} + alpha p_{j-1}, and sums r_j . z_j and r_j . r_j;
//           at the outputs it writes q_j = K p_j (other set) and sums
//           p_j . q_j, q_j . z_j and q_j . D^-1 q_j (all sums FP64).
//           The scalar kernel turns these into alpha_j and, by expanding
//           (r_j - alpha_j q_j) . D^-1 (r_j - alpha_j q_j), the next rho and
//           beta: standard PCG whose x, r update is carried into the next
//           pass instead of a pass of its own.  Both p buffers and both q
//           buffers are zeroed when a solve starts and stay finite, so
//           alpha = beta = 0 needs no special case.
//   RESID : FP64 arithmetic on the FP64 solution x: r = -K (x + chi^k), i.e.
//           f - K x with f = -sum_e E_e P_e^T K_0 chi^k added at the element;
//           stored in the vector precision into the current r, with FP64
//           sums of r for the mean projection.  Flag 0 (initial) treats x as
//           zero.
//   APPLY : plain q = K p (component entry point and tests).
#include <type_traits>

#include "common.hpp"
#include "hexop.hpp"
#include "kernels.hpp"

namespace shh {

enum { MODE_PCG = 0, MODE_RESID = 1, MODE_APPLY = 2, MODE_MGDIR = 3, MODE_MGPRE = 4, MODE_MGPOST = 5 };

// Waves per SIMD that the compiler aims at.  Two workgroups share a CU up to 128
// registers (FP32, four waves; the post-smoothing pass keeps two values in scratch
// for it) or 168 (FP64, three).  The FP64 pre-smoothing pass fits when told to; the
// FP64 direction and post-smoothing passes would spill (a 24^3 FP64 solve 27.4
// instead of 25.5 ms).
template <typename TC, int MODE>
constexpr int WPE = sizeof(TC) == 4 ? 4 : (MODE == MODE_MGPRE ? 3 : 1);
template <typename TC, typename TS, int MODE, bool TALL = false>
__global__ __launch_bounds__((Tile<TC, TALL>::THREADS))
    __attribute__((amdgpu_waves_per_eu(WPE<TC, MODE>)))
void stencil_kernel(LaunchArgs la) {
  // tile geometry of this compute precision
  using TT = Tile<TC, TALL>;
  constexpr int TX = TT::X, TY = TT::Y, HX = TT::HX, HY = TT::HY, EXC = TT::EXC, EYC = TT::EYC;
  constexpr int NHALO = TT::NHALO, NELEMC = TT::NELEMC, STENCIL_THREADS = TT::THREADS;
  constexpr int NINT = TT::NINT, NRING = TT::NRING;
  constexpr int TW = tiling_of<TC, TALL>();
  __shared__ TC nbuf[2][3][NHALO];
  __shared__ TC ebuf[2][12][NELEMC];
  __shared__ TC mbuf[2][NHALO];  // element moduli, by the halo slot of the element's lower corner
  __shared__ double red[(MODE == MODE_PCG ? 5 : (MODE == MODE_RESID ? 3 : 2)) * 16];
  // post-smoothing: one plane of the coarse correction around the tile
  constexpr int CXC = TX / 2 + 2, CYC = TY / 2 + 2, NCO = MODE == MODE_MGPOST ? 3 * CXC * CYC : 1;
  constexpr int CPT = (NCO + STENCIL_THREADS - 1) / STENCIL_THREADS;
  __shared__ TC cbuf[NCO];
  // FP32 pre-smoothing: a plane of the residual, summed over z, in a margin of
  // zeros (one before, two behind)
  constexpr bool RESTR = MODE == MODE_MGPRE && sizeof(TC) == 4;
  constexpr int RX = TX + 3, RY = TY + 3, RCX = TX / 2 + 1, RCY = TY / 2 + 1, NRC = 3 * RCX * RCY;
  static_assert(!RESTR || NRC <= STENCIL_THREADS, "one coarse value a thread");
  __shared__ TC rbuf[RESTR ? 3 * RX * RY : 1];

  Work w;
  if (!decode_work(la, w)) return;
  const SHH_CONST SlotDev *s = to_const(w.slot);
  const SHH_CONST CgState *st = to_const(s->st);
  const int rhs = w.rhs;
  // load cases whose CG has stopped are skipped (Sec. 4.2.2: per-right-hand-
  // side convergence); the multigrid passes likewise
  if ((MODE == MODE_PCG || MODE >= MODE_MGDIR) && !st->active[rhs]) return;
  if (MODE == MODE_RESID) {
    if (w.flag == RES_RECOMPUTE && !st->active[rhs]) return;
    if (w.flag == RES_FINAL && !(st->ff[rhs] > s->ffloor * s->ffloor)) return;
  }
  // an operator call on moduli that its caller will refuse leaves the output alone
  if (MODE == MODE_APPLY || (MODE == MODE_RESID && w.flag == RES_LOAD)) {
    const double emax = st->Emax;
    if (!(emax > 0.0 && emax < INFINITY)) return;
  }

  // n <= 512: every byte offset into one load case's [3][n^3] vector fits in
  // 32 bits.  Per-lane offsets are fixed per thread; plane and component
  // offsets are wave-uniform scalars.
  const int n = s->n;
  const uint32_t plane = (uint32_t)n * (uint32_t)n;
  const long long nn = s->nn;
  const int tile = w.tile;
  const int tix = tile % s->tiles_x[TW];
  const int tiy = (tile / s->tiles_x[TW]) % s->tiles_y[TW];
  const int tiz = tile / (s->tiles_x[TW] * s->tiles_y[TW]);
  const int x0 = tix * TX, y0 = tiy * TY, z0 = tiz * s->tz;
  const int z1 = min(z0 + s->tz, n);
  const int tid = threadIdx.x;

  using TL = typename std::conditional<MODE == MODE_RESID, double, TS>::type;
  constexpr uint32_t SL = sizeof(TL), SS = sizeof(TS), SC = sizeof(TC);

  // element-column role.  In FP32 every thread runs the element work (the last
  // wave is there anyway) and only its stores are masked: values defined under a
  // branch and carried around the loop cost a register copy each, a fifth of the
  // loop's vector instructions.  The FP64 kernels and the Jacobi CG pass keep the
  // branch: without it their registers pass the limit for two workgroups on a CU.
  constexpr bool BRANCH = sizeof(TC) == 8 || MODE == MODE_PCG;
  const bool is_elem = tid < NELEMC;
  const int ecol = is_elem ? tid : NELEMC - 1;
  const int ecx = ecol % EXC, ecy = ecol / EXC;
  // output role (also the owner of the node in the PCG update)
  const int ox = tid % TX, oy = tid / TX;
  const bool is_out = tid < NINT && x0 + ox < n && y0 + oy < n;
  const uint32_t ooff = ((uint32_t)(y0 + oy) * n + (uint32_t)(x0 + ox)) * SS;
  // staging role: slot 0 of thread t < NINT is its own interior node; ring
  // nodes fill the remaining slot-0 threads and then slot 1 of the first ones
  // The element moduli of a layer are staged with a node plane: element
  // column (ecx, ecy) is the voxel whose lower corner is halo node (ecx, ecy),
  // so the thread staging that node loads the voxel's E_e at the same offset
  // (hel; without the branch the last row and column ride along).  Keeping every global load in the staging batch means the element
  // work never waits on the memory counter, which retires in issue order.
  bool hval[2], hel[2];
  int hslot[2];
  uint32_t hoS[2], hoL[2], hoC[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    int h;
    if (k == 0 && tid < NINT) {
      h = (oy + 1) * HX + ox + 1;
      hval[k] = true;
    } else {
      const int j = k == 0 ? tid - NINT : tid + STENCIL_THREADS - NINT;
      hval[k] = j < NRING;
      h = hval[k] ? ring_h<HX, HY>(j) : 0;
    }
    hslot[k] = h;
    const int hx = h % HX, hy = h / HX;
    const uint32_t o = (uint32_t)wrapi(y0 - 1 + hy, n) * n + (uint32_t)wrapi(x0 - 1 + hx, n);
    hoS[k] = o * SS;
    hoL[k] = o * SL;
    hoC[k] = o * SC;
    hel[k] = hval[k] && hx < EXC && hy < EYC;
  }

  // every thread's first slot holds a node
  static_assert(STENCIL_THREADS <= NHALO, "slot 0 is never empty");
  auto stages = [&](int k) { return !BRANCH && k == 0 ? true : hval[k]; };

  const SHH_CONST TC *kop;
  if constexpr (sizeof(TC) == 8) kop = (const SHH_CONST TC *)s->kop64;
  else kop = (const SHH_CONST TC *)s->kop32;
  // one resource for the moduli and, in the CG pass, D^-1 behind them (the two
  // arrays are adjacent in the slot, D^-1 at byte offset dOff)
  const char *Ebase;
  if constexpr (sizeof(TC) == 8) Ebase = (const char *)s->E64;
  else Ebase = (const char *)s->E32;
  constexpr bool MGF = MODE >= MODE_MGPRE;  // a smoothing step fused behind the operator
  constexpr bool WITH_D = MODE == MODE_PCG || MGF;
  const uint32_t dOff = WITH_D ? (uint32_t)((const char *)s->Dinv - Ebase) : 0u;
  const rsrc_t rE = make_rsrc(Ebase, WITH_D ? (uint64_t)dOff + (uint64_t)nn * SS : (uint64_t)nn * SC);

  // component c of a load case's vector starts c * n^3 elements in
  const uint32_t cS[3] = {0u, (uint32_t)nn * SS, 2u * (uint32_t)nn * SS};
  const uint32_t cL[3] = {0u, (uint32_t)nn * SL, 2u * (uint32_t)nn * SL};
  const long long vbase = (long long)rhs * 3 * nn;
  const uint64_t vbytesS = 3ull * nn * SS, vbytesL = 3ull * nn * SL;
  // PCG: rA = r_{j-1}, rB = q_{j-1}, rC = p_{j-1}; rR, rQ, rP the new set; rX
  // RESID: rA = FP64 x, rQ = current r.  APPLY: rA = p, rQ = q (or the pair the flag names).
  // MGDIR (the multigrid CG's direction pass): rA = z (mgd), rC = p_{j-1}, rP = p_j, rQ = q, rX: the
  // x update of the iteration before (x += alpha p_{j-1}) rides along, since p_{j-1} is read anyway.
  // The two smoothing passes (q = K v is consumed, not stored; b = r[pc] before, r[pc ^ 1] after PRE):
  //   PRE:  staged b' = b - alpha q (the CG update) as d0 = D b' / theta;  r = b' - K d0 (the
  //         residual the restriction takes) -> q[1] (FP32: its restriction's shares), b' -> the
  //         other r buffer
  //   POST: staged x = D b' / theta + P x_c, P the interpolation from level 1;
  //         z = x + D (b' - K x) / theta -> mgd, partials b' . z, b' . b'
  // Neither d0 nor x is ever stored: each is formed again from b'.
  rsrc_t rA, rB, rC, rR, rQ, rP, rX, rD;
  TC alpha = TC(0), beta = TC(0);
  TC ith = TC(0);
  if constexpr (MGF) {
    ith = (TC)s->mgc;
    const int pc = st->pcur[rhs];
    if constexpr (MODE == MODE_MGPRE) {
      alpha = (TC)st->alpha[rhs];
      rA = make_rsrc((const TS *)s->r[pc] + vbase, vbytesS);
      rB = make_rsrc((const TS *)s->q[0] + vbase, vbytesS);
      rX = make_rsrc((const TS *)s->r[pc ^ 1] + vbase, vbytesS);
      rR = make_rsrc((const TS *)s->q[1] + vbase, vbytesS);
    } else {
      const uint64_t cnn = (uint64_t)nn >> 3;
      rA = make_rsrc((const TS *)s->r[pc ^ 1] + vbase, vbytesS);
      rB = make_rsrc((const TS *)s->mgxc + (long long)rhs * 3 * cnn, 3ull * cnn * SS);
      rX = make_rsrc((const TS *)s->mgd + vbase, vbytesS);
    }
  } else if constexpr (MODE == MODE_MGDIR) {
    const int pc = st->mgpar[rhs];
    rA = make_rsrc((const TS *)s->mgd + vbase, vbytesS);
    rC = make_rsrc((const TS *)s->p[pc] + vbase, vbytesS);
    rP = make_rsrc((const TS *)s->p[pc ^ 1] + vbase, vbytesS);
    rQ = make_rsrc((const TS *)s->q[0] + vbase, vbytesS);
    rX = make_rsrc((const TS *)s->x + vbase, vbytesS);
    alpha = (TC)st->alpha[rhs];
    beta = (TC)st->beta[rhs];
  } else if constexpr (MODE == MODE_PCG) {
    const int pc = st->pcur[rhs];
    rA = make_rsrc((const TS *)s->r[pc] + vbase, vbytesS);
    rB = make_rsrc((const TS *)s->q[pc] + vbase, vbytesS);
    rC = make_rsrc((const TS *)s->p[pc] + vbase, vbytesS);
    rR = make_rsrc((const TS *)s->r[pc ^ 1] + vbase, vbytesS);
    rQ = make_rsrc((const TS *)s->q[pc ^ 1] + vbase, vbytesS);
    rP = make_rsrc((const TS *)s->p[pc ^ 1] + vbase, vbytesS);
    rX = make_rsrc((const TS *)s->x + vbase, vbytesS);
    alpha = (TC)st->alpha[rhs];
    beta = (TC)st->beta[rhs];
  } else if constexpr (MODE == MODE_RESID) {
    rA = make_rsrc(s->x64 + vbase, vbytesL);
    rQ = make_rsrc((const TS *)s->r[st->pcur[rhs]] + vbase, vbytesS);
  } else {
    rA = make_rsrc((const TS *)s->p[0] + vbase, vbytesL);
    rQ = make_rsrc((const TS *)s->q[0] + vbase, vbytesS);
  }
  const bool zero_x = (MODE == MODE_RESID) && (w.flag == RES_INIT || w.flag == RES_LOAD);

  // FP64 partial sums: PCG r.z, r.r, p.q, q.z, q.D^-1 q; RESID sums of r
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  // owned-node values kept from staging to output (two steps later), by
  // parity of the step that staged them: z, D^-1 and p of the node
  TC own_z[2][3], own_p[2][3], own_d[2];
  // pending update of the CG: nothing to apply after a (re)start
  const bool upd = (MODE == MODE_MGDIR || MODE == MODE_MGPRE) && alpha != TC(0);

  // Post-smoothing, the coarse correction at the staged nodes: fine node x
  // takes the mean of the coarse nodes floor(x / 2) and floor((x + 1) / 2) per
  // axis (the same node twice where x is even).  z0 is even, so the planes
  // alternate odd, even, ... from z0 - 1; an odd plane 2 Z + 1 brings in coarse
  // plane Z + 1, which is loaded two steps ahead (one value per thread), put in
  // LDS one step ahead and kept interpolated in x-y (cxy) for the even plane
  // after it.  Interpolating from global memory at the time of use instead
  // costs 24 registers in flight.
  const int nc = n >> 1;
  const uint32_t cplane = (uint32_t)nc * (uint32_t)nc;
  TC cxy[2][3], raw_cc[CPT];
  uint32_t coff[CPT];
  int cpos[2][4];
  auto issue_c = [&](int Z) {
    if constexpr (MODE == MODE_MGPOST) {
      const uint32_t pz = (uint32_t)wrap1(Z, nc) * cplane * SS;
#pragma unroll
      for (int k = 0; k < CPT; ++k)
        if (tid + k * STENCIL_THREADS < NCO) raw_cc[k] = (TC)bload<TS>(rB, coff[k], pz);
    }
  };
  auto write_c = [&]() {
    if constexpr (MODE == MODE_MGPOST) {
#pragma unroll
      for (int k = 0; k < CPT; ++k)
        if (tid + k * STENCIL_THREADS < NCO) cbuf[tid + k * STENCIL_THREADS] = raw_cc[k];
    }
  };

  // ---- plane staging, split into issue (loads into registers), finish
  //      (combine, store to LDS) and commit (store owned values) so that the
  //      loads of a plane are in flight during the previous plane's element
  //      work.
  //      Node planes z0-1 .. z1 are touched, so a single wrap suffices.
  TL raw_a[2][3];
  TS raw_b[2][3], raw_c[2][3], raw_d[2], raw_x[3];
  TC raw_e[2];
  // node plane z, and the element layer z - 1 below it
  auto issue = [&](int z) {
    const uint32_t pz = (uint32_t)wrap1(z, n) * plane;
    const uint32_t pe = (uint32_t)wrap1(z - 1, n) * plane;
    const bool ownz = z >= z0 && z < z1;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!stages(k)) continue;
      if (!BRANCH || hel[k]) raw_e[k] = bload<TC>(rE, hoC[k], pe * SC);
      if constexpr (MODE == MODE_PCG) {
        raw_d[k] = bload<TS>(rE, hoS[k], dOff + pz * SS);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          raw_a[k][c] = bload<TS>(rA, hoS[k], pz * SS + cS[c]);
          raw_b[k][c] = bload<TS>(rB, hoS[k], pz * SS + cS[c]);
          raw_c[k][c] = bload<TS>(rC, hoS[k], pz * SS + cS[c]);
        }
        if (k == 0 && is_out && ownz) {
#pragma unroll
          for (int c = 0; c < 3; ++c) raw_x[c] = bload<TS>(rX, hoS[0], pz * SS + cS[c]);
        }
      } else if constexpr (MODE == MODE_RESID) {
#pragma unroll
        for (int c = 0; c < 3; ++c) raw_a[k][c] = zero_x ? 0.0 : bload<TL>(rA, hoL[k], pz * SL + cL[c]);
      } else if constexpr (MGF) {
        raw_d[k] = bload<TS>(rE, hoS[k], dOff + pz * SS);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          raw_a[k][c] = bload<TS>(rA, hoS[k], pz * SS + cS[c]);
          if constexpr (MODE == MODE_MGPRE) raw_b[k][c] = upd ? bload<TS>(rB, hoS[k], pz * SS + cS[c]) : TS(0);
        }
      } else if constexpr (MODE == MODE_MGDIR) {
        // beta = 0 starts a new direction: the old one is not read
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          raw_a[k][c] = bload<TS>(rA, hoS[k], pz * SS + cS[c]);
          raw_c[k][c] = upd || beta != TC(0) ? bload<TS>(rC, hoS[k], pz * SS + cS[c]) : TS(0);
        }
        if (k == 0 && is_out && ownz && upd) {
#pragma unroll
          for (int c = 0; c < 3; ++c) raw_x[c] = bload<TS>(rX, hoS[0], pz * SS + cS[c]);
        }
      } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) raw_a[k][c] = bload<TL>(rA, hoL[k], pz * SL + cL[c]);
      }
    }
  };
  // the owned node's new r, p, x, written by commit() after the next plane's
  // loads are issued (so that waiting for those loads never waits for these
  // stores: the memory counter retires in issue order)
  TS out_r[3], out_p[3], out_x[3];
  auto commit = [&](int z) {
    if constexpr (MODE == MODE_PCG) {
      const uint32_t pz = (uint32_t)wrap1(z, n) * plane;
      const bool ownz = z >= z0 && z < z1;
      if (is_out && ownz) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const uint32_t so = pz * SS + cS[c];
          bstore<TS>(out_r[c], rR, hoS[0], so);
          bstore<TS>(out_p[c], rP, hoS[0], so);
          bstore<TS>(out_x[c], rX, hoS[0], so);
        }
      }
    } else if constexpr (MODE == MODE_MGDIR) {
      const uint32_t pz = (uint32_t)wrap1(z, n) * plane;
      const bool ownz = z >= z0 && z < z1;
      if (is_out && ownz) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          bstore<TS>(out_p[c], rP, hoS[0], pz * SS + cS[c]);
          if (upd) bstore<TS>(out_x[c], rX, hoS[0], pz * SS + cS[c]);
        }
      }
    } else if constexpr (MODE == MODE_MGPRE) {
      const uint32_t pz = (uint32_t)wrap1(z, n) * plane;
      const bool ownz = z >= z0 && z < z1;
      if (is_out && ownz) {
#pragma unroll
        for (int c = 0; c < 3; ++c) bstore<TS>(out_x[c], rX, hoS[0], pz * SS + cS[c]);
      }
    }
  };
  auto finish = [&](int z, auto bc) {
    constexpr int b = decltype(bc)::value;
    const uint32_t pz = (uint32_t)wrap1(z, n) * plane;
    const bool ownz = z >= z0 && z < z1;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!stages(k)) continue;
      if (!BRANCH || hel[k]) mbuf[b][hslot[k]] = raw_e[k];
      if constexpr (MODE == MODE_PCG) {
        const TC dk = (TC)raw_d[k];
        TC rn[3], zn[3], pn[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          rn[c] = (TC)raw_a[k][c] - alpha * (TC)raw_b[k][c];
          zn[c] = dk * rn[c];
          pn[c] = beta * (TC)raw_c[k][c] + zn[c];
          nbuf[b][c][hslot[k]] = pn[c];
        }
        if (k == 0 && (!BRANCH || (is_out && ownz))) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            out_r[c] = (TS)rn[c];
            out_p[c] = (TS)pn[c];
            out_x[c] = (TS)((TC)raw_x[c] + alpha * (TC)raw_c[0][c]);
            own_z[b][c] = zn[c];
            own_p[b][c] = pn[c];
          }
          own_d[b] = dk;
          if (is_out && ownz) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const double r64 = (double)rn[c];
              acc[0] += r64 * (double)zn[c];
              acc[1] += r64 * r64;
            }
          }
        }
      } else if constexpr (MGF) {
        const TC dk = (TC)raw_d[k] * ith;
        TC bv[3], v[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          bv[c] = (TC)raw_a[k][c];
          if constexpr (MODE == MODE_MGPRE) bv[c] -= alpha * (TC)raw_b[k][c];
          v[c] = dk * bv[c];
        }
        if constexpr (MODE == MODE_MGPOST) {
          if constexpr (b == 0) {  // odd plane: the coarse plane above it comes in
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const TC *cb = cbuf + c * CXC * CYC;
              const TC up = TC(0.25) * ((cb[cpos[k][0]] + cb[cpos[k][1]]) + (cb[cpos[k][2]] + cb[cpos[k][3]]));
              v[c] += TC(0.5) * (cxy[k][c] + up);
              cxy[k][c] = up;
            }
          } else {
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] += cxy[k][c];
          }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) nbuf[b][c][hslot[k]] = v[c];
        if (k == 0 && (!BRANCH || (is_out && ownz))) {
          // own_p: the staged value, own_z: b'
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            own_p[b][c] = v[c];
            own_z[b][c] = bv[c];
            out_x[c] = (TS)bv[c];
          }
          own_d[b] = dk;
        }
      } else if constexpr (MODE == MODE_MGDIR) {
        TC pn[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          pn[c] = (TC)raw_a[k][c] + beta * (TC)raw_c[k][c];
          nbuf[b][c][hslot[k]] = pn[c];
        }
        if (k == 0 && (!BRANCH || (is_out && ownz))) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            out_p[c] = (TS)pn[c];
            out_x[c] = (TS)((TC)raw_x[c] + alpha * (TC)raw_c[0][c]);
            own_p[b][c] = pn[c];
          }
        }
      } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) nbuf[b][c][hslot[k]] = (TC)raw_a[k][c];
      }
    }
  };
  // x-y Hadamard coefficients of the 2x2 node block of this element column
  auto xy_hadamard = [&](auto bc, TC (&A)[3][4]) {
    constexpr int b = decltype(bc)::value;
    const int i00 = ecy * HX + ecx;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const TC p00 = nbuf[b][c][i00], p10 = nbuf[b][c][i00 + 1];
      const TC p01 = nbuf[b][c][i00 + HX], p11 = nbuf[b][c][i00 + HX + 1];
      const TC sx0 = p00 + p10, dx0 = p10 - p00, sx1 = p01 + p11, dx1 = p11 - p01;
      A[c][0] = sx0 + sx1;
      A[c][1] = dx0 + dx1;
      A[c][2] = sx1 - sx0;
      A[c][3] = dx1 - dx0;
    }
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;

  // Values carried from one element layer to the next: the x-y Hadamard
  // coefficients of the lower node plane (A) and the upper-plane half of the
  // layer below (Bc).
  TC A[3][4], Bc[3][4];

  // prologue: planes z0-1 and z0 staged, plane z0+1 in flight
  if constexpr (MODE == MODE_MGPOST) {
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int i = tid + k * STENCIL_THREADS, r = i % (CXC * CYC);
      coff[k] = (((uint32_t)(i / (CXC * CYC)) * nc) * cplane + (uint32_t)wrapi(y0 / 2 - 1 + r / CXC, nc) * nc +
                 (uint32_t)wrapi(x0 / 2 - 1 + r % CXC, nc)) * SS;
    }
    issue_c(z0 / 2);
    // coarse plane z0 / 2 - 1 straight from memory, once per workgroup
    const uint32_t pz = (uint32_t)wrap1(z0 / 2 - 1, nc) * cplane * SS;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      if (!stages(k)) continue;
      const int hx = hslot[k] % HX, hy = hslot[k] / HX;
      const int cx[2] = {(hx + 1) >> 1, (hx >> 1) + 1}, cy[2] = {(hy + 1) >> 1, (hy >> 1) + 1};
      TC v[4][3];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        cpos[k][j] = cy[j >> 1] * CXC + cx[j & 1];
        const uint32_t o = ((uint32_t)wrapi(y0 / 2 - 1 + cy[j >> 1], nc) * nc +
                            (uint32_t)wrapi(x0 / 2 - 1 + cx[j & 1], nc)) * SS;
#pragma unroll
        for (int c = 0; c < 3; ++c) v[j][c] = (TC)bload<TS>(rB, o, pz + (uint32_t)c * cplane * nc * SS);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) cxy[k][c] = TC(0.25) * ((v[0][c] + v[1][c]) + (v[2][c] + v[3][c]));
    }
    write_c();
  }
  // Pre-smoothing, the restriction: a workgroup sums its own nodes' share of
  // the coarse right-hand side P^T r (coarse planes z0 / 2 .. z1 / 2, RCX x RCY
  // nodes of each, the last ones shared with the next workgroup) and stores it
  // where the residual itself went, [tile][coarse plane][3][RCY][coarse columns];
  // mg_gather_kernel adds the shares.  Over z in registers: an odd plane
  // completes coarse plane Z and starts Z + 1; over x and y from rbuf.  The
  // residual's 12 bytes a node and load case are neither written nor read back
  // by a restriction kernel: one 128^3 design, this pass 149 -> 134 us and the
  // restriction 42 -> 16.  (FP64 has no registers left for it.)
  TC zac[3] = {TC(0), TC(0), TC(0)};
  const int rcols = min(TX, n) / 2 + 1;
  const int rc = tid / (RCX * RCY), ry = (tid / RCX) % RCY, rx = tid % RCX;
  const uint32_t rplane = 3u * RCY * (uint32_t)rcols * SS;
  const uint32_t roff =
      (uint32_t)tile * (uint32_t)(s->tz / 2 + 1) * rplane + ((uint32_t)((rc * RCY + ry) * rcols) + rx) * SS;
  auto restrict_store = [&](int Z) {  // coarse plane Z of the run
    if constexpr (RESTR) {
      if (tid < NRC && rx < rcols) {
        const TC *rb = rbuf + (rc * RY + 2 * ry) * RX + 2 * rx;
        auto row = [&](int y) { return rb[y * RX + 1] + TC(0.5) * (rb[y * RX] + rb[y * RX + 2]); };
        bstore<TS, 0>((TS)(row(1) + TC(0.5) * (row(0) + row(2))), rR, roff, (uint32_t)Z * rplane);
      }
    }
  };
  if constexpr (RESTR) {
    for (int i = tid; i < 3 * RX * RY; i += STENCIL_THREADS) rbuf[i] = TC(0);
  }
  issue(z0 - 1);
  if constexpr (MODE == MODE_MGPOST) __syncthreads();
  finish(z0 - 1, B0{});
  issue_c(z0 / 2 + 1);
  issue(z0);
  commit(z0 - 1);
  __syncthreads();
  if (!BRANCH || is_elem) {
    xy_hadamard(B0{}, A);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int m = 0; m < 4; ++m) Bc[c][m] = TC(0);
  }
  finish(z0, B1{});
  write_c();
  const int S = z1 - z0 + 1;  // element layers z0-1 .. z1-1
  if (S > 1) issue(z0 + 1);
  commit(z0);
  __syncthreads();

  // one element layer: kk = z0 - 1 + sl lies between node planes kk and kk+1;
  // the layer's node planes sit in nbuf[b] and nbuf[b ^ 1] with b = sl & 1
  auto step = [&](const int sl, auto bc) {
    constexpr int b = decltype(bc)::value;
    constexpr int bn = b ^ 1;
    using BN = std::integral_constant<int, bn>;
    const int kk = z0 - 1 + sl;
    // the owned values of output plane kk (staged two steps ago, same parity)
    // before this step's staging replaces them
    TC oz[3], op[3], od = TC(0);
    if constexpr (MODE == MODE_PCG) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        oz[c] = own_z[b][c];
        op[c] = own_p[b][c];
      }
      od = own_d[b];
    } else if constexpr (MODE == MODE_MGDIR) {
#pragma unroll
      for (int c = 0; c < 3; ++c) op[c] = own_p[b][c];
    } else if constexpr (MGF) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        op[c] = own_p[b][c];
        oz[c] = own_z[b][c];
      }
      od = own_d[b];
    }
    if (!BRANCH || is_elem) {
      TC An[3][4];
      xy_hadamard(BN{}, An);
      // layer kk's modulus was staged with node plane kk+1
      const TC e = mbuf[bn][ecy * HX + ecx];
      TC h[3][8], y[3][8];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        h[c][0] = TC(0);  // rigid mode: not read by hex_unit
#pragma unroll
        for (int m = 1; m < 4; ++m) h[c][m] = A[c][m] + An[c][m];
#pragma unroll
        for (int m = 0; m < 4; ++m) h[c][m + 4] = An[c][m] - A[c][m];
      }
      if constexpr (MODE == MODE_RESID) add_chi_any<TC>(rhs, h);
      // lower node plane kk: this layer's lower half completes the upper half
      // carried from the layer below (Bc); its four x-y corners go to LDS
      // (y[c][0] == 0)
      auto corners = [&](int c, TC L0, TC L1, TC L2, TC L3) {
        const TC u0 = L0 - L1, u1 = L0 + L1, v0 = L2 - L3, v1 = L2 + L3;
        ebuf[b][c * 4 + 0][tid] = u0 - v0;
        ebuf[b][c * 4 + 1][tid] = u1 - v1;
        ebuf[b][c * 4 + 2][tid] = u0 + v0;
        ebuf[b][c * 4 + 3][tid] = u1 + v1;
      };
      if constexpr (BRANCH) {
        hex_apply<TC>(kop, h, y, e);
        if (sl > 0) {
#pragma unroll
          for (int c = 0; c < 3; ++c)
            corners(c, Bc[c][0] - y[c][4], Bc[c][1] + (y[c][1] - y[c][5]), Bc[c][2] + (y[c][2] - y[c][6]),
                    Bc[c][3] + (y[c][3] - y[c][7]));
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          Bc[c][0] = y[c][4];
#pragma unroll
          for (int m = 1; m < 4; ++m) Bc[c][m] = y[c][m] + y[c][m + 4];
        }
      } else {
        // the modulus scales the halves in the same multiply-add
        hex_unit<TC>(kop, h, y);
        TC L[3][4];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          L[c][0] = Bc[c][0] - e * y[c][4];
          Bc[c][0] = e * y[c][4];
#pragma unroll
          for (int m = 1; m < 4; ++m) {
            L[c][m] = Bc[c][m] + e * (y[c][m] - y[c][m + 4]);
            Bc[c][m] = e * (y[c][m] + y[c][m + 4]);
          }
        }
        if (sl > 0 && is_elem) {
#pragma unroll
          for (int c = 0; c < 3; ++c) corners(c, L[c][0], L[c][1], L[c][2], L[c][3]);
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int m = 0; m < 4; ++m) A[c][m] = An[c][m];
    }
    // stage node plane kk+2 (its loads were issued a step ago), issue kk+3
    if (sl + 1 < S) finish(z0 + sl + 1, bc);
    if constexpr (b == 0) issue_c((z0 + sl + 4) / 2);  // the upper coarse plane of z0 + sl + 3
    else write_c();
    if (sl + 2 < S) issue(z0 + sl + 2);
    if (sl + 1 < S) commit(z0 + sl + 1);
    __syncthreads();
    if (sl > 0 && is_out) {
      // node (x0+ox, y0+oy, kk) is corner (ax, ay) of element column
      // (ox + 1 - ax, oy + 1 - ay)
      const int e00 = (oy + 1) * EXC + ox + 1;
      TC qv[3];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        qv[c] = (ebuf[b][c * 4 + 0][e00] + ebuf[b][c * 4 + 1][e00 - 1]) +
                (ebuf[b][c * 4 + 2][e00 - EXC] + ebuf[b][c * 4 + 3][e00 - EXC - 1]);
      const uint32_t pk = (uint32_t)kk * plane * SS;
      if constexpr (MODE == MODE_PCG) {
        const double d64 = (double)od;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          bstore<TS>((TS)qv[c], rQ, ooff, pk + cS[c]);
          const double q64 = (double)qv[c];
          acc[2] += (double)op[c] * q64;
          acc[3] += (double)oz[c] * q64;
          acc[4] += d64 * q64 * q64;
        }
      } else if constexpr (MODE == MODE_MGDIR) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          bstore<TS>((TS)qv[c], rQ, ooff, pk + cS[c]);
          acc[0] += (double)op[c] * (double)qv[c];
        }
      } else if constexpr (MODE == MODE_MGPRE) {
        // oz = b'
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const TC rv = oz[c] - qv[c];
          if constexpr (!RESTR) bstore<TS>((TS)rv, rR, ooff, pk + cS[c]);
          else if constexpr (b == 1) zac[c] += rv;  // even plane
          else {
            rbuf[(c * RY + oy + 1) * RX + ox + 1] = zac[c] + TC(0.5) * rv;
            zac[c] = TC(0.5) * rv;
          }
        }
      } else if constexpr (MODE == MODE_MGPOST) {
        // op = x, oz = b', od = D / theta
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const TC zv = op[c] + od * (oz[c] - qv[c]);
          bstore<TS>((TS)zv, rX, ooff, pk + cS[c]);
          const double b64 = (double)oz[c];
          acc[0] += b64 * (double)zv;
          acc[1] += b64 * b64;
        }
      } else if constexpr (MODE == MODE_RESID) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const TS rv = (TS)(-qv[c]);
          bstore<TS>(rv, rQ, ooff, pk + cS[c]);
          acc[c] += (double)rv;
        }
      } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) bstore<TS>((TS)qv[c], rQ, ooff, pk + cS[c]);
      }
    }
    // the plane written two barriers ago (an odd plane again writes rbuf after
    // the next one)
    if constexpr (RESTR && b == 1) {
      if (sl > 1) restrict_store((sl - 3) / 2);
    }
  };
  int sl = 0;
  for (; sl + 1 < S; sl += 2) {
    step(sl, B0{});
    step(sl + 1, B1{});
  }
  if (sl < S) step(sl, B0{});
  if constexpr (RESTR) {  // the last whole coarse plane and the share of the one above
    __syncthreads();
    restrict_store((z1 - z0) / 2 - 1);
    __syncthreads();
    if (is_out) {
#pragma unroll
      for (int c = 0; c < 3; ++c) rbuf[(c * RY + oy + 1) * RX + ox + 1] = zac[c];
    }
    __syncthreads();
    restrict_store((z1 - z0) / 2);
  }

  // workgroup partials only; the scalar kernel that follows reduces them
  double *parts = w.slot->partials + ((long long)rhs * s->maxparts + tile) * PSTRIDE;
  if constexpr (MODE == MODE_PCG) {
    block_sum<5>(acc, red, STENCIL_THREADS);
    if (tid == 0) {
#pragma unroll
      for (int i = 0; i < 5; ++i) parts[i] = acc[i];
    }
  } else if constexpr (MODE == MODE_MGPOST) {
    double a2[2] = {acc[0], acc[1]};
    block_sum<2>(a2, red, STENCIL_THREADS);
    if (tid == 0) {
      parts[0] = a2[0];
      parts[1] = a2[1];
    }
  } else if constexpr (MODE == MODE_MGDIR) {
    double a1[1] = {acc[0]};
    block_sum<1>(a1, red, STENCIL_THREADS);
    if (tid == 0) parts[0] = a1[0];
  } else if constexpr (MODE == MODE_RESID) {
    double a3[3] = {acc[0], acc[1], acc[2]};
    block_sum<3>(a3, red, STENCIL_THREADS);
    if (tid == 0) {
#pragma unroll
      for (int i = 0; i < 3; ++i) parts[i] = a3[i];
    }
  }
}

// one mode in a tiling; TS is the vectors' type where the kernel computes in FP64
template <int MODE, typename TS>
static hipError_t launch_f64(const LaunchArgs &la, int tiling, hipStream_t st) {
  if (la.total == 0) return hipSuccess;
  if (tiling == TILING_F64_TALL)
    stencil_kernel<double, TS, MODE, true><<<la.grid(), Tile<double, true>::THREADS, 0, st>>>(la);
  else
    stencil_kernel<double, TS, MODE><<<la.grid(), Tile<double>::THREADS, 0, st>>>(la);
  return hipGetLastError();
}

template <int MODE>
static hipError_t launch_mode(const LaunchArgs &la, int tiling, hipStream_t st) {
  if (tiling != TILING_F32) return launch_f64<MODE, double>(la, tiling, st);
  if (la.total == 0) return hipSuccess;
  stencil_kernel<float, float, MODE><<<la.grid(), Tile<float>::THREADS, 0, st>>>(la);
  return hipGetLastError();
}

hipError_t launch_stencil_pcg(const LaunchArgs &la, int tiling, hipStream_t st) {
  return launch_mode<MODE_PCG>(la, tiling, st);
}

// prec: of the vectors; tiling: an FP64 one
hipError_t launch_stencil_resid(const LaunchArgs &la, int prec, int tiling, hipStream_t st) {
  return prec == 0 ? launch_f64<MODE_RESID, double>(la, tiling, st) : launch_f64<MODE_RESID, float>(la, tiling, st);
}

hipError_t launch_stencil_apply(const LaunchArgs &la, int tiling, hipStream_t st) {
  return launch_mode<MODE_APPLY>(la, tiling, st);
}

// Voxel-level passes of the multigrid-preconditioned CG, in the vector
// precision: SMG_DIR the CG direction p_j = z + beta p_{j-1} (into the other
// p buffer) with the x update of the iteration before, q = K p_j and per-tile
// partials p_j . q; SMG_PRE the CG's residual update and the pre-smoothing
// step; SMG_POST the coarse correction and the post-smoothing step (per-tile
// partials b . z, b . b).
hipError_t launch_stencil_mg(const LaunchArgs &la, int tiling, int op, hipStream_t st) {
  switch (op) {
    case SMG_DIR: return launch_mode<MODE_MGDIR>(la, tiling, st);
    case SMG_PRE: return launch_mode<MODE_MGPRE>(la, tiling, st);
    case SMG_POST: return launch_mode<MODE_MGPOST>(la, tiling, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace shh
