// Kernels of the geometric multigrid preconditioner (see mg.hpp): setup
// (Galerkin element matrices, nodal stencils, diagonals, power iteration) and
// the V-cycle and CG sweeps.  T is the working precision of the slot.
#include "kernels.hpp"
#include "mg.hpp"

namespace shh {

// ---------------------------------------------------------------------------
// setup
// ---------------------------------------------------------------------------

// Element matrices are kept entry by entry ([24][24][elements]: neighbouring
// threads, which hold neighbouring elements, read and write neighbouring
// words) and formed row by row (grid y).  The 128^3 hierarchy takes 0.17 ms in
// these kernels and 0.03 in the stencils; with the matrices one after the other
// and the stencil summed in memory it took 1.16 and 0.40.

// Level-1 element matrices: K_E = sum_f E_f G_f over the 8 voxels of coarse
// element E.
template <typename T>
__global__ __launch_bounds__(256) void mg_elem1_kernel(const SlotDev *s, const MgDev *mg) {
  const MgLevel &c = mg->lv[1];
  const unsigned E = blockIdx.x * 256 + threadIdx.x;
  if (E >= (unsigned)c.nn) return;
  const int i = blockIdx.y, nc = c.n, nf = s->n;
  const int X = int(E % nc), Y = int((E / nc) % nc), Z = int(E / ((unsigned)nc * nc));
  const double *Ef = s->E64;
  const T *G = (const T *)mg->G + i * 24;
  double row[24];
#pragma unroll
  for (int j = 0; j < 24; ++j) row[j] = 0.0;
  for (int f = 0; f < 8; ++f) {
    const int fx = f & 1, fy = (f >> 1) & 1, fz = f >> 2;
    const double e = Ef[((long long)(2 * Z + fz) * nf + (2 * Y + fy)) * nf + (2 * X + fx)];
#pragma unroll
    for (int j = 0; j < 24; ++j) row[j] += e * (double)G[f * 576 + j];
  }
  T *K = (T *)c.Ke + (long long)i * 24 * c.nn + E;
#pragma unroll
  for (int j = 0; j < 24; ++j) K[j * c.nn] = (T)row[j];
}

// Trilinear weight of coarse corner a at fine corner b of child f (per axis:
// fine position (f + b) / 2 in the coarse element).
__device__ __forceinline__ double qweight(int f, int b, int a) {
  double w = 1.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int pos2 = ((f >> d) & 1) + ((b >> d) & 1);  // 0, 1 or 2 halves
    const int ad = (a >> d) & 1;
    const double p = 0.5 * pos2;
    w *= ad ? p : 1.0 - p;
  }
  return w;
}

// G2[f] = Q_f2^T G_f1 Q_f2 for the 64 voxels f = 4 (4 z + y) + x of a level-2
// element (child f2 of it, child f1 of that one), FP64.
template <typename T>
__global__ __launch_bounds__(192) void mg_g2_kernel(const MgDev *mg) {
  const int f = blockIdx.x, x = f & 3, y = (f >> 2) & 3, z = f >> 4;
  const int f1 = (x & 1) | ((y & 1) << 1) | ((z & 1) << 2), f2 = (x >> 1) | ((y >> 1) << 1) | ((z >> 1) << 2);
  const T *G = (const T *)mg->G + f1 * 576;
  for (int t = threadIdx.x; t < 576; t += 192) {
    const int i = t / 24, j = t % 24, a = i / 3, ci = i % 3, ap = j / 3, cj = j % 3;
    double sum = 0.0;
    for (int b = 0; b < 8; ++b) {
      const double qa = qweight(f2, b, a);
      if (qa == 0.0) continue;
      for (int bp = 0; bp < 8; ++bp) sum += qa * qweight(f2, bp, ap) * (double)G[(3 * b + ci) * 24 + 3 * bp + cj];
    }
    mg->G2[f * 576 + t] = sum;
  }
}

// Level-2 element matrices from the 64 voxels of an element, where level 1 keeps
// no element matrices (it runs from the moduli).
template <typename T>
__global__ __launch_bounds__(256) void mg_elem2_kernel(const SlotDev *s, const MgDev *mg) {
  const MgLevel &c = mg->lv[2];
  const unsigned E = blockIdx.x * 256 + threadIdx.x;
  if (E >= (unsigned)c.nn) return;
  const int i = blockIdx.y, nc = c.n, nf = s->n;
  const int X = int(E % nc), Y = int((E / nc) % nc), Z = int(E / ((unsigned)nc * nc));
  const SHH_CONST double *G2 = to_const((const double *)mg->G2) + i * 24;
  double row[24];
#pragma unroll
  for (int j = 0; j < 24; ++j) row[j] = 0.0;
  for (int yz = 0; yz < 16; ++yz) {
    const double *Ef = s->E64 + ((long long)(4 * Z + (yz >> 2)) * nf + 4 * Y + (yz & 3)) * nf + 4 * X;
    double e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = Ef[k];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < 24; ++j) row[j] += e[k] * G2[(4 * yz + k) * 576 + j];
  }
  T *K = (T *)c.Ke + (long long)i * 24 * c.nn + E;
#pragma unroll
  for (int j = 0; j < 24; ++j) K[j * c.nn] = (T)row[j];
}

// Level l + 1 element matrices from level l: K_E = sum_f Q_f^T K_f Q_f.  Eight
// lanes share a row, one child each (one thread per row took 300 us at 16^3:
// 648 loads in turn).
template <typename T>
__global__ __launch_bounds__(256) void mg_elemc_kernel(const MgDev *mg, int l) {
  const MgLevel &fl = mg->lv[l];
  const MgLevel &cl = mg->lv[l + 1];
  const unsigned t = blockIdx.x * 256 + threadIdx.x, E = t >> 3;
  const int f = t & 7;
  if (E >= (unsigned)cl.nn) return;  // all eight lanes of an element or none
  const int i = blockIdx.y, a = i / 3, ci = i % 3;
  const int nc = cl.n, nf = fl.n;
  const int X = int(E % nc), Y = int((E / nc) % nc), Z = int(E / ((unsigned)nc * nc));
  const long long fnn = fl.nn, cnn = cl.nn;
  const T *K = (const T *)fl.Ke + ((long long)(2 * Z + (f >> 2)) * nf + (2 * Y + ((f >> 1) & 1))) * nf + (2 * X + (f & 1));
  // w = Q_f[:, i]^T K_f: rows 3 b' + ci of K_f weighted by q(f, b', a)
  double w[24];
#pragma unroll
  for (int j = 0; j < 24; ++j) w[j] = 0.0;
  for (int bp = 0; bp < 8; ++bp) {
    const double q = qweight(f, bp, a);
    if (q == 0.0) continue;
    const T *kr = K + (3 * bp + ci) * 24 * fnn;
#pragma unroll
    for (int j = 0; j < 24; ++j) w[j] += q * (double)kr[j * fnn];
  }
  // row = w Q_f: column 3 a' + c sums w[3 b + c] q(f, b, a'); then over the children
  T *out = (T *)cl.Ke + (long long)i * 24 * cnn + E;
#pragma unroll
  for (int ap = 0; ap < 8; ++ap) {
    double row[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const double q = qweight(f, b, ap);
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) row[cc] += q * w[3 * b + cc];
    }
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
#pragma unroll
      for (int off = 1; off < 8; off <<= 1) row[cc] += __shfl_xor(row[cc], off, 64);
      if (f == ap) out[(3 * ap + cc) * cnn] = (T)row[cc];
    }
  }
}

// Nodal stencil of level l from its element matrices (the 14 stored offsets),
// and D^-1.  Node v is corner a of element v - a; entry (v, v - a + b)
// gathers K_e[a][b].  One thread per (node, stored offset: grid y); the
// corners a that have a corner b = a + offset in their element add up.
template <typename T>
__global__ __launch_bounds__(256) void mg_stencil_kernel(const MgDev *mg, int l) {
  const MgLevel &L = mg->lv[l];
  const unsigned v = blockIdx.x * 256 + threadIdx.x;
  if (v >= (unsigned)L.nn) return;
  const int n = L.n, k = blockIdx.y, w = 13 + k;
  const long long nn = L.nn;
  const int dz = w / 9 - 1, dy = (w / 3) % 3 - 1, dx = w % 3 - 1;
  const int x = int(v % n), y = int((v / n) % n), z = int(v / ((unsigned)n * n));
  const T *Ke = (const T *)L.Ke;
  T acc[9];
#pragma unroll
  for (int e = 0; e < 9; ++e) acc[e] = T(0);
  double diag[3] = {0.0, 0.0, 0.0};
  for (int a = 0; a < 8; ++a) {
    const int ax = a & 1, ay = (a >> 1) & 1, az = a >> 2;
    const int bx = ax + dx, by = ay + dy, bz = az + dz;
    if ((bx | by | bz) & ~1) continue;  // each is 0 or 1
    const int b = bx | (by << 1) | (bz << 2);
    const T *K = Ke + (3 * a * 24 + 3 * b) * nn + ((long long)wrapi(z - az, n) * n + wrapi(y - ay, n)) * n +
                 wrapi(x - ax, n);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int cp = 0; cp < 3; ++cp) {
        const T kv = K[(c * 24 + cp) * nn];
        acc[3 * c + cp] += kv;
        if (cp == c) diag[c] += (double)kv;
      }
  }
  T *S = (T *)L.S + (long long)k * 9 * nn + v;
#pragma unroll
  for (int e = 0; e < 9; ++e) S[e * nn] = acc[e];
  if (k != 0) return;
  T *Dinv = (T *)L.Dinv;
#pragma unroll
  for (int c = 0; c < 3; ++c) Dinv[c * nn + v] = diag[c] > 0.0 ? (T)(1.0 / diag[c]) : T(0);
}

// ---------------------------------------------------------------------------
// operator, transfer and coarsest solve (levels >= 1)
// ---------------------------------------------------------------------------

// The coarse-level Chebyshev sweep that follows an operator pass, applied
// to q = A_l v at node v, load case k (entry j = (3 k + c) nn + v):
// (degree-2 Chebyshev smoothing of A x = b from x = 0, then of the corrected x):
//   MGE_NONE:  q = A v
//   MGE_STEP1: (v = d0) r = b - q;  d1 = c1 d0 + c2 D^-1 r;  x = d0 + d1;  d1 into q
//   MGE_RES:   (v = d1, in q) r -= q: the residual the restriction takes
//   MGE_POST:  (v = x) r = b - q;  d = D^-1 r / theta;  x + d into q
//   MGE_LAST:  (v = d) x = (x + d, in q) + c1 d + c2 D^-1 (r - q)
// No pass writes the vector its operator reads.
// The level's vectors and coefficients, read once per thread into scalar
// registers: a field read after a store would be read again (the store might
// have changed it), behind a wait for the store.
template <typename T>
struct MgEpi {
  SHH_GLOBAL T *q, *r, *x, *d;
  const SHH_GLOBAL T *b;
  T c1, c2, inv_theta;
};
template <typename T>
__device__ __forceinline__ MgEpi<T> mg_epi(const MgLevel &L) {
  MgEpi<T> E;
  E.q = to_global((T *)L.q);
  E.r = to_global((T *)L.r);
  E.x = to_global((T *)L.x);
  E.d = to_global((T *)L.d);
  E.b = to_global((const T *)L.b);
  E.c1 = (T)L.c1;
  E.c2 = (T)L.c2;
  E.inv_theta = (T)L.inv_theta;
  return E;
}
// Inputs of the sweep at entry j (loaded for every output of a thread before
// its first store, so the loads overlap).
template <typename T, int EP>
__device__ __forceinline__ void mg_epi_load(const MgEpi<T> &E, long long j, T (&in)[3]) {
  if constexpr (EP == MGE_STEP1) {
    in[0] = E.d[j];
    in[1] = E.b[j];
  } else if constexpr (EP == MGE_RES) {
    in[0] = E.r[j];
  } else if constexpr (EP == MGE_POST) {
    in[0] = E.b[j];
    in[1] = E.x[j];
  } else if constexpr (EP == MGE_LAST) {
    in[0] = E.q[j];
    in[1] = E.d[j];
    in[2] = E.r[j];
  }
}
template <typename T, int EP>
__device__ __forceinline__ void mg_epilogue(const MgEpi<T> &E, long long j, T dinv, T a, const T (&in)[3]) {
  if constexpr (EP == MGE_NONE) {
    E.q[j] = a;
  } else if constexpr (EP == MGE_STEP1) {
    const T d0 = in[0];
    const T rv = in[1] - a;
    const T d1 = E.c1 * d0 + E.c2 * dinv * rv;
    E.r[j] = rv;
    E.x[j] = d0 + d1;
    E.q[j] = d1;
  } else if constexpr (EP == MGE_RES) {
    E.r[j] = in[0] - a;
  } else if constexpr (EP == MGE_POST) {
    const T rv = in[0] - a;
    const T dv = dinv * rv * E.inv_theta;
    E.r[j] = rv;
    E.d[j] = dv;
    E.q[j] = in[1] + dv;
  } else {  // MGE_LAST
    E.x[j] = in[0] + E.c1 * in[1] + E.c2 * dinv * (in[2] - a);
  }
}

// the operator's input vector of an epilogue (MGE_NONE: x)
template <typename T, int EP>
__device__ __forceinline__ const T *mg_operand(const MgLevel &L) {
  if constexpr (EP == MGE_STEP1 || EP == MGE_LAST) return (const T *)L.d;
  else if constexpr (EP == MGE_RES) return (const T *)L.q;
  else return (const T *)L.x;
}

// q = A_l v (v = x or d of the level) on levels of at most 32^3 nodes, where a
// pass is bound by the latency of a thread's chain of gathers and not by
// bytes: the 27 offsets of 64 nodes are split over the G waves of a workgroup
// (a wave takes 27 / G offsets, its loads in flight together), which meet in
// LDS; then wave g finishes rows g, g + G, ... of the RHS * 3 (load case,
// component) rows.  One thread per node and load case walking all 27 offsets
// took 12 us a pass at 6^3 as at 24^3 (one design).  G = 3 (planes) with all
// six load cases reads the stencil once; G = 9 (rows) with two load cases per
// workgroup gives the smallest levels enough threads.  Both add the offsets in
// the same order -- rows of three, planes of three rows, three planes -- so a
// design's result does not depend on the launch it shares.
template <typename T>
__device__ __forceinline__ T mg_fma(T a, T b, T c) {
  if constexpr (sizeof(T) == 4) return __builtin_fmaf(a, b, c);
  else return __builtin_fma(a, b, c);
}

// p[r][c] += the three offsets of row (dz, dy) of the stencil at node v, zero
// rows left out; wrapped neighbours x - 1, x, x + 1 of plane row zy
template <typename T, int RHS>
__device__ __forceinline__ void mg_row(const SHH_GLOBAL T *S, const SHH_GLOBAL T *in, long long nn, unsigned v,
                                       unsigned zy, const unsigned (&xs)[3], int row, const bool (&act)[RHS],
                                       T (&p)[RHS][3]) {
  T blk[3][9], val[3][RHS][3];
#pragma unroll
  for (int o = 0; o < 3; ++o) {
    const int w = row * 3 + o;  // uniform over the wave
    const unsigned u = zy + xs[o];
    const bool lower = w < 13;  // A[v][u] = A[u][v]^T, stored at u for offset 26 - w
    const SHH_GLOBAL T *Sw = S + (long long)((lower ? 13 - w : w - 13) * 9) * nn + (lower ? u : v);
#pragma unroll
    for (int k = 0; k < 9; ++k) blk[o][k] = Sw[k * nn];
#pragma unroll
    for (int r = 0; r < RHS; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c)  // an inactive load case reads one broadcast value
        val[o][r][c] = in[((long long)r * 3 + c) * nn + (act[r] ? u : 0u)];
  }
#pragma unroll
  for (int r = 0; r < RHS; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) p[r][c] = T(0);
#pragma unroll
  for (int o = 0; o < 3; ++o) {
    if (row * 3 + o < 13) {
#pragma unroll
      for (int r = 0; r < RHS; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int k = 0; k < 3; ++k) p[r][c] = mg_fma<T>(blk[o][3 * k + c], val[o][r][k], p[r][c]);
    } else {
#pragma unroll
      for (int r = 0; r < RHS; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int k = 0; k < 3; ++k) p[r][c] = mg_fma<T>(blk[o][3 * c + k], val[o][r][k], p[r][c]);
    }
  }
}

// the 27 / G offsets of group g into LDS partials part[g][3 r + c][lane]
template <typename T, int RHS, int G>
__device__ __forceinline__ void mg_split_sum(const MgLevel &L, const T *operand, unsigned v, int g,
                                             const bool (&act)[RHS], bool zero_row, T (*part)[RHS * 3][64]) {
  const int n = L.n, lane = threadIdx.x & 63;
  const SHH_GLOBAL T *S = to_global((const T *)L.S), *in = to_global(operand);
  const unsigned row = v / (unsigned)n;
  const int x = int(v - row * (unsigned)n), y = int(row % (unsigned)n), z = int(row / (unsigned)n);
  const unsigned xs[3] = {unsigned(wrap1(x - 1, n)), unsigned(x), unsigned(wrap1(x + 1, n))};
  T acc[RHS][3];
#pragma unroll
  for (int r = 0; r < RHS; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[r][c] = T(0);
  if (!zero_row) {
    if constexpr (G == 9) {
      const int dz = g / 3 - 1, dy = g % 3 - 1;
      mg_row<T, RHS>(S, in, L.nn, v, unsigned(wrap1(z + dz, n) * n + wrap1(y + dy, n)) * n, xs, g, act, acc);
    } else {
      const unsigned zo = unsigned(wrap1(z + g - 1, n) * n);
#pragma unroll 1  // three rows in flight would spill
      for (int j = 0; j < 3; ++j) {
        T p[RHS][3];
        mg_row<T, RHS>(S, in, L.nn, v, (zo + unsigned(wrap1(y + j - 1, n))) * n, xs, 3 * g + j, act, p);
#pragma unroll
        for (int r = 0; r < RHS; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c) acc[r][c] = j == 0 ? p[r][c] : acc[r][c] + p[r][c];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < RHS; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) part[g][3 * r + c][lane] = acc[r][c];
}

template <typename T, int RHS, int G>
__device__ __forceinline__ T mg_split_total(T (*part)[RHS * 3][64], int q, int lane) {
  if constexpr (G == 9) {
    T s[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
      s[k] = (part[3 * k][q][lane] + part[3 * k + 1][q][lane]) + part[3 * k + 2][q][lane];
    return (s[0] + s[1]) + s[2];
  } else {
    return (part[0][q][lane] + part[1][q][lane]) + part[2][q][lane];
  }
}

// grid x = 64-node blocks, y = groups of RHS load cases, z = slot
template <typename T, int RHS, int G, int EP>
__global__ __launch_bounds__(64 * G) __attribute__((amdgpu_waves_per_eu(2))) void mg_apply_split_kernel(MgBatch B, int l, int live) {
  __shared__ T part[G][RHS * 3][64];
  constexpr int IT = (RHS * 3 + G - 1) / G;
  const MgLevel &L = B.mg[blockIdx.z]->lv[l];
  const long long nn = L.nn;
  if ((long long)blockIdx.x * 64 >= nn) return;
  const int r0 = blockIdx.y * RHS;
  // live: load cases that have converged (or broken down) are skipped, as in
  // the voxel-level passes (Sec. 4.2.2: per-right-hand-side convergence)
  bool act[RHS];
  bool any = false;
#pragma unroll
  for (int r = 0; r < RHS; ++r) {
    act[r] = !live || B.slot[blockIdx.z]->st->active[r0 + r] != 0;
    any = any || act[r];
  }
  if (!any) return;
  const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool inr = blockIdx.x * 64 + lane < (unsigned)nn;
  const unsigned v = inr ? blockIdx.x * 64 + lane : 0u;
  const SHH_GLOBAL T *Dv = to_global((const T *)L.Dinv);
  // a node with a zero diagonal has a zero row (every element around it
  // culled): A v = 0 there without reading its stencil
  mg_split_sum<T, RHS, G>(L, mg_operand<T, EP>(L) + (long long)r0 * 3 * nn, v, g, act, Dv[v] == T(0), part);
  // the inputs of this thread's share of the fused sweep, loaded before the
  // waves meet
  const MgEpi<T> E = mg_epi<T>(L);
  T dv[IT], ein[IT][3];
  bool mine[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int q = g + i * G;
    bool on = false;  // uniform over the wave
#pragma unroll
    for (int r = 0; r < RHS; ++r) on = on || (q / 3 == r && act[r]);
    mine[i] = inr && on;
    if (mine[i]) {
      dv[i] = Dv[(long long)(q % 3) * nn + v];
      mg_epi_load<T, EP>(E, ((long long)r0 * 3 + q) * nn + v, ein[i]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int q = g + i * G;
    if (mine[i])
      mg_epilogue<T, EP>(E, ((long long)r0 * 3 + q) * nn + v, dv[i], mg_split_total<T, RHS, G>(part, q, lane), ein[i]);
  }
}

// q = A_l v on levels of more than 32^3 nodes, all six load cases, for two
// z-adjacent nodes per thread (every smoothing level is even): the vector values of the two
// planes between them are loaded once for both (12 % faster per launch than
// one node per thread).  Occupancy 2 waves per SIMD in FP32 (230 registers;
// holding it to 3 waves spills).  An inactive load case's gathers read one
// broadcast element instead of branching around them (7 % faster), and the
// fused sweep loads all of a node's inputs before its first store.
template <typename T, int EP>
__global__ __launch_bounds__(256) void mg_apply_pair_kernel(MgBatch B, int l, int live) {
  const MgLevel &L = B.mg[blockIdx.z]->lv[l];
  const long long nn = L.nn;
  const int n = L.n;
  const long long plane = (long long)n * n;
  const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= unsigned(nn / 2)) return;
  bool act[NRHS];
  bool any = false;
#pragma unroll
  for (int r = 0; r < NRHS; ++r) {
    act[r] = !live || B.slot[blockIdx.z]->st->active[r] != 0;
    any = any || act[r];
  }
  if (!any) return;
  // 32-bit index arithmetic (n <= 512)
  const unsigned zp = t / unsigned(plane);
  const unsigned xy = t - zp * unsigned(plane);
  const int y = int(xy / unsigned(n)), x = int(xy - unsigned(y) * unsigned(n)), z0 = 2 * int(zp);
  const long long v0 = (long long)z0 * plane + xy;
  const SHH_GLOBAL T *S = to_global((const T *)L.S);
  const SHH_GLOBAL T *Dv = to_global((const T *)L.Dinv);
  const SHH_GLOBAL T *in = to_global(mg_operand<T, EP>(L));
  // nodes with a zero diagonal have a zero row (every element around them
  // culled): A v = 0 there without reading their stencil
  const bool zero_rows = Dv[v0] == T(0) && Dv[v0 + plane] == T(0);
  T acc[2][NRHS][3];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int r = 0; r < NRHS; ++r)
#pragma unroll
      for (int c = 0; c < 3; ++c) acc[k][r][c] = T(0);
  if (!zero_rows) {
#pragma unroll
    for (int pz = 0; pz < 4; ++pz) {  // planes z0 - 1 .. z0 + 2
      const long long pzo = (long long)wrap1(z0 - 1 + pz, n) * plane;
      // three offsets per trip (one and nine measured slower)
#pragma unroll 3
      for (int o = 0; o < 9; ++o) {
        const int dx = o % 3 - 1, dy = o / 3 - 1;
        const long long u = pzo + (long long)wrap1(y + dy, n) * n + wrap1(x + dx, n);
        T val[NRHS][3];
#pragma unroll
        for (int r = 0; r < NRHS; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c)  // an inactive load case reads one broadcast
            val[r][c] = in[((long long)r * 3 + c) * nn + (act[r] ? u : 0)];  // value: no branch, no traffic
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int dz = pz - 1 - k;
          if (dz < -1 || dz > 1) continue;
          const int w = (dz + 1) * 9 + o;
          const long long v = v0 + k * plane;
          T blk[9];
          if (w >= 13) {
#pragma unroll
            for (int e = 0; e < 9; ++e) blk[e] = S[((w - 13) * 9 + e) * nn + v];
          } else {
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
              for (int cp = 0; cp < 3; ++cp) blk[3 * c + cp] = S[((13 - w) * 9 + 3 * cp + c) * nn + u];
          }
#pragma unroll
          for (int r = 0; r < NRHS; ++r)
#pragma unroll
            for (int c = 0; c < 3; ++c)
              acc[k][r][c] += blk[3 * c] * val[r][0] + blk[3 * c + 1] * val[r][1] + blk[3 * c + 2] * val[r][2];
        }
      }
    }
  }
  // output stage, per node: every load of its sweep before its first store
  const MgEpi<T> E = mg_epi<T>(L);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const long long vk = v0 + k * plane;
    T dv[3], ein[NRHS][3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c) dv[c] = Dv[(long long)c * nn + vk];
#pragma unroll
    for (int r = 0; r < NRHS; ++r)
      if (act[r])
#pragma unroll
        for (int c = 0; c < 3; ++c) mg_epi_load<T, EP>(E, ((long long)r * 3 + c) * nn + vk, ein[r][c]);
#pragma unroll
    for (int r = 0; r < NRHS; ++r)
      if (act[r])
#pragma unroll
        for (int c = 0; c < 3; ++c)
          mg_epilogue<T, EP>(E, ((long long)r * 3 + c) * nn + vk, dv[c], acc[k][r][c], ein[r][c]);
  }
}

// two-wide element pairs of the fine vectors (x = 2X and 2X + 1)
template <typename T> struct Pair2 { using type = T __attribute__((ext_vector_type(2))); };

// b_{l+1} = P^T r_l, the residual after the pre-smoother (its last operator
// pass leaves it in r): coarse node I collects fine nodes 2I + o,
// o in {-1, 0, 1}^3, with weight prod (o == 0 ? 1 : 1/2).  One thread per
// coarse node, grid y = load case.  Per fine row the pair (2X, 2X + 1) is one
// two-wide load; the odd node 2X - 1 is the pair of the lane below (a
// shuffle), loaded only where that lane holds another row or wave.  Node
// indices fit 32 bits (n <= 512): 64-bit divisions would cost more than the
// kernel's memory traffic.  Where the coarse level is smoothed, its first
// Chebyshev direction d = D^-1 b / theta is written along (a sweep of its own
// before).
template <typename T>
__global__ __launch_bounds__(256) void mg_restrict_kernel(MgBatch B, int l) {
  using T2 = typename Pair2<T>::type;
  const MgDev *mg = B.mg[blockIdx.z];
  const MgLevel &F = mg->lv[l];
  const MgLevel &C = mg->lv[l + 1];
  const unsigned I = blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  // in-range lanes are a prefix of the wave, so the lane below an in-range
  // lane is in range too
  if (I >= (unsigned)C.nn || !B.slot[blockIdx.z]->st->active[k]) return;
  const int nc = C.n, nf = F.n;
  const unsigned row = I / (unsigned)nc;
  const int X = int(I - row * (unsigned)nc), Y = int(row % (unsigned)nc), Z = int(row / (unsigned)nc);
  const bool own_left = X == 0 || (threadIdx.x & 63u) == 0;
  const int xl = X == 0 ? nf - 1 : 2 * X - 1;
  const SHH_GLOBAL T *r = to_global((const T *)F.r) + (long long)k * 3 * F.nn;
  // all loads are issued before the first shuffle waits on one
  unsigned rowo[9];
#pragma unroll
  for (int oz = 0; oz < 3; ++oz)
#pragma unroll
    for (int oy = 0; oy < 3; ++oy)
      rowo[3 * oz + oy] =
          (unsigned(wrap1(2 * Z + oz - 1, nf)) * unsigned(nf) + unsigned(wrap1(2 * Y + oy - 1, nf))) * unsigned(nf);
  const bool smooth = l + 1 < mg->L;
  const SHH_GLOBAL T *Dc = to_global((const T *)C.Dinv);
  T dv[3] = {T(0), T(0), T(0)};
  if (smooth) {
#pragma unroll
    for (int c = 0; c < 3; ++c) dv[c] = Dc[(long long)c * C.nn + I];
  }
  T2 v[9][3];
#pragma unroll
  for (int o = 0; o < 9; ++o)
#pragma unroll
    for (int c = 0; c < 3; ++c) v[o][c] = *(const SHH_GLOBAL T2 *)(r + (long long)c * F.nn + rowo[o] + 2 * X);
  T left[9][3];
#pragma unroll
  for (int o = 0; o < 9; ++o)
#pragma unroll
    for (int c = 0; c < 3; ++c) left[o][c] = __shfl_up(v[o][c].y, 1);
  if (own_left) {
#pragma unroll
    for (int o = 0; o < 9; ++o)
#pragma unroll
      for (int c = 0; c < 3; ++c) left[o][c] = r[(long long)c * F.nn + rowo[o] + xl];
  }
  T acc[3] = {T(0), T(0), T(0)};
#pragma unroll
  for (int o = 0; o < 9; ++o) {
    const T wyz = T((o / 3 != 1 ? 0.5 : 1.0) * (o % 3 != 1 ? 0.5 : 1.0));
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] += wyz * (v[o][c].x + T(0.5) * (v[o][c].y + left[o][c]));
  }
  const long long cnn = C.nn;  // read once: the stores below might alias it
  const T ith = (T)C.inv_theta;
  SHH_GLOBAL T *b = to_global((T *)C.b) + (long long)k * 3 * cnn;
  SHH_GLOBAL T *d = to_global((T *)C.d) + (long long)k * 3 * cnn;
#pragma unroll
  for (int c = 0; c < 3; ++c) b[c * cnn + I] = acc[c];
  if (smooth) {
#pragma unroll
    for (int c = 0; c < 3; ++c) d[c * cnn + I] = dv[c] * acc[c] * ith;
  }
}

// b_1 = P^T r_0 from the shares that the FP32 pre-smoothing pass left in r_0
// (stencil.hip): a coarse node takes its own tile's, and on a tile's first
// plane, row or column also the last one of the tile before.  One thread per
// coarse node; d is written as by the restriction.
__global__ __launch_bounds__(256) void mg_gather_kernel(MgBatch B) {
  using TT = Tile<float>;
  constexpr int CX = TT::X / 2, CY = TT::Y / 2;
  const MgDev *mg = B.mg[blockIdx.z];
  const SlotDev *s = B.slot[blockIdx.z];
  const MgLevel &C = mg->lv[1];
  const unsigned I = blockIdx.x * 256 + threadIdx.x;
  const int k = blockIdx.y;
  if (I >= (unsigned)C.nn || !s->st->active[k]) return;
  const int nc = C.n, cz = s->tz / 2, cols = min(CX, nc) + 1;
  const int tx = s->tiles_x[1], ty = s->tiles_y[1], runs = s->tiles_z;
  const unsigned row = I / (unsigned)nc;
  const int X = int(I - row * (unsigned)nc), Y = int(row % (unsigned)nc), Z = int(row / (unsigned)nc);
  // tile and place in it, own and (where there is one) the tile before
  struct Axis {
    int t[2], at[2], m;
  };
  auto axis = [nc](int i, int step, int tiles) {
    Axis a;
    a.t[0] = i / step;
    a.at[0] = i - a.t[0] * step;
    a.m = a.at[0] == 0 ? 2 : 1;
    a.t[1] = i == 0 ? tiles - 1 : a.t[0] - 1;
    a.at[1] = i == 0 ? nc - step * (tiles - 1) : step;
    return a;
  };
  const Axis ax = axis(X, CX, tx), ay = axis(Y, CY, ty), az = axis(Z, cz, runs);
  const SHH_GLOBAL float *r = to_global((const float *)mg->lv[0].r) + (long long)k * 3 * mg->lv[0].nn;
  const SHH_GLOBAL float *Dc = to_global((const float *)C.Dinv);
  const long long cnn = C.nn;
  const bool smooth = mg->L > 1;
  float dv[3] = {0.0f, 0.0f, 0.0f}, acc[3] = {0.0f, 0.0f, 0.0f};
  if (smooth) {
#pragma unroll
    for (int c = 0; c < 3; ++c) dv[c] = Dc[c * cnn + I];
  }
  const unsigned cst = (unsigned)((CY + 1) * cols);
#pragma unroll
  for (int iz = 0; iz < 2; ++iz)
#pragma unroll
    for (int iy = 0; iy < 2; ++iy)
#pragma unroll
      for (int ix = 0; ix < 2; ++ix) {
        if (iz >= az.m || iy >= ay.m || ix >= ax.m) continue;
        const unsigned tile = unsigned((az.t[iz] * ty + ay.t[iy]) * tx + ax.t[ix]);
        const unsigned o = (tile * unsigned(cz + 1) + unsigned(az.at[iz])) * 3u * cst + unsigned(ay.at[iy] * cols + ax.at[ix]);
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] += r[o + c * cst];
      }
  const float ith = (float)C.inv_theta;
  SHH_GLOBAL float *b = to_global((float *)C.b) + (long long)k * 3 * cnn;
  SHH_GLOBAL float *d = to_global((float *)C.d) + (long long)k * 3 * cnn;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    b[c * cnn + I] = acc[c];
    if (smooth) d[c * cnn + I] = dv[c] * acc[c] * ith;
  }
}

// x_l += P x_{l+1}: fine node 2I + a, a in {0, 1}^3, takes the coarse nodes
// I + i with i_d in {0, a_d}, weight 1/2 per axis with a_d = 1.  One thread
// per coarse node (grid y = load case) updates its 2 x 2 x 2 fine block as
// four two-wide pairs; 32-bit node indices as in the restriction.
template <typename T>
__global__ __launch_bounds__(256) void mg_prolong_kernel(MgBatch B, int l) {
  using T2 = typename Pair2<T>::type;
  const MgDev *mg = B.mg[blockIdx.z];
  const MgLevel &F = mg->lv[l];
  const MgLevel &C = mg->lv[l + 1];
  const unsigned I = blockIdx.x * blockDim.x + threadIdx.x;
  const int k = blockIdx.y;
  if (I >= (unsigned)C.nn || !B.slot[blockIdx.z]->st->active[k]) return;
  const int nc = C.n, nf = F.n;
  const long long cnn = C.nn, fnn = F.nn;  // read once: the stores below might alias them
  const unsigned row = I / (unsigned)nc;
  const int X = int(I - row * (unsigned)nc), Y = int(row % (unsigned)nc), Z = int(row / (unsigned)nc);
  const int X1 = X + 1 == nc ? 0 : X + 1;
  const unsigned cy[2] = {unsigned(Y), unsigned(Y + 1 == nc ? 0 : Y + 1)};
  const unsigned cz[2] = {unsigned(Z), unsigned(Z + 1 == nc ? 0 : Z + 1)};
  const SHH_GLOBAL T *xc = to_global((const T *)C.x) + (long long)k * 3 * cnn;
  SHH_GLOBAL T *xf = to_global((T *)F.x) + (long long)k * 3 * fnn;
  // every load (coarse values, then the fine pairs) is issued before the
  // first store
  T cv[3][2][2][2];  // [c][z][y][x] offsets 0 / +1
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int iz = 0; iz < 2; ++iz)
#pragma unroll
      for (int iy = 0; iy < 2; ++iy) {
        const SHH_GLOBAL T *v = xc + (long long)c * cnn + (cz[iz] * unsigned(nc) + cy[iy]) * unsigned(nc);
        cv[c][iz][iy][0] = v[X];
        cv[c][iz][iy][1] = v[X1];
      }
  unsigned fi[2][2];
#pragma unroll
  for (int az = 0; az < 2; ++az)
#pragma unroll
    for (int ay = 0; ay < 2; ++ay)
      fi[az][ay] = ((2 * unsigned(Z) + az) * unsigned(nf) + 2 * unsigned(Y) + ay) * unsigned(nf) + 2 * X;
  T2 f[3][2][2];
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int az = 0; az < 2; ++az)
#pragma unroll
      for (int ay = 0; ay < 2; ++ay) f[c][az][ay] = *(const SHH_GLOBAL T2 *)(xf + (long long)c * fnn + fi[az][ay]);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int az = 0; az < 2; ++az)
#pragma unroll
      for (int ay = 0; ay < 2; ++ay) {
        T s[2];
#pragma unroll
        for (int ix = 0; ix < 2; ++ix) {
          const T yz0 = ay ? T(0.5) * (cv[c][0][0][ix] + cv[c][0][1][ix]) : cv[c][0][0][ix];
          const T yz1 = ay ? T(0.5) * (cv[c][1][0][ix] + cv[c][1][1][ix]) : cv[c][1][0][ix];
          s[ix] = az ? T(0.5) * (yz0 + yz1) : yz0;
        }
        T2 o = f[c][az][ay];
        o.x += s[0];
        o.y += T(0.5) * (s[0] + s[1]);
        *(SHH_GLOBAL T2 *)(xf + (long long)c * fnn + fi[az][ay]) = o;
      }
}

// Coarsest level: x = Mc b for all load cases.  Sixteen lanes share a row (its
// 3 n_c^3 entries are read once, coalesced) and combine their partial sums by
// shuffles; a workgroup takes 16 rows.  (One workgroup per load case, four
// lanes a row, took 33 us at 4^3: 192 rows in three rounds of 48 dependent
// uncoalesced loads.)
template <typename T>
__global__ __launch_bounds__(256) void mg_coarsest_kernel(MgBatch B) {
  const MgDev *mg = B.mg[blockIdx.z];
  const MgLevel &L = mg->lv[mg->L];
  const int nd = mg->ndof_c;
  if ((int)blockIdx.x * 16 >= nd) return;
  const int *active = B.slot[blockIdx.z]->st->active;
  bool act[NRHS];
  bool any = false;
#pragma unroll
  for (int k = 0; k < NRHS; ++k) {
    act[k] = active[k] != 0;
    any = any || act[k];
  }
  if (!any) return;
  const long long nn = L.nn;
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4), part = threadIdx.x & 15;
  const double *M = mg->Mc + (long long)min(row, nd - 1) * nd;
  const T *b = (const T *)L.b;
  double acc[NRHS];
#pragma unroll
  for (int k = 0; k < NRHS; ++k) acc[k] = 0.0;
#pragma unroll 4
  for (int j = part; j < nd; j += 16) {
    const double m = M[j];
    const int at = (j % 3) * (int)nn + j / 3;
#pragma unroll
    for (int k = 0; k < NRHS; ++k) acc[k] += m * (double)b[k * 3 * (int)nn + at];
  }
#pragma unroll
  for (int k = 0; k < NRHS; ++k)
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) acc[k] += __shfl_xor(acc[k], off, 64);
  T *x = (T *)L.x;
#pragma unroll
  for (int k = 0; k < NRHS; ++k)
    if (part == k && row < nd && act[k]) x[(k * 3 + row % 3) * (int)nn + row / 3] = (T)acc[k];
}

// CG scalars of the multigrid-preconditioned solve (one workgroup per load
// case; per-tile partials of the voxel-level stencil passes: the direction
// pass for ALPHA, the last post-smoothing sweep for RESTART and BETA).
//   RESTART: rho = r . z after a (re)started V-cycle, beta = 0
//   REPLACE: the same after a residual replacement, the direction kept:
//            beta = rho' / (rho the last iteration started from)
//   ALPHA:   alpha = rho / p . K p; the new direction becomes current
//   BETA:    rho' = r . z, ||r||^2 -> convergence; beta = rho' / rho
// After a V-cycle (all but ALPHA) the residual buffer that its pre-smoothing
// pass wrote becomes current.  alpha stays set after BETA, whatever the load
// case's state: x += alpha p is applied by the next direction pass or, where
// none follows, before the next FP64 residual.
__global__ __launch_bounds__(VEC_THREADS) void mg_scalar_kernel(MgBatch B, int phase) {
  __shared__ double red[2 * 16];
  const SlotDev *s = B.slot[blockIdx.z];
  const int k = blockIdx.x;
  CgState *st = s->st;
  const double *parts = s->partials + (long long)k * s->maxparts * PSTRIDE;
  double tot[2];
  sum_partials<2, PSTRIDE>(parts, s->ntiles[s->wt], tot, red, VEC_THREADS);
  if (threadIdx.x != 0) return;
  // the passes before this ran for the active load cases only
  if (!st->active[k]) return;
  if (phase != MGS_ALPHA) st->pcur[k] ^= 1;
  if (phase == MGS_RESTART || phase == MGS_REPLACE) {
    // (the replacement's residual phase has since overwritten rho and beta
    // with the Jacobi recurrences; rho_mg kept the iteration's own rho)
    // The direction is kept only while the replaced residual agrees with the
    // recursive one (r . z within a factor 2 of it: rho_prev holds the
    // recursive value); a larger drift restarts.
    const double rho = tot[0], rho0 = st->rho_mg[k], rho_rec = st->rho_prev[k];
    const bool keep = phase == MGS_REPLACE && rho0 > 0.0 && rho_rec > 0.0 && rho <= 2.0 * rho_rec &&
                      rho >= 0.5 * rho_rec;
    st->beta[k] = keep ? rho / rho0 : 0.0;
    st->rho[k] = rho;
    st->alpha[k] = 0.0;
    if (!(rho > 0.0) || !isfinite(rho)) {
      st->status[k] = ST_BREAKDOWN;
      st->active[k] = 0;
    }
  } else if (phase == MGS_ALPHA) {
    st->mgpar[k] ^= 1;
    const double sigma = tot[0], rho = st->rho[k];
    const bool ok = isfinite(sigma) && sigma > 0.0 && rho > 0.0;
    st->alpha[k] = ok ? rho / sigma : 0.0;
    if (!ok) {
      st->status[k] = ST_BREAKDOWN;
      st->active[k] = 0;
    }
  } else {
    const double rho_n = tot[0], rr = tot[1];
    st->iters[k] += 1;
    st->rr[k] = rr;
    const double rel = sqrt(rr / st->ff[k]);
    st->rel[k] = rel;
    const double rho = st->rho[k];
    const bool ok = isfinite(rho_n) && rho_n >= 0.0;
    st->beta[k] = ok && rho > 0.0 ? rho_n / rho : 0.0;
    st->rho_mg[k] = rho;
    st->rho[k] = rho_n;
    if (rel <= s->rtol) {
      st->status[k] = ST_CONVERGED;
      st->active[k] = 0;
    } else if (!ok || !isfinite(rel)) {
      st->status[k] = ST_BREAKDOWN;
      st->active[k] = 0;
    } else if (st->iters[k] >= s->max_iter) {
      st->status[k] = ST_MAXIT;
      st->active[k] = 0;
    }
  }
}

// Power iteration for lambda_max(D^-1 A) of every coarse smoothing level of a
// batch of slots (grid z = slot), on load case 0, the level's x and q taking
// turns as the vector.  One launch is one step of all levels: a level's blocks
// of 64 nodes follow those of the level above it.  (Four launches per step and
// level before: the steps of a single 128^3 design took 4.8 of its 9 ms of setup.)
//   step:   x' = s D^-1 A x with s the last step's 1 / ||x||, and partial sums
//           of x.A x, x.D x (their ratio is the Rayleigh quotient of D^-1 A,
//           self-adjoint in the D inner product) and ||x'||^2
//   reduce: the partials of each level; the largest quotient into lmax
__device__ __forceinline__ int mg_power_level(const MgDev *mg, int &block, int &first) {
  first = 0;
  for (int l = 1; l < mg->L; ++l) {
    const int nb = int((mg->lv[l].nn + 63) / 64);
    if (block < nb) return l;
    block -= nb;
    first += nb;
  }
  return 0;
}

template <typename T>
__global__ __launch_bounds__(256) void mg_power_init_kernel(MgBatch B, int l) {
  if (l >= B.mg[blockIdx.z]->L) return;
  const MgLevel &L = B.mg[blockIdx.z]->lv[l];
  const unsigned j = blockIdx.x * 256 + threadIdx.x;
  if (j >= 3 * (unsigned)L.nn) return;
  uint32_t h = j * 2654435761u + 0x9e3779b9u;
  h ^= h >> 16;
  h *= 0x85ebca6bu;
  h ^= h >> 13;
  ((T *)L.x)[j] = (T)((double)(h & 0xffffff) / 16777216.0 - 0.5);
}

template <typename T>
__global__ __launch_bounds__(192) void mg_power_step_kernel(MgBatch B, int step) {
  __shared__ T part[3][3][64];
  __shared__ double red[3 * 16];
  const SlotDev *s = B.slot[blockIdx.z];
  int block = blockIdx.x, first;
  const int l = mg_power_level(B.mg[blockIdx.z], block, first);
  if (l == 0) return;
  const MgLevel &L = B.mg[blockIdx.z]->lv[l];
  const long long nn = L.nn;
  // a level without a stencil has A x in q already and keeps its vector in x
  const bool have = l == 1 && B.mg[blockIdx.z]->l1free;
  const T *x = (const T *)(!have && step & 1 ? L.q : L.x);
  T *xn = (T *)(have || step & 1 ? L.x : L.q);
  const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool inr = (unsigned)block * 64 + lane < (unsigned)nn;
  const unsigned v = inr ? block * 64 + lane : 0u;
  const T *Dv = (const T *)L.Dinv;
  const bool act[1] = {true};
  if (!have) mg_split_sum<T, 1, 3>(L, x, v, g, act, Dv[v] == T(0), part);
  __syncthreads();
  double acc[3] = {0.0, 0.0, 0.0};
  if (inr) {  // wave g finishes component g
    const long long j = g * nn + v;
    const T qv = have ? ((const T *)L.q)[j] : mg_split_total<T, 1, 3>(part, g, lane), di = Dv[j];
    const double xo = (double)x[j];
    acc[1] = xo * (double)qv;
    acc[2] = di != T(0) ? xo * xo / (double)di : 0.0;
    const T w = (T)((double)(di * qv) * L.pw_scale);
    xn[j] = w;
    acc[0] = (double)w * (double)w;
  }
  block_sum<3>(acc, red, 192);
  if (threadIdx.x == 0) {
    double *p = s->partials + (long long)(first + block) * PSTRIDE;
    p[0] = acc[0];
    p[1] = acc[1];
    p[2] = acc[2];
  }
}

// grid x = level - 1, z = slot: reduce the partials, keep the largest Rayleigh
// quotient in lmax and the normalization for the next step (a vanishing or
// non-finite step leaves lmax = -1, which the host reports as a breakdown).
__global__ __launch_bounds__(VEC_THREADS) void mg_power_reduce_kernel(MgBatch B) {
  __shared__ double red[3 * 16];
  const SlotDev *s = B.slot[blockIdx.z];
  const int l = blockIdx.x + 1;
  // the slot's own descriptor in device memory, written only here
  MgDev *mg = const_cast<MgDev *>(B.mg[blockIdx.z]);
  if (l >= mg->L) return;
  int first = 0;
  for (int k = 1; k < l; ++k) first += int((mg->lv[k].nn + 63) / 64);
  MgLevel &L = mg->lv[l];
  double tot[3];
  sum_partials<3, PSTRIDE>(s->partials + (long long)first * PSTRIDE, int((L.nn + 63) / 64), tot, red, VEC_THREADS);
  if (threadIdx.x != 0) return;
  const double nrm = sqrt(tot[0]);
  if (!(nrm > 0.0) || !isfinite(nrm) || !(tot[2] > 0.0) || L.lmax < 0.0) {
    L.lmax = -1.0;
    L.pw_scale = 0.0;
    return;
  }
  L.lmax = fmax(L.lmax, tot[1] / tot[2]);
  L.pw_scale = 1.0 / nrm;
}

// The coarsest level's dense inverse, FP64: assemble the operator from the
// stored stencil blocks (row 3 v + c gathers every block of node v, the lower
// offsets transposed from the neighbours), add gamma / nn to each component's
// constant block (gamma = mean diagonal; this makes the operator nonsingular
// on the rigid translations and leaves its inverse on the range equal to the
// pseudo-inverse), then invert in place by Gauss-Jordan elimination over blocks
// of 32 (the matrix is symmetric positive definite, so no pivoting):
//   P = A_kk^-1;  R_j = P A_kj, C_i = A_ik (panel kernel, into scratch);
//   A_kk = P, A_kj = R_j, A_ik = -C_i P, A_ij -= C_i R_j (update kernel).
// One workgroup sweeping the whole matrix in global memory row by row took
// 1.8 ms at 4^3 (192 rows) and grew with the cube: 7^3 has 1029.
// Grid z = slot throughout.
constexpr int IB = 32;  // block edge
struct InvScratch {
  double *P, *R, *Cc, *mean;  // [IB][IB], [blocks][IB][IB] twice, the mean diagonal
  __device__ InvScratch(double *base, int nblk) : P(base), R(base + IB * IB), Cc(R + nblk * IB * IB),
                                                  mean(Cc + nblk * IB * IB) {}
};

template <typename T>
__global__ __launch_bounds__(256) void mg_inv_assemble_kernel(MgBatch B) {
  __shared__ double red[16];
  const MgDev *mg = B.mg[blockIdx.z];
  const MgLevel &L = mg->lv[mg->L];
  const int n = L.n, m = mg->ndof_c, nn = int(L.nn);
  if ((int)blockIdx.x * 4 >= m) return;
  const T *S = (const T *)L.S;
  double acc[1] = {0.0};
  for (int i = threadIdx.x; i < m; i += 256) acc[0] += (double)S[4 * (i % 3) * nn + i / 3];
  block_sum<1>(acc, red, 256);
  if (threadIdx.x == 0) red[0] = acc[0];
  __syncthreads();
  // a stencil past the range of FP32 has no inverse: a zero matrix, all of whose
  // pivots vanish below, leaves the coarsest level out of the cycle
  const bool finite = isfinite(red[0]);
  const double mean_diag = finite ? red[0] / m : 0.0, add = mean_diag / double(nn);
  if (blockIdx.x == 0 && threadIdx.x == 0) *InvScratch((double *)mg->inv, (m + IB - 1) / IB).mean = mean_diag;
  // one wave per row: the constant blocks, then the 81 stencil entries on top
  // (27 distinct neighbours: n >= 3)
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= m) return;
  const int v = row / 3, c = row % 3;
  double *A = mg->Mc + (long long)row * m;
  const int x = v % n, y = (v / n) % n, z = v / (n * n);
  for (int j = lane; j < m; j += 64) {
    const int u = j / 3, cp = j % 3;
    // offset of u from v on the periodic grid, if within one node
    auto off = [n](int a, int b) {
      const int d = a - b;
      return d == n - 1 ? -1 : (d == 1 - n ? 1 : d);
    };
    const int dx = off(u % n, x), dy = off((u / n) % n, y), dz = off(u / (n * n), z);
    double a = c == cp ? add : 0.0;
    if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1) {
      const int w = (dz + 1) * 9 + (dy + 1) * 3 + dx + 1;
      a += w >= 13 ? (double)S[((w - 13) * 9 + 3 * c + cp) * nn + v] : (double)S[((13 - w) * 9 + 3 * cp + c) * nn + u];
    }
    A[j] = finite ? a : 0.0;
  }
}

// Step k, grid x = block t: every workgroup inverts A_kk for itself (one
// barrier per pivot), block k stores it, the others their R_t and C_t.  A pivot
// at or below 1e-12 of the mean diagonal is a vanishing pivot of the (positive
// semidefinite) Schur complement: the dof is a null direction beyond the rigid
// translations (nodes whose elements are all culled, pieces that float at this
// level).  It is taken out -- row and column zero, in P and hence in R, C P and
// the updates -- so the result stays a symmetric generalized inverse.  Never
// taken on the floored operator.
__global__ __launch_bounds__(256) void mg_inv_panel_kernel(MgBatch B, int k) {
  __shared__ double P[IB][IB + 1], M[IB][IB + 1], rowp[2][IB], colp[2][IB];
  const MgDev *mg = B.mg[blockIdx.z];
  const int m = mg->ndof_c, nblk = (m + IB - 1) / IB, t = blockIdx.x;
  if (k >= nblk || t >= nblk) return;
  InvScratch W((double *)mg->inv, nblk);
  const double *A = mg->Mc;
  const double floor_ = 1e-12 * *W.mean;
  const int bk = min(IB, m - k * IB), bt = min(IB, m - t * IB);
  const int i = threadIdx.x >> 3, j0 = (threadIdx.x & 7) * 4;
  double a[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)  // past the matrix: the identity
    a[e] = i < bk && j0 + e < bk ? A[(long long)(k * IB + i) * m + k * IB + j0 + e] : (i == j0 + e ? 1.0 : 0.0);
  for (int p = 0; p < bk; ++p) {
    const int b = p & 1;
    if (i == p)
#pragma unroll
      for (int e = 0; e < 4; ++e) rowp[b][j0 + e] = a[e];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (j0 + e == p) colp[b][i] = a[e];
    __syncthreads();
    const double piv = rowp[b][p], f = colp[b][i];
    const bool ok = piv > floor_;
    const double inv = ok ? 1.0 / piv : 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = j0 + e;
      const double r = j == p ? inv : rowp[b][j] * inv;
      if (!ok) a[e] = i == p || j == p ? 0.0 : a[e];
      else a[e] = i == p ? r : (j == p ? 0.0 : a[e]) - f * r;
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (t == k) W.P[i * IB + j0 + e] = a[e];
    P[i][j0 + e] = a[e];
  }
  if (t == k) return;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    M[i][j0 + e] = i < bk && j0 + e < bt ? A[(long long)(k * IB + i) * m + t * IB + j0 + e] : 0.0;
    W.Cc[(t * IB + i) * IB + j0 + e] = i < bt && j0 + e < bk ? A[(long long)(t * IB + i) * m + k * IB + j0 + e] : 0.0;
  }
  __syncthreads();
  double r[4] = {0.0, 0.0, 0.0, 0.0};
  for (int q = 0; q < bk; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] += P[i][q] * M[q][j0 + e];
#pragma unroll
  for (int e = 0; e < 4; ++e) W.R[(t * IB + i) * IB + j0 + e] = r[e];
}

__global__ __launch_bounds__(256) void mg_inv_update_kernel(MgBatch B, int k) {
  __shared__ double X[IB][IB + 1], Y[IB][IB + 1];
  const MgDev *mg = B.mg[blockIdx.z];
  const int m = mg->ndof_c, nblk = (m + IB - 1) / IB, tj = blockIdx.x, ti = blockIdx.y;
  if (k >= nblk || tj >= nblk || ti >= nblk) return;
  InvScratch W((double *)mg->inv, nblk);
  const int bi = min(IB, m - ti * IB), bj = min(IB, m - tj * IB), bk = min(IB, m - k * IB);
  const int i = threadIdx.x >> 3, j0 = (threadIdx.x & 7) * 4;
  const double *src = ti == k ? (tj == k ? W.P : W.R + tj * IB * IB) : nullptr;
  const double *right = tj == k ? W.P : W.R + tj * IB * IB;
  if (!src) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      X[i][j0 + e] = W.Cc[(ti * IB + i) * IB + j0 + e];
      Y[i][j0 + e] = right[i * IB + j0 + e];
    }
    __syncthreads();
  }
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (!src)
    for (int q = 0; q < bk; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += X[i][q] * Y[q][j0 + e];
  double *A = mg->Mc;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (i >= bi || j0 + e >= bj) continue;
    double &o = A[(long long)(ti * IB + i) * m + tj * IB + j0 + e];
    o = src ? src[i * IB + j0 + e] : (tj == k ? 0.0 : o) - acc[e];
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static unsigned blocks_for(long long count, int per) { return (unsigned)((count + per - 1) / per); }

hipError_t mg_launch_elem1(const SlotDev *d_slot, const MgDev *d_mg, long long nn1, int prec, hipStream_t st) {
  const dim3 g(blocks_for(nn1, 256), 24);
  if (prec == 0) mg_elem1_kernel<double><<<g, 256, 0, st>>>(d_slot, d_mg);
  else mg_elem1_kernel<float><<<g, 256, 0, st>>>(d_slot, d_mg);
  return hipGetLastError();
}

// mixed precision only: level 1 has its element matrices in FP64 solves
hipError_t mg_launch_elem2(const SlotDev *d_slot, const MgDev *d_mg, long long nn2, hipStream_t st) {
  mg_g2_kernel<float><<<64, 192, 0, st>>>(d_mg);
  mg_elem2_kernel<float><<<dim3(blocks_for(nn2, 256), 24), 256, 0, st>>>(d_slot, d_mg);
  return hipGetLastError();
}

hipError_t mg_launch_elemc(const MgDev *d_mg, int l, long long nn_next, int prec, hipStream_t st) {
  const dim3 g(blocks_for(nn_next * 8, 256), 24);
  if (prec == 0) mg_elemc_kernel<double><<<g, 256, 0, st>>>(d_mg, l);
  else mg_elemc_kernel<float><<<g, 256, 0, st>>>(d_mg, l);
  return hipGetLastError();
}

size_t mg_inverse_scratch_bytes(int ndof) {
  const size_t nblk = (ndof + IB - 1) / IB;
  return sizeof(double) * ((2 * nblk + 1) * IB * IB + 1);
}

hipError_t mg_launch_coarse_inverse(const MgBatch &B, int ndof_max, int prec, hipStream_t st) {
  const dim3 ga(blocks_for(ndof_max, 4), 1, B.count);
  if (prec == 0) mg_inv_assemble_kernel<double><<<ga, 256, 0, st>>>(B);
  else mg_inv_assemble_kernel<float><<<ga, 256, 0, st>>>(B);
  const unsigned nblk = blocks_for(ndof_max, IB);
  for (unsigned k = 0; k < nblk; ++k) {
    mg_inv_panel_kernel<<<dim3(nblk, 1, B.count), 256, 0, st>>>(B, k);
    mg_inv_update_kernel<<<dim3(nblk, nblk, B.count), 256, 0, st>>>(B, k);
  }
  return hipGetLastError();
}

hipError_t mg_launch_stencil(const MgDev *d_mg, int l, long long nn, int prec, hipStream_t st) {
  const dim3 g(blocks_for(nn, 256), MG_HALF);
  if (prec == 0) mg_stencil_kernel<double><<<g, 256, 0, st>>>(d_mg, l);
  else mg_stencil_kernel<float><<<g, 256, 0, st>>>(d_mg, l);
  return hipGetLastError();
}

// whether a level takes the large-level form: two nodes per thread, or level 1
// in mixed precision from the moduli (the choice is made design by design: the
// sums run in another order)
bool mg_apply_wide(long long nn) { return nn > 32768; }

namespace {
template <typename T, int EP>
void launch_apply_ep(const MgBatch &B, int l, long long nn_max, bool wide, hipStream_t st, int live) {
  if (wide) {
    mg_apply_pair_kernel<T, EP><<<dim3(blocks_for(nn_max / 2, 256), 1, B.count), 256, 0, st>>>(B, l, live);
  } else if (nn_max > 4096) {
    constexpr int R = sizeof(T) == 4 ? NRHS : 2;  // FP64: six cases would not fit the registers
    mg_apply_split_kernel<T, R, 3, EP>
        <<<dim3(blocks_for(nn_max, 64), NRHS / R, B.count), 192, 0, st>>>(B, l, live);
  } else {
    mg_apply_split_kernel<T, 2, 9, EP>
        <<<dim3(blocks_for(nn_max, 64), NRHS / 2, B.count), 576, 0, st>>>(B, l, live);
  }
}
template <typename T>
void launch_apply(const MgBatch &B, int l, long long nn_max, bool wide, hipStream_t st, int live, int ep) {
  switch (ep) {
    case MGE_STEP1: launch_apply_ep<T, MGE_STEP1>(B, l, nn_max, wide, st, live); break;
    case MGE_RES: launch_apply_ep<T, MGE_RES>(B, l, nn_max, wide, st, live); break;
    case MGE_POST: launch_apply_ep<T, MGE_POST>(B, l, nn_max, wide, st, live); break;
    case MGE_LAST: launch_apply_ep<T, MGE_LAST>(B, l, nn_max, wide, st, live); break;
    default: launch_apply_ep<T, MGE_NONE>(B, l, nn_max, wide, st, live); break;
  }
}
}  // namespace

// nn_max: the largest of the level over the batch; wide: every design of the
// batch takes the two-nodes-per-thread form (mg_apply_wide), else none does
hipError_t mg_launch_apply(const MgBatch &B, int l, long long nn_max, bool wide, int prec,
                           hipStream_t st, int live, int ep) {
  if (prec == 0) launch_apply<double>(B, l, nn_max, wide, st, live, ep);
  else launch_apply<float>(B, l, nn_max, wide, st, live, ep);
  return hipGetLastError();
}

hipError_t mg_launch_restrict(const MgBatch &B, int l, long long nn_coarse_max, int prec,
                              hipStream_t st) {
  const dim3 g(blocks_for(nn_coarse_max, 256), NRHS, B.count);
  if (prec == 0) mg_restrict_kernel<double><<<g, 256, 0, st>>>(B, l);
  else mg_restrict_kernel<float><<<g, 256, 0, st>>>(B, l);
  return hipGetLastError();
}

hipError_t mg_launch_gather(const MgBatch &B, long long nn_coarse_max, hipStream_t st) {
  mg_gather_kernel<<<dim3(blocks_for(nn_coarse_max, 256), NRHS, B.count), 256, 0, st>>>(B);
  return hipGetLastError();
}

// bytes of a load case's restriction shares in the pre-smoothing pass (they
// take the place of its residual)
size_t mg_share_bytes(int n, int tz, int ntiles) {
  using TT = Tile<float>;
  return sizeof(float) * (size_t)ntiles * (tz / 2 + 1) * 3 * (TT::Y / 2 + 1) * (std::min(TT::X, n) / 2 + 1);
}

hipError_t mg_launch_prolong(const MgBatch &B, int l, long long nn_coarse_max, int prec, hipStream_t st) {
  const dim3 g(blocks_for(nn_coarse_max, 256), NRHS, B.count);
  if (prec == 0) mg_prolong_kernel<double><<<g, 256, 0, st>>>(B, l);
  else mg_prolong_kernel<float><<<g, 256, 0, st>>>(B, l);
  return hipGetLastError();
}

hipError_t mg_launch_coarsest(const MgBatch &B, int ndof_max, int prec, hipStream_t st) {
  const dim3 g(blocks_for(ndof_max, 16), 1, B.count);
  if (prec == 0) mg_coarsest_kernel<double><<<g, 256, 0, st>>>(B);
  else mg_coarsest_kernel<float><<<g, 256, 0, st>>>(B);
  return hipGetLastError();
}

hipError_t mg_launch_scalar(const MgBatch &B, int phase, hipStream_t st) {
  mg_scalar_kernel<<<dim3(NRHS, 1, B.count), VEC_THREADS, 0, st>>>(B, phase);
  return hipGetLastError();
}

// the start vector of level l (l = 1, 2, ... in turn), then step k of all levels;
// blocks_max: the most 64-node blocks over a design's levels; levels: the most levels
hipError_t mg_launch_power_init(const MgBatch &B, int l, long long nn_max, int prec, hipStream_t st) {
  const dim3 g(blocks_for(3 * nn_max, 256), 1, B.count);
  if (prec == 0) mg_power_init_kernel<double><<<g, 256, 0, st>>>(B, l);
  else mg_power_init_kernel<float><<<g, 256, 0, st>>>(B, l);
  return hipGetLastError();
}

hipError_t mg_launch_power(const MgBatch &B, int k, long long blocks_max, int levels, int prec, hipStream_t st) {
  const dim3 g((unsigned)blocks_max, 1, B.count), gr((unsigned)levels, 1, B.count);
  if (prec == 0) mg_power_step_kernel<double><<<g, 192, 0, st>>>(B, k);
  else mg_power_step_kernel<float><<<g, 192, 0, st>>>(B, k);
  mg_power_reduce_kernel<<<gr, VEC_THREADS, 0, st>>>(B);
  return hipGetLastError();
}

}  // namespace shh
